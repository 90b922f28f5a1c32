"""What setd_batch_info reports of a tile choice, given to setd_batch_set_tiles of
another batch of the same instances, is the same choice: the same report, and
steps with the same bits (the tile, and how many waves share its contraction,
decide the order of every sum).  Choices set by hand are reported as they were
set."""
import pytest

from tests.gpu_util import dev, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

SIZES = [(16, 24), (40, 33), (130, 64), (17, 80)]


def _batch():
    probs = [wl.schnakenberg_2d(n1, n2, dv=8.0 + k, instance=k, tau=1e-3) for k, (n1, n2) in enumerate(SIZES)]
    B = setd.Batch([p.dims for p in probs], [[[dev(M) for M in Ac] for Ac in p.A] for p in probs], probs[0].tau)
    u = torch().zeros(B.total, dtype=torch().float64, device="cuda")
    for b, p in enumerate(probs):
        for c in range(2):
            B.field(u, b, c).copy_(dev(p.U0[c]))
    return probs, B, u


def _steps(probs, B, u):
    B.step(u, 3, probs[0].g_kind, [p.params for p in probs])
    return u


@pytest.mark.parametrize("tiles", [("2x2x4", "4x2x2"), ("2x4x1", "2x2x1"), ("4x2x4", "2x4x1"), ("4x4x1", "4x2x4"),
                                   ("2x2x2", "4x4x1"), ("4x2x2", "2x2x4"), (None, None)])
def test_info_sets_the_same_choice(tiles, monkeypatch):
    probs, B, u = _batch()
    if tiles[0] is not None:
        monkeypatch.setenv("SETD_TILE_MODE1", tiles[0])
        monkeypatch.setenv("SETD_TILE_MODEB", tiles[1])
    info = B.tune()
    monkeypatch.delenv("SETD_TILE_MODE1", raising=False)
    monkeypatch.delenv("SETD_TILE_MODEB", raising=False)
    ref = _steps(probs, B, u)
    _, C, v = _batch()
    C.set_tiles(info["mode1"], info["modeB"])
    again = C.info()
    say("tiles", tiles, info, again)
    assert (again["mode1"], again["modeB"]) == (info["mode1"], info["modeB"]) and again["tuned"]
    assert torch().equal(_steps(probs, C, v), ref)


@pytest.mark.parametrize("mode1,modeB", [((2, 2, 0), (4, 4, 0)), ((4, 2, 2048), (2, 4, 8192)), ((4, 4, 1), (2, 2, 7)),
                                         ((2, 4, 2 ** 31 - 1), (4, 2, 2 ** 23))])
def test_choices_set_by_hand(mode1, modeB):
    probs, B, u = _batch()
    B.set_tiles(mode1, modeB)
    assert (B.info()["mode1"], B.info()["modeB"]) == (mode1, modeB)
    _, C, v = _batch()
    C.set_tiles(mode1[:2] + (0,), modeB[:2] + (0,))   # a cap changes no sum
    assert torch().equal(_steps(probs, B, u), _steps(probs, C, v))
