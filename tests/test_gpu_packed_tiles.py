"""Every tile of the FP64 kernels on packed matrices, which contexts use, forced
by SETD_TILE_MODE1 / SETD_TILE_MODEB on grids that the one-pass kernels leave to
them: 2D with a side above 64 (mode 1, sums of two terms) and thin 3D grids of
more than 256 rows (mode 1, mode 2 over several slabs whose columns are and are
not neighbours, sums of three terms); n below, at and past whole chunks of 8. A
NaN in what a result is added to stays in its entry.

Tolerance: products at 1e-13 and sums of terms of up to 18 times the result."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

TILES = ["1x1x4", "1x4x1", "2x2x4", "2x2x2", "2x2x1", "4x2x4", "4x2x2", "4x2x1", "5x2x4", "5x2x1", "7x1x4", "7x2x1",
         "4x4x1"]
GRIDS = [(65, 47), (113, 70), (72, 5), (7, 130), (260, 9, 5), (261, 9, 5), (264, 16, 3), (257, 3, 20)]


@pytest.fixture(scope="module")
def problems():
    out = []
    for dims in GRIDS:
        prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
        ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau)
        V, W0 = wl.random_tensor(dims, 5), wl.random_tensor(dims, 6)
        bank = oracle.PhiBank(prob.A[1], prob.tau)
        out.append((dims, ctx, V, W0, bank.split_apply(2, "f", V), bank.split_apply(1, 2, V)))
    return out


@pytest.mark.parametrize("tile", TILES)
def test_every_tile(problems, tile, monkeypatch):
    monkeypatch.setenv("SETD_TILE_MODE1", tile)
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for dims, ctx, V, W0, ref2, ref1 in problems:
        say("packed tile", tile, dims)
        W = dev(W0)
        ctx.split_phi_apply(1, 2, setd.STAGE_F, dev(V), W, scale=0.3, beta=1.0)
        assert rel_err(host(W, dims), 0.3 * ref2 + W0) < 2e-12, dims
        W.fill_(float("nan"))
        ctx.split_phi_apply(1, 1, setd.STAGE_2, dev(V), W)
        assert rel_err(host(W, dims), ref1) < 2e-12, dims


@pytest.mark.parametrize("tile", TILES)
def test_nan_in_the_base_stays(problems, tile, monkeypatch):
    monkeypatch.setenv("SETD_TILE_MODE1", tile)
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for dims, ctx, V, W0, ref2, _ in problems:
        for at in (tuple(n - 1 for n in dims), (0,) * len(dims), (dims[0] - 1,) + (0,) * (len(dims) - 1)):
            B = W0.copy()
            B[at] = np.nan
            W = dev(B)
            ctx.split_phi_apply(1, 2, setd.STAGE_F, dev(V), W, scale=0.3, beta=1.0)
            assert np.array_equal(np.isnan(host(W, dims)), np.isnan(B)), (tile, dims, at)
