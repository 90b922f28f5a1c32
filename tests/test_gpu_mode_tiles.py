"""Every tile of the FP64 mode-product kernels (SETD_TILE_MODE1 / SETD_TILE_MODEB
force one) against the oracle, at the sizes where a tile can go wrong:
contractions shorter than a chunk of 8, of exactly whole chunks and with every
kind of remainder, extents below one block of 16 and one past it, several
slabs per tile, tensors that are only 8-byte aligned, sums of several terms.

Tolerance: the products' 1e-13 of the largest entry (n <= 300 products of
uniform entries, each rounded to 2^-53)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

TOL = 1e-13
TILES = ["1x1x4", "2x2x4", "2x2x2", "2x2x1", "4x2x4", "4x2x2", "4x2x1", "5x2x4", "5x2x1", "7x1x4", "7x2x1", "4x4x1"]
SHAPES = [(3, 5, 2), (8, 16, 3), (17, 9, 4), (16, 33, 2), (31, 100, 5), (113, 7, 1), (1, 300, 2), (300, 1, 3),
          (65, 47, 3)]


@pytest.mark.parametrize("tile", TILES)
def test_every_tile(tile, monkeypatch):
    monkeypatch.setenv("SETD_TILE_MODE1", tile)
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for dims in SHAPES:
        say("tile", tile, dims)
        T, W0 = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2)
        Ls = [wl.random_matrix(n, 3 + k, scale=0.3) for k, n in enumerate(dims)]
        N = int(np.prod(dims))
        V = torch().empty(N + 1, dtype=torch().float64, device="cuda")[1:]   # 8-byte aligned only
        V.copy_(dev(T))
        W = torch().empty(N + 1, dtype=torch().float64, device="cuda")[1:]
        W.copy_(dev(W0))
        setd.tucker_apply(V, W, dims, [dev(L) for L in Ls], alpha=0.7, beta=1.0)
        assert rel_err(host(W, dims), 0.7 * oracle.tucker(T, Ls) + W0) < TOL, dims
        for mu in range(3):
            mats = [None] * 3
            mats[mu] = dev(Ls[mu])
            setd.tucker_apply(V, W, dims, mats)
            assert rel_err(host(W, dims), oracle.mode_product(T, Ls[mu], mu + 1)) < TOL, (dims, mu)


@pytest.mark.parametrize("tile", TILES)
def test_every_tile_sums_terms(tile, monkeypatch):
    """The terms of a split action summed along the contraction (two and three
    terms, whose parts may split between waves), with a non-finite input
    confined to what depends on it."""
    for dims in [(12, 10), (33, 50), (9, 21, 17), (20, 18, 40)]:
        prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
        ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau)
        bank = oracle.PhiBank(prob.A[1], prob.tau)
        V, W0 = wl.random_tensor(dims, 5), wl.random_tensor(dims, 6)
        monkeypatch.setenv("SETD_TILE_MODE1", tile)
        monkeypatch.setenv("SETD_TILE_MODEB", tile)
        W = dev(W0)
        say("terms", tile, dims)
        ctx.split_phi_apply(1, 2, setd.STAGE_F, dev(V), W, scale=0.3, beta=1.0)
        # three terms of up to 18 times the sum
        assert rel_err(host(W, dims), 0.3 * bank.split_apply(2, "f", V) + W0) < 20 * TOL, dims


@pytest.mark.parametrize("tile", TILES)
def test_nonfinite_stays_in_its_fibre(tile, monkeypatch):
    """A NaN in one fibre reaches that fibre's results and no others (the
    clamped and masked loads never multiply another fibre's values)."""
    monkeypatch.setenv("SETD_TILE_MODE1", tile)
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    dims = (21, 19, 5)
    T = wl.random_tensor(dims, 9)
    T[20, 18, 2] = np.nan
    for mu in range(3):
        n = dims[mu]
        mats = [None] * 3
        mats[mu] = dev(wl.random_matrix(n, 4))
        W = torch().empty(T.size, dtype=torch().float64, device="cuda")
        setd.tucker_apply(dev(T), W, dims, mats)
        bad = np.zeros(dims, dtype=bool)
        at = [20, 18, 2]
        at[mu] = slice(None)
        bad[tuple(at)] = True
        assert np.array_equal(np.isnan(host(W, dims)), bad), (tile, mu)


@pytest.mark.parametrize("tile", ["2x2x4", "2x2x2", "2x2x1", "2x4x1", "4x2x4", "4x2x2", "4x2x1", "4x4x1"])
def test_every_tile_of_the_batch(tile, monkeypatch):
    """The tiles that the batched integrator tries, whose waves may split the
    contraction, over instances of unequal size (the last round of a workgroup
    has waves without a tile), in two and three dimensions.  Tolerance: the
    batched integrator's 1e-12 of the largest value."""
    monkeypatch.setenv("SETD_TILE_MODE1", tile)
    monkeypatch.setenv("SETD_TILE_MODEB", tile)
    for probs in ([wl.schnakenberg_2d(n1, n2, instance=q, tau=1e-3)
                   for q, (n1, n2) in enumerate([(16, 24), (7, 9), (33, 47), (128, 50), (2, 65)])],
                  [wl.fhn_3d(dims=dims) for dims in [(5, 18, 9), (33, 16, 17)]]):
        B = setd.Batch([p.dims for p in probs], [[[dev(M) for M in Ac] for Ac in p.A] for p in probs], probs[0].tau)
        info = B.tune()
        say("batch tile", tile, info)
        u = torch().zeros(B.total, dtype=torch().float64, device="cuda")
        for q, p in enumerate(probs):
            for c in range(2):
                B.field(u, q, c).copy_(dev(p.U0[c]))
        B.step(u, 3, probs[0].g_kind, [p.params for p in probs])
        for q, p in enumerate(probs):
            ref = oracle.integrate(p.U0, p.A, p.tau, 3, p.g_kind, p.params)
            for c in range(2):
                assert rel_err(host(B.field(u, q, c), p.dims), ref[c]) < 1e-12, (p.dims, c)
