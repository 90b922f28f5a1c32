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


F32_TILES = ["1x1", "2x2", "4x2", "4x4", "5x2", "5x4", "7x2", "8x2"]


def test_every_f32_tile_same_bits(monkeypatch):
    """The FP32 kernels form every sum in an order that depends on the mode and
    the size alone: every tile gives the same bits, with neighbouring columns
    that end inside a slab (n1 odd, even, a multiple of 4), fewer columns than
    a tile's lane holds, and remainders of 16 of every kind.  Against the
    oracle 1e-5 of the largest entry (2^-24 times sums of up to 300 terms)."""
    for dims in [(3, 5, 2), (16, 16, 16), (31, 100, 5), (34, 9, 33), (113, 7, 1), (1, 300, 2), (300, 1, 3), (65, 47, 3),
                 (64, 130, 18), (129,), (2, 2), (300, 50)]:
        T, W0 = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2)
        Ls = [wl.random_matrix(n, 3 + k, scale=1.0 / np.sqrt(n)) for k, n in enumerate(dims)]
        ref = 0.7 * oracle.tucker(T, Ls) + W0
        first = None
        for tile in F32_TILES:
            monkeypatch.setenv("SETD_TILE_F32_MODE1", tile)
            monkeypatch.setenv("SETD_TILE_F32_MODEB", tile)
            W = dev(W0)
            setd.tucker_apply(dev(T), W, dims, [dev(L) for L in Ls], alpha=0.7, beta=1.0, prec=setd.PREC_F32)
            got = host(W, dims)
            say("f32 tile", tile, dims, "rel_inf %.2e" % rel_err(got, ref))
            assert rel_err(got, ref) < 1e-5, (tile, dims)
            first = got if first is None else first
            assert np.array_equal(got, first), (tile, dims)


@pytest.mark.parametrize("dims", [(33, 50), (21, 18, 17), (20, 18, 40)])
def test_every_f32_tile_sums_terms(dims, monkeypatch):
    """As above for the sums of terms of a step: the same bits with every tile."""
    prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
    ref = oracle.integrate(prob.U0, prob.A, prob.tau, 2, prob.g_kind, prob.params)
    first = None
    for tile in F32_TILES:
        monkeypatch.setenv("SETD_TILE_F32_MODE1", tile)
        monkeypatch.setenv("SETD_TILE_F32_MODEB", tile)
        ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau, setd.PREC_F32)
        u = torch().cat([dev(f) for f in prob.U0])
        ctx.step(u, 2, prob.g_kind, prob.params)
        got = u.cpu().numpy()
        first = got if first is None else first
        assert np.array_equal(got, first), tile
    for c in range(2):
        e = rel_err(first[c * ctx.N:(c + 1) * ctx.N], np.asarray(ref[c]).ravel(order="F"))
        say("f32 terms", dims, "field", c, "rel_inf %.2e" % e)
        assert e < 1e-3   # the error of FP32 products over a step is checked elsewhere


@pytest.mark.parametrize("prec,tol", [(setd.PREC_BF16X3, 1e-5), (setd.PREC_BF16X2, 1e-3)])
def test_every_bf16_tile_same_bits(prec, tol, monkeypatch):
    """The bf16 forms as the FP32 ones: the same bits with every tile, single
    products and sums of terms.  Against the oracle 1e-5 for three pieces
    (about FP32), 1e-3 for two (2^-16 times sums of up to 300 terms)."""
    tiles = ["1x1", "2x2", "4x2", "4x4"]
    for dims in [(3, 5, 2), (32, 32, 32), (31, 100, 5), (34, 9, 33), (113, 7, 1), (1, 300, 2), (33, 50), (64, 130, 18),
                 (129,), (2, 2), (65, 47, 3)]:
        T, W0 = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2)
        Ls = [wl.random_matrix(n, 3 + k, scale=1.0 / np.sqrt(n)) for k, n in enumerate(dims)]
        ref = 0.7 * oracle.tucker(T, Ls) + W0
        first = None
        for tile in tiles:
            monkeypatch.setenv("SETD_TILE_BF16_MODE1", tile)
            monkeypatch.setenv("SETD_TILE_BF16_MODEB", tile)
            W = dev(W0)
            setd.tucker_apply(dev(T), W, dims, [dev(L) for L in Ls], alpha=0.7, beta=1.0, prec=prec)
            got = host(W, dims)
            say("bf16 tile", tile, dims, "rel_inf %.2e" % rel_err(got, ref))
            assert rel_err(got, ref) < tol, (tile, dims)
            first = got if first is None else first
            assert np.array_equal(got, first), (tile, dims)
    for dims in [(33, 50), (21, 18, 17)]:
        prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
        first = None
        for tile in tiles:
            monkeypatch.setenv("SETD_TILE_BF16_MODE1", tile)
            monkeypatch.setenv("SETD_TILE_BF16_MODEB", tile)
            ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau, prec)
            u = torch().cat([dev(f) for f in prob.U0])
            ctx.step(u, 2, prob.g_kind, prob.params)
            got = u.cpu().numpy()
            first = got if first is None else first
            assert np.isfinite(got).all() and np.array_equal(got, first), tile
