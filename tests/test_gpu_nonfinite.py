"""NaN and infinities in the one-pass kernels: in a slab they stay in that slab,
in a matrix's row or column they reach what that row or column enters, as the
plain products say; in a fused 2D step they stay in their component when nothing
couples the two. And the fused steps of one component and of dense matrices
against the oracle and against the steps that are not fused.

Tolerance: the integrator's 1e-12."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402


@pytest.mark.parametrize("dims", [(40, 30, 9), (64, 64, 5), (65, 17, 4), (130, 20, 3), (200, 40, 2), (256, 9, 7)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_tensor_in_one_slab(dims, bad):
    T = wl.random_tensor(dims, 1)
    Ls = [wl.random_matrix(dims[0], 2), wl.random_matrix(dims[1], 3)]
    for at in ((dims[0] - 1, dims[1] - 1, 1), (0, 0, 0), (dims[0] // 2, 0, dims[2] - 1)):
        X = T.copy()
        X[at] = bad
        W = torch().empty(T.size, dtype=torch().float64, device="cuda")
        say("nonfinite slab", dims, bad, at)
        setd.tucker_apply(dev(X), W, dims, [dev(Ls[0]), dev(Ls[1]), None])
        want = np.zeros(dims, dtype=bool)
        want[:, :, at[2]] = True
        got = host(W, dims)
        assert np.array_equal(~np.isfinite(got), want), at
        X[at] = T[at]
        X[:, :, at[2]] = 0.0
        ref = oracle.mode_product(oracle.mode_product(X, Ls[0], 1), Ls[1], 2)
        assert rel_err(np.where(want, 0.0, got), ref) < 1e-13


@pytest.mark.parametrize("dims", [(40, 30, 3), (64, 64), (130, 20, 2), (17, 33)])
def test_matrix(dims):
    """Positive data: an infinite entry of a matrix gives +inf in every result
    that its row forms (mode 1: row i; mode 2: row j), and no other."""
    rng = np.random.default_rng(4)
    T = rng.uniform(0.5, 1.0, dims)
    for mu in (0, 1):
        for at in ((dims[mu] - 1, dims[mu] - 1), (0, dims[mu] - 1), (dims[mu] // 2, 0)):
            Ls = [rng.uniform(0.5, 1.0, (n, n)) for n in dims[:2]]
            Ls[mu][at] = np.inf
            W = torch().empty(T.size, dtype=torch().float64, device="cuda")
            say("nonfinite matrix", dims, mu, at)
            setd.tucker_apply(dev(T), W, dims, [dev(L) for L in Ls] + [None] * (len(dims) - 2))
            want = np.zeros(dims, dtype=bool)
            want[(at[0],) if mu == 0 else (slice(None), at[0])] = True
            got = host(W, dims)
            assert np.array_equal(np.isposinf(got), want) and np.isfinite(got[~want]).all(), (mu, at)


@pytest.mark.parametrize("dims", [(16, 16), (33, 17), (64, 64), (5, 60)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_fused_step_keeps_the_components_apart(dims, bad):
    p = wl.schnakenberg_2d(*dims)
    A = [[dev(M) for M in Ac] for Ac in p.A]
    clean = torch().cat([dev(f) for f in p.U0])
    N = dims[0] * dims[1]
    ref = clean.clone()
    setd.Context(dims, A, p.tau).step(ref, 2, wl.G_NONE, ())
    for c in (0, 1):
        for at in (0, N - 1, N // 2):
            u = clean.clone()
            u[c * N + at] = bad
            setd.Context(dims, A, p.tau).step(u, 2, wl.G_NONE, ())
            say("fused step", dims, bad, c, at)
            assert not torch().isfinite(u[c * N:(c + 1) * N]).any()
            assert torch().equal(u[(1 - c) * N:(2 - c) * N], ref[(1 - c) * N:(2 - c) * N])


def _compare(ctx, u0, g_kind, params, steps):
    """The fused steps and the recorded ones, which form F, G and the stage
    differences in kernels of their own."""
    u, v = u0.clone(), u0.clone()
    rec = torch().empty(6 * u.numel(), dtype=torch().float64, device="cuda")
    ctx.step(u, steps, g_kind, params)
    for _ in range(steps):
        ctx.step_record(v, rec, g_kind, params)
    assert rel_err(u.cpu().numpy(), v.cpu().numpy()) < 1e-14
    return u.cpu().numpy()


@pytest.mark.parametrize("dims", [(2, 3), (16, 16), (17, 33), (48, 50), (64, 64)])
@pytest.mark.parametrize("dense", [False, True])
def test_one_component(dims, dense):
    """No reaction; the oracle's step takes two components, so it runs the field
    twice."""
    rng = np.random.default_rng(8)
    A = [wl.neumann_d2(n) for n in dims]
    if dense:
        for mu, n in enumerate(dims):
            E = rng.standard_normal((n, n))
            A[mu] = A[mu] - 5.0 * (E @ E.T) / n
    U0 = wl.random_tensor(dims, 20)
    ctx = setd.Context(dims, [[dev(M) for M in A]], 1e-3)
    got = _compare(ctx, dev(U0), wl.G_NONE, (), 3)
    ref = oracle.integrate([U0, U0.copy()], [A, A], 1e-3, 3, wl.G_NONE, ())
    e = rel_err(got, np.asarray(ref[0]).ravel(order="F"))
    say("one component", dims, dense, "rel_inf %.2e" % e)
    assert e < 1e-12


@pytest.mark.parametrize("dims", [(3, 2), (16, 48), (33, 17), (64, 64)])
def test_dense_matrices(dims):
    p = wl.schnakenberg_2d(*dims)
    rng = np.random.default_rng(9)
    for c in range(2):
        for mu, n in enumerate(dims):
            E = rng.standard_normal((n, n))
            p.A[c][mu] = p.A[c][mu] - 5.0 * (E @ E.T) / n
    ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in p.A], p.tau)
    got = _compare(ctx, torch().cat([dev(f) for f in p.U0]), p.g_kind, p.params, 3)
    ref = oracle.integrate(p.U0, p.A, p.tau, 3, p.g_kind, p.params)
    for c in range(2):
        e = rel_err(got[c * ctx.N:(c + 1) * ctx.N], np.asarray(ref[c]).ravel(order="F"))
        say("dense", dims, "field", c, "rel_inf %.2e" % e)
        assert e < 1e-12
