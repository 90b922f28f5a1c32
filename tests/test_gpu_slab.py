"""The one-pass product of modes 1 and 2 (a Tucker group's first two modes,
n1 <= 256) against the oracle, at the sizes where it can go wrong: fewer than
four blocks of i_1 (waves without work), block counts that leave waves or
workgroups a smaller share, contractions with remainders, one slab and many,
one and two terms, with and without a base.

Tolerance: three terms of up to 18 times their sum, products at 1e-13."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

TOL = 2e-12
# 3D: n1 over the block counts 1 .. 16, n2 below and past two column tiles;
# 2D (two terms, n <= 64)
SHAPES = [(2, 5, 3), (16, 16, 4), (17, 33, 2), (48, 40, 3), (63, 64, 2), (65, 31, 9), (80, 80, 5), (113, 100, 2),
          (128, 70, 40), (129, 17, 3), (150, 49, 2), (193, 130, 2), (200, 9, 3), (256, 40, 2), (241, 300, 2),
          (2, 2), (5, 64), (16, 17), (33, 50), (64, 64), (64, 3)]


@pytest.mark.parametrize("dims", SHAPES)
def test_modes_1_and_2_in_one_pass(dims):
    prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
    ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau)
    bank = oracle.PhiBank(prob.A[1], prob.tau)
    V, W0 = wl.random_tensor(dims, 5), wl.random_tensor(dims, 6)
    for ell, stage, key in ((1, setd.STAGE_2, 2), (2, setd.STAGE_F, "f")):
        ref = bank.split_apply(ell, key, V)
        W = dev(W0)
        say("one pass", dims, ell)
        ctx.split_phi_apply(1, ell, stage, dev(V), W, scale=0.3, beta=1.0)
        assert rel_err(host(W, dims), 0.3 * ref + W0) < TOL, (dims, ell)
        ctx.split_phi_apply(1, ell, stage, dev(V), W)
        assert rel_err(host(W, dims), ref) < TOL, (dims, ell)


@pytest.mark.parametrize("dims", [(2, 2), (16, 8), (33, 17), (64, 64), (65, 100), (130, 7), (200, 40), (256, 31), (300, 9),
                                  (20, 9, 30), (40, 50, 3), (100, 37, 20), (17, 33, 5, 4), (3, 64, 90)])
@pytest.mark.parametrize("own", [True, False])
def test_matrices_as_given(dims, own):
    """Tucker operators that read their matrices unpacked: one pass or single
    products, every subset of modes, with and without the caller's workspace.
    n <= 300 products of uniform entries: 1e-13 of the largest result."""
    T, W0 = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2)
    Ls = [wl.random_matrix(n, 3 + k, scale=0.3) for k, n in enumerate(dims)]
    ws = None if own else torch().empty(setd.tucker_workspace_bytes(dims) // 8 + 1, dtype=torch().float64, device="cuda")
    d = len(dims)
    for mask in range(1, 2 ** d):
        mats = [Ls[mu] if mask >> mu & 1 else None for mu in range(d)]
        ref = T
        for mu in range(d):
            if mats[mu] is not None:
                ref = oracle.mode_product(ref, mats[mu], mu + 1)
        for alpha, beta in ((1.0, 0.0), (-0.7, 1.0), (0.5, 0.25)):
            W = dev(W0)
            say("as given", dims, mask, alpha, beta)
            setd.tucker_apply(dev(T), W, dims, [None if L is None else dev(L) for L in mats], alpha=alpha, beta=beta,
                              workspace=ws)
            assert rel_err(host(W, dims), alpha * ref + beta * W0) < 1e-13, (dims, mask, alpha, beta)


def test_matrix_inside_the_result():
    """A matrix that lies in W's memory is used as it was before the call."""
    dims = (40, 30)
    T = wl.random_tensor(dims, 1)
    L = [wl.random_matrix(40, 2), wl.random_matrix(30, 3)]
    W = dev(wl.random_tensor(dims, 4))
    W[:900].copy_(dev(L[1]))
    setd.tucker_apply(dev(T), W, dims, [dev(L[0]), W[:900]])
    assert rel_err(host(W, dims), oracle.tucker(T, L)) < 1e-13
