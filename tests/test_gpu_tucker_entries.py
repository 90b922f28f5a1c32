"""The Tucker operator through its three entries (the library's workspace, the
caller's, the scratch array of setd_tucker_apply_noalloc) gives the same bits:
which kernels run depends on the sizes alone.  Few slabs, where one pass
competes with two products, on both sides of that choice (FP64); one, two and
all modes applied."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402


@pytest.mark.parametrize("dims", [(64, 64), (96, 96), (128, 128), (160, 160), (200, 64), (200, 100), (256, 64), (64, 1000),
                                  (250, 100), (200, 200), (64, 64, 16), (128, 128, 4), (160, 160, 3), (90, 20, 9),
                                  (16, 3, 200)])
def test_same_bits(dims):
    d = len(dims)
    T, W0 = wl.random_tensor(dims, 1), wl.random_tensor(dims, 2)
    Ls = [wl.random_matrix(n, 3 + k, scale=0.3) for k, n in enumerate(dims)]
    ws = torch().empty(setd.tucker_workspace_bytes(dims) // 8 + 1, dtype=torch().float64, device="cuda")
    for mask in ([2 ** d - 1, 3] if d == 3 else [3]):
        mats = [Ls[mu] if mask >> mu & 1 else None for mu in range(d)]
        ref = T
        for mu in range(d):
            if mats[mu] is not None:
                ref = oracle.mode_product(ref, mats[mu], mu + 1)
        for alpha, beta in ((1.0, 0.0), (-0.7, 1.0)):
            dm = [None if L is None else dev(L) for L in mats]
            Wa, Wb, Wc = dev(W0), dev(W0), dev(W0)
            setd.tucker_apply(dev(T), Wa, dims, dm, alpha=alpha, beta=beta)
            setd.tucker_apply(dev(T), Wb, dims, dm, alpha=alpha, beta=beta, workspace=ws)
            setd.tucker_apply_noalloc(dev(T), Wc, dims, dm, alpha=alpha, beta=beta)
            say("entries", dims, mask, alpha, beta)
            assert rel_err(host(Wa, dims), alpha * ref + beta * W0) < 1e-13
            assert torch().equal(Wa, Wb), (dims, mask, "workspace")
            assert torch().equal(Wa, Wc), (dims, mask, "noalloc")


@pytest.mark.parametrize("dims", [(40, 30, 20), (60, 50, 40), (24, 24, 24, 8)])
def test_matrices_inside_the_workspace(dims):
    """Matrices that lie where a call keeps its intermediates are used as they
    were before the call."""
    T = wl.random_tensor(dims, 1)
    Ls = [wl.random_matrix(n, 3 + k, scale=0.3) for k, n in enumerate(dims)]
    ws = torch().zeros(setd.tucker_workspace_bytes(dims) // 8 + 1, dtype=torch().float64, device="cuda")
    mats, at = [], 0
    N = int(np.prod(dims))
    for L in Ls:   # one after another from the start of the first intermediate
        mats.append(ws[at:at + L.size])
        mats[-1].copy_(dev(L))
        at += L.size
    assert at <= 2 * N
    W = torch().empty(N, dtype=torch().float64, device="cuda")
    setd.tucker_apply(dev(T), W, dims, mats, workspace=ws)
    assert rel_err(host(W, dims), oracle.tucker(T, Ls)) < 1e-13
