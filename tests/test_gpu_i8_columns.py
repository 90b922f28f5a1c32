"""The int8 slicing form where the columns of all slabs are taken in a row:
slabs that end inside a group of 128 columns and inside a workgroup of 32
fibres, contractions around every run of 16 and k-step of 64 up to the one
chunk of 256 and past it, a single slab, and a non-finite fibre at a slab's
end.  Tolerance: 1e-7 of the largest entry, the form's kernel bound (each
operand is rounded to 30 bits; about sqrt(n) 2^-29 of it)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

TOL = 1e-7


@pytest.mark.parametrize("dims", [(5, 15, 40), (31, 16, 9), (33, 17, 18), (130, 48, 5), (127, 63, 7), (3, 64, 129),
                                  (20, 65, 33), (9, 241, 16), (17, 255, 6), (40, 256, 10), (12, 257, 11), (1, 100, 70),
                                  (70, 1, 30), (129, 2, 255)])
def test_columns_of_all_slabs(dims):
    T, W0 = wl.random_tensor(dims, 2), wl.random_tensor(dims, 3)
    Ls = [wl.random_matrix(n, 20 + k, scale=1.0 / np.sqrt(n)) for k, n in enumerate(dims)]
    for mats in ([None, dev(Ls[1]), None], [None, None, dev(Ls[2])], [dev(L) for L in Ls]):
        ref = T
        for k in range(3):
            if mats[k] is not None:
                ref = oracle.mode_product(ref, Ls[k], k + 1)
        W = dev(W0)
        setd.tucker_apply(dev(T), W, dims, mats, alpha=0.7, beta=1.0, prec=setd.PREC_I8X4)
        e = rel_err(host(W, dims) - W0, 0.7 * ref)
        say("i8 columns", dims, [m is not None for m in mats], "rel_inf %.2e" % e)
        assert e < TOL, dims


def test_nonfinite_fibre_at_a_slab_end():
    dims = (33, 20, 6)
    T = wl.random_tensor(dims, 4)
    T[32, 7, 2] = np.inf
    L = wl.random_matrix(20, 5, scale=0.2)
    W = torch().empty(int(np.prod(dims)), dtype=torch().float64, device="cuda")
    setd.tucker_apply(dev(T), W, dims, [None, dev(L), None], prec=setd.PREC_I8X4)
    got = host(W, dims)
    bad = ~np.isfinite(got)
    assert bad[32, :, 2].all()
    bad[32, :, 2] = False
    assert not bad.any()
