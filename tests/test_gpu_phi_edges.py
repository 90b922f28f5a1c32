"""phi builds at the edges of the 16 x 16 tiles and of the algorithm: sizes
around a tile, every order, no squaring, one, and many; the kept workspace
between calls that grow, shrink, release it, or run from two threads at once.

Tolerance: a few FP64 ulps of the largest entry against the oracle's exact
spectral evaluation (as for the Neumann matrices elsewhere), 1e-15."""
import ctypes
import threading

import pytest

import oracle
from tests.gpu_util import dev, rel_err, say, torch
from workloads import neumann_d2

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402
from paper_2310_07551_amd import _lib   # noqa: E402


def _check(got, A, tau, ell):
    n = A.shape[0]
    ref = oracle.phi_all(tau * A, ell)
    for k in range(ell + 1):
        assert rel_err(got[k].cpu().numpy().reshape(n, n, order="F"), ref[k]) < 1e-15, (n, tau, k)


@pytest.mark.parametrize("n", [2, 3, 15, 16, 17, 31, 33, 64, 65, 130])
def test_sizes_orders_squarings(n):
    A = neumann_d2(n)
    norm = abs(A).sum(0).max()
    for ell in (0, 1, 2, 4):
        for tau in (0.7 / norm, 1.5 / norm, 300.0 / norm, 0.0):
            say("phi edges", n, ell, tau)
            _check(setd.phi_matrices(dev(A), tau, ell), A, tau, ell)


def test_workspace_is_kept_and_released():
    A, B = neumann_d2(200), neumann_d2(40)
    for M in (A, B, A):
        _check(setd.phi_matrices(dev(M), 1e-3, 2), M, 1e-3, 2)
    _lib.check(_lib.load().setd_release_workspace())
    _check(setd.phi_matrices(dev(B), 1e-2, 3), B, 1e-2, 3)
    _lib.check(_lib.load().setd_release_workspace())
    assert _lib.load().setd_sync(ctypes.c_void_p(0)) == 0


def test_two_threads_build_at_once():
    mats = [neumann_d2(96), neumann_d2(130)]
    devs = [dev(M) for M in mats]
    torch().cuda.synchronize()
    out = [[], []]

    def work(k):
        s = torch().cuda.Stream()
        with torch().cuda.stream(s):
            for _ in range(6):
                out[k].append(setd.phi_matrices(devs[k], 1e-3, 2))
        s.synchronize()

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for k in range(2):
        _check(out[k][0], mats[k], 1e-3, 2)
        assert all(torch().equal(o, out[k][0]) for o in out[k])
