"""Calls on a card with little memory left, while the library keeps memory that
it could do without (destroyed contexts' blocks, the idle workspace of phi
builds): an allocation that would fail takes that first, so that every call that
fits into what is free and kept succeeds, with the same bits as before."""
import contextlib

import numpy as np
import pytest

from tests.gpu_util import dev, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402
from paper_2310_07551_amd import _lib   # noqa: E402

MIB = 1 << 20
DIMS = (64, 96, 128)


def _free():
    torch().cuda.synchronize()
    torch().cuda.empty_cache()
    return torch().cuda.mem_get_info()[0]


def _release():
    _lib.check(_lib.load().setd_release_workspace())


@contextlib.contextmanager
def _left(mib):
    """Holds all but about `mib` MiB of the card."""
    hold, free = [], _free()
    try:
        while free > (mib + 24) * MIB:   # one large allocation leaves more free than it seems
            hold.append(torch().empty(free - mib * MIB, dtype=torch().uint8, device="cuda"))
            free = torch().cuda.mem_get_info()[0]
        say("free", free // MIB, "MiB")
        yield
    finally:
        hold.clear()
        torch().cuda.empty_cache()


def _context():
    prob = wl.fhn_3d(dims=DIMS)
    return setd.Context(DIMS, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau)


def _keep():
    """A destroyed context's memory in the library's list; returns its bytes."""
    _release()
    before = _free()
    _context().close()
    kept = before - _free()
    say("kept", kept // MIB, "MiB")
    assert kept > 300 * MIB
    return kept


def _phi(n, ell):
    A = dev(wl.neumann_d2(n))
    out = torch().empty((ell + 1) * n * n, dtype=torch().float64, device="cuda")
    st = torch().cuda.current_stream().cuda_stream
    return out, lambda: _lib.check(_lib.load().setd_phi_matrices(A.data_ptr(), n, 1e-6, ell, out.data_ptr(), st))


@pytest.mark.parametrize("n,ell,mib", [(1024, 4, 100),    # 285 MB, more than the kept workspace of phi builds holds
                                       (1024, 1, 60)])    # 184 MB, the kept workspace grows
def test_phi_build(n, ell, mib):
    out, call = _phi(n, ell)
    call()
    ref = out.cpu()
    out.zero_()
    _keep()
    with _left(mib):
        say("phi", n, ell)
        call()
        assert torch().equal(out.cpu(), ref)


def test_tucker_workspace():
    dims = (260, 240, 300)   # two intermediates of 150 MB, packed matrices
    T = torch().rand(int(np.prod(dims)), dtype=torch().float64, device="cuda")
    W = torch().empty_like(T)
    mats = [dev(wl.random_matrix(n, 3 + k, scale=0.1)) for k, n in enumerate(dims)]
    setd.tucker_apply(T, W, dims, mats)
    ref = W.cpu()
    W.zero_()
    _keep()
    with _left(60):
        say("tucker", dims)
        setd.tucker_apply(T, W, dims, mats)
        assert torch().equal(W.cpu(), ref)


def test_raw_tucker_workspace():
    dims = (40, 50, 4000)   # matrices read as given, one intermediate of 64 MB
    T = torch().rand(int(np.prod(dims)), dtype=torch().float64, device="cuda")
    W = torch().empty_like(T)
    mats = [dev(wl.random_matrix(n, 3 + k, scale=0.1)) for k, n in enumerate(dims)]
    setd.tucker_apply(T, W, dims, mats)
    ref = W.cpu()
    W.zero_()
    _keep()
    with _left(24):
        say("raw tucker", dims)
        setd.tucker_apply(T, W, dims, mats)
        assert torch().equal(W.cpu(), ref)


def test_context_takes_the_idle_phi_workspace():
    _release()
    before = _free()
    ctx = _context()
    need = before - _free()
    ctx.close()
    _release()
    out, call = _phi(1024, 1)
    call()   # leaves 184 MB with the library
    prob = wl.fhn_3d(dims=DIMS)
    A = [[dev(M) for M in Ac] for Ac in prob.A]
    with _left(need // MIB - 60):
        say("context of", need // MIB, "MiB")
        ctx = setd.Context(DIMS, A, prob.tau)
        ctx.close()


def test_too_little_is_an_error_and_the_next_call_works():
    out, call = _phi(1024, 4)
    _release()
    with _left(60):
        with pytest.raises(setd.SetdError) as ei:
            call()
        assert ei.value.code == _lib.SETD_ENOMEM
    call()
    _lib.check(_lib.load().setd_sync(None))   # the error of the failed call is not reported again

