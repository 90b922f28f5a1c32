"""Memory of destroyed contexts that the library keeps for later ones: contexts
of every arithmetic built in memory that is full of NaN from an earlier one
agree with the oracle (nothing relies on cleared memory), several threads make
and drop contexts at once, and setd_release_workspace gives the memory back.
Tolerances: the arithmetics' own, 1e-12 (FP64) and 1e-5."""
import threading

import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err, rel_l2, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402
from paper_2310_07551_amd import _lib   # noqa: E402


def _run(prob, dims, prec, steps, nan=False):
    ctx = setd.Context(dims, [[dev(M) for M in Ac] for Ac in prob.A], prob.tau, prec)
    u = torch().cat([dev(f) for f in prob.U0])
    if nan:
        u.fill_(float("nan"))
    ctx.step(u, steps, prob.g_kind, prob.params)
    out = u.cpu().numpy()
    ctx.close()
    return out


@pytest.mark.parametrize("prec", [setd.PREC_F64, setd.PREC_F32, setd.PREC_BF16X3, setd.PREC_I8X4])
def test_memory_full_of_nan(prec):
    for dims in [(33, 20, 18), (64, 40), (17, 31, 40)]:
        prob = wl.fhn_3d(dims=dims) if len(dims) == 3 else wl.schnakenberg_2d(*dims)
        _lib.check(_lib.load().setd_release_workspace())
        for p in (setd.PREC_F64, prec):
            assert np.isnan(_run(prob, dims, p, 1, nan=True)).all()
        # a little smaller, so that rows and panels end elsewhere in the blocks
        d2 = tuple(n - 1 for n in dims)
        prob = wl.fhn_3d(dims=d2) if len(dims) == 3 else wl.schnakenberg_2d(*d2)
        ref = oracle.integrate(prob.U0, prob.A, prob.tau, 2, prob.g_kind, prob.params)
        got = _run(prob, d2, prec, 2)
        N = int(np.prod(d2))
        for c in range(2):
            e = rel_l2(got[c * N:(c + 1) * N], np.asarray(ref[c]).ravel(order="F"))
            say("kept memory", prec, d2, "field", c, "rel_l2 %.2e" % e)
            assert e < (1e-12 if prec == setd.PREC_F64 else 1e-5)


def test_threads_share_the_kept_blocks():
    dims = [(32, 24), (24, 30), (40, 16)]
    probs = [wl.schnakenberg_2d(*d) for d in dims]
    refs = [oracle.integrate(p.U0, p.A, p.tau, 2, p.g_kind, p.params) for p in probs]
    bad = []

    def work(k):
        try:
            with torch().cuda.stream(torch().cuda.Stream()):
                for _ in range(4):
                    got = _run(probs[k], dims[k], setd.PREC_F64, 2)
                    N = int(np.prod(dims[k]))
                    for c in range(2):
                        if rel_err(got[c * N:(c + 1) * N], np.asarray(refs[k][c]).ravel(order="F")) > 1e-12:
                            bad.append((k, c))
        except Exception as e:   # reported by the assertion below
            bad.append((k, repr(e)))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad


def test_release_gives_it_back():
    prob = wl.fhn_3d(dims=(64, 64, 64))
    lib = _lib.load()
    _lib.check(lib.setd_release_workspace())
    torch().cuda.synchronize()
    free0 = torch().cuda.mem_get_info()[0]
    _run(prob, (64, 64, 64), setd.PREC_F64, 1)
    kept = free0 - torch().cuda.mem_get_info()[0]
    say("kept", kept >> 20, "MiB")
    assert kept > (64 << 20)
    _lib.check(lib.setd_release_workspace())
    left = free0 - torch().cuda.mem_get_info()[0]
    say("left", left >> 20, "MiB")
    assert left < (32 << 20)   # less than the state that the tensors of this test hold
