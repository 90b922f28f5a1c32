"""The stage difference formed inside the pass over a slab (2D FP64 steps up to
64 x 64) against the oracle and against the step that records its stage
quantities, which forms it in a kernel of its own: extents around the blocks of
16, contractions with every kind of remainder of 8, the smallest and the
largest slab.

Tolerance: the integrator's 1e-12 of the largest value against the oracle;
1e-14 between the two forms (the same operations, fused differently)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, rel_err, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402


@pytest.mark.parametrize("dims", [(2, 2), (3, 64), (64, 3), (16, 16), (17, 33), (31, 15), (48, 50), (63, 61), (64, 64)])
def test_stage_difference_in_the_slab(dims):
    prob = wl.schnakenberg_2d(*dims)
    A = [[dev(M) for M in Ac] for Ac in prob.A]
    ctx = setd.Context(dims, A, prob.tau)
    u0 = torch().cat([dev(f) for f in prob.U0])
    u, v = u0.clone(), u0.clone()
    rec = torch().empty(6 * u.numel(), dtype=torch().float64, device="cuda")
    ctx.step(u, 3, prob.g_kind, prob.params)
    for _ in range(3):
        ctx.step_record(v, rec, prob.g_kind, prob.params)
    ref = oracle.integrate(prob.U0, prob.A, prob.tau, 3, prob.g_kind, prob.params)
    got = u.cpu().numpy()
    N = ctx.N
    for c in range(2):
        e = rel_err(got[c * N:(c + 1) * N], np.asarray(ref[c]).ravel(order="F"))
        say("slab diff", dims, "field", c, "rel_inf %.2e" % e)
        assert e < 1e-12
    assert rel_err(got, v.cpu().numpy()) < 1e-14
