"""Products whose launch comes near the 2^32 threads that a grid may have: modes
of size 1 and 3 over 2^30 and 2^31 entries, where the smallest tiles would need
more. A product by a 1 x 1 matrix is checked whole, one by a 3 x 3 matrix on
its first and last fibres.

Tolerance: one product rounded to the type of the arithmetic (2^-53, 2^-24, two
or three bf16 pieces 2^-16 and 2^-24); three of them added up four times that."""
import pytest

from tests.gpu_util import dev, say, torch
import workloads as wl

pytestmark = pytest.mark.gpu

import paper_2310_07551_amd as setd   # noqa: E402

EPS = {setd.PREC_F64: 2.0 ** -53, setd.PREC_F32: 2.0 ** -22, setd.PREC_BF16X3: 2.0 ** -22, setd.PREC_BF16X2: 2.0 ** -14}


@pytest.mark.parametrize("prec,dims,mu", [
    (setd.PREC_F64, (4096, 4096, 128, 1), 3), (setd.PREC_F64, (4096, 128, 1, 4096), 2),
    (setd.PREC_F32, (4096, 4096, 64, 1), 3), (setd.PREC_F32, (1, 4096, 4096, 64), 0),
    (setd.PREC_BF16X3, (4096, 4096, 64, 1), 3), (setd.PREC_BF16X2, (4096, 64, 1, 4096), 2)])
def test_size_one(prec, dims, mu):
    N = 1
    for n in dims:
        N *= n
    say("large grid", prec, dims, mu, "%.0f GB" % (N * 8 / 1e9))
    V = torch().empty(N, dtype=torch().float64, device="cuda")
    V.uniform_(0.5, 1.0)
    W = torch().full((N,), float("nan"), dtype=torch().float64, device="cuda")
    mats = [None] * 4
    mats[mu] = torch().tensor([0.75], dtype=torch().float64, device="cuda")
    setd.tucker_apply(V, W, dims, mats, prec=prec)
    V.mul_(0.75).sub_(W).abs_()
    worst = V.max().item()
    say("  worst difference %.2e" % worst)
    assert worst <= EPS[prec]


def test_size_three():
    dims = (4096, 4096, 3, 40)
    N = 4096 * 4096 * 3 * 40
    V = torch().empty(N, dtype=torch().float64, device="cuda")
    V.uniform_(-1.0, 1.0)
    W = torch().full((N,), float("nan"), dtype=torch().float64, device="cuda")
    M = wl.random_matrix(3, 4)
    say("large grid", dims)
    setd.tucker_apply(V, W, dims, [None, None, dev(M), None])
    v, w = V.view(40, 3, -1), W.view(40, 3, -1)   # slowest index first
    Md = torch().from_numpy(M).cuda()
    for b in (0, 39):
        for i in range(3):
            ref = sum(Md[i, p] * v[b, p] for p in range(3))
            assert (w[b, i] - ref).abs().max().item() <= 4 * 2.0 ** -53
