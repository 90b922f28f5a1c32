"""Performance cases of the split-ETD3 library: the calls that its users make,
over the sizes they make them at.

Five kinds of call, each through the package's public entry points:

tucker  one Tucker operator W <- alpha V x_1 M_1 ... x_d M_d + beta W
step    time steps of an integration context (split-ETD3, its second-order and
        complex-coefficient relatives; FP64 and the reduced-precision forms)
batch   time steps of many independent grids of uneven size
grad    a differentiated run: forward integration, loss, backward pass
phi     phi-functions of one matrix (the set-up of every new step size)

The grids are the 2D Schnakenberg and 3D FitzHugh-Nagumo problems of the
`workloads` package (64^2, 128^3, 256^3 and the uneven batch) and the paper's
own sizes (n = 64, 100, 150, 200 in 3D; 150, 300, 450, 600 in 2D), which are
not multiples of any tile.  Matrices and initial data are built here, on the
GPU, from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2310_07551_amd as setd
from paper_2310_07551_amd import autograd as setd_autograd

PREC = {"f64": setd.PREC_F64, "f32": setd.PREC_F32, "bf16x3": setd.PREC_BF16X3, "i8x4": setd.PREC_I8X4}
BATCH_SIDES = (64, 96, 128, 192, 256, 384, 512)
FHN = (0.5, 2.0, 0.0)             # eps, a1, a0
SCHNAKENBERG = (100.0, 0.1, 0.9)  # gamma, a, b


def listed():
    return [
        # one small operator: the latency of a single call (packing, launches, workspace)
        dict(name="tucker_64x64", kind="tucker", d=2, n1=64, n2=64, n3=1, beta=0.0, prec="f64"),
        # one operator on a grid that no tile divides, added to a result
        dict(name="tucker_150x150x150", kind="tucker", d=3, n1=150, n2=150, n3=150, beta=1.0, prec="f64"),
        # the smallest integration: many short steps, bound by launches
        dict(name="schnakenberg_64x64", kind="step", d=2, n1=64, n2=64, n3=1, prec="f64", method="etd3", steps=10),
        # the paper's 2D grid on its server
        dict(name="schnakenberg_300x300", kind="step", d=2, n1=300, n2=300, n3=1, prec="f64", method="etd3", steps=5),
        # the paper's smaller 3D grid
        dict(name="fhn_100x100x100", kind="step", d=3, n1=100, n2=100, n3=100, prec="f64", method="etd3", steps=2),
        # the 3D workload of ordinary size, and the large one
        dict(name="fhn_128x128x128", kind="step", d=3, n1=128, n2=128, n3=128, prec="f64", method="etd3", steps=2),
        dict(name="fhn_256x256x256", kind="step", d=3, n1=256, n2=256, n3=256, prec="f64", method="etd3", steps=1),
        # reduced precision: the form that keeps 1e-5 at the large grid, and
        # plain FP32 at the paper's largest
        dict(name="fhn_256x256x256_i8x4", kind="step", d=3, n1=256, n2=256, n3=256, prec="i8x4", method="etd3", steps=1),
        dict(name="fhn_200x200x200_f32", kind="step", d=3, n1=200, n2=200, n3=200, prec="f32", method="etd3", steps=1),
        # a parameter study: uneven independent grids advanced together
        dict(name="batch_16", kind="batch", count=16, sides_seed=1, odd=False, steps=2),
        # fitting parameters: forward and backward through a short run
        dict(name="grad_64x64x64", kind="grad", d=3, n1=64, n2=64, n3=64, steps=5),
        # a new step size: the phi-functions of one direction
        dict(name="phi_256", kind="phi", n=256, ell=2, stiff=42.1),
    ]


# the largest listed pass, in the unit of _cost
_LIMIT = 2 * 15 * 3 * 2 * 256 ** 4


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A side of a grid: any size, or one that programmers like."""
    n = _log_int(rng, lo, hi)
    r = rng.random()
    if r < 0.25:
        n = max(lo, min(hi, 32 * round(n / 32)))
    elif r < 0.45:
        n = max(lo, min(hi, 10 * round(n / 10)))
    return n


def _grid(rng, d, lo, hi, most):
    if rng.random() < 0.5:
        n = _side(rng, lo, hi)
        dims = [n] * d
    else:
        dims = [_side(rng, lo, hi) for _ in range(d)]
    while math.prod(dims) > most:
        k = dims.index(max(dims))
        dims[k] = int(dims[k] * 0.9)
    return dims + [1] * (3 - d)


def draw(rng):
    kind = rng.choice(["tucker", "step", "step", "step", "batch", "grad", "phi"])
    while True:
        if kind == "tucker":
            d = rng.choice([2, 3])
            n1, n2, n3 = _grid(rng, d, 16, 600 if d == 2 else 256, 256 ** 3)
            case = dict(kind=kind, d=d, n1=n1, n2=n2, n3=n3, beta=rng.choice([0.0, 1.0, 0.5]),
                        prec=rng.choice(["f64", "f64", "f64", "i8x4"]))
        elif kind == "step":
            d = rng.choice([2, 3, 3])
            n1, n2, n3 = _grid(rng, d, 32, 600 if d == 2 else 256, 256 ** 3)
            prec = rng.choice(["f64", "f64", "f64", "f64", "i8x4", "i8x4", "f32", "bf16x3"])
            method = rng.choice(["etd3", "etd3", "etd3", "etd2", "cplx"]) if prec == "f64" else "etd3"
            case = dict(kind=kind, d=d, n1=n1, n2=n2, n3=n3, prec=prec, method=method, steps=rng.choice([1, 2, 5]))
        elif kind == "batch":
            case = dict(kind=kind, count=_log_int(rng, 3, 32), sides_seed=rng.randrange(1000), odd=rng.random() < 0.4,
                        steps=rng.choice([1, 2, 3]))
        elif kind == "grad":
            d = rng.choice([2, 3])
            n1, n2, n3 = _grid(rng, d, 24, 200 if d == 2 else 96, 96 ** 3)
            case = dict(kind=kind, d=d, n1=n1, n2=n2, n3=n3, steps=rng.choice([2, 3, 5, 8]))
        else:
            case = dict(kind=kind, n=_side(rng, 24, 512), ell=rng.choice([1, 2, 2, 3]), stiff=rng.choice([1.0, 10.0, 42.1]))
        if _cost(case) <= _LIMIT:
            return case


def _dims(case):
    return tuple([case["n1"], case["n2"], case["n3"]][:case["d"]])


def _batch_dims(case):
    rng = np.random.default_rng(12345 + case["sides_seed"])
    dims = []
    for _ in range(case["count"]):
        n1, n2 = (int(x) for x in rng.choice(np.asarray(BATCH_SIDES), size=2))
        if case["odd"]:
            n1, n2 = n1 - int(rng.integers(0, 17)), n2 - int(rng.integers(0, 17))
        dims.append((n1, n2))
    return dims


# ---- problem data -----------------------------------------------------------
def _offdiag(n, diff):
    """Off-diagonal entry of diff * D2: D2 the centred second difference on n
    vertices of [0, 1], homogeneous Neumann through ghost points."""
    h = 1.0 / (n - 1)
    return diff * (1.0 / (h * h))


def _neumann(n, diff):
    """diff * D2, column-major in a flat GPU tensor."""
    a = _offdiag(n, diff)
    D = torch.zeros(n, n, dtype=torch.float64)
    i = torch.arange(1, n - 1)
    D[i, i - 1] = a
    D[i, i] = -2 * a
    D[i, i + 1] = a
    D[0, 0], D[0, 1] = -2 * a, 2 * a
    D[n - 1, n - 2], D[n - 1, n - 1] = 2 * a, -2 * a
    return D.t().contiguous().reshape(-1).cuda()


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _problem(d):
    """(diffusion of u and v, reaction, its parameters, step size)."""
    if d == 2:
        return (1.0, 10.0), setd.G_SCHNAKENBERG, SCHNAKENBERG, 1e-3
    return (1.0, 42.1), setd.G_FHN, FHN, 1e-2


def _initial(d, N, g):
    """u and v, each N values: the steady state and small noise."""
    if d == 2:
        gamma, a, b = SCHNAKENBERG
        w = 0.02 * torch.rand(2, N, dtype=torch.float64, device="cuda", generator=g) - 0.01
        w[0] += a + b
        w[1] += b / (a + b) ** 2
        return w
    return 0.01 * torch.randn(2, N, dtype=torch.float64, device="cuda", generator=g)


def _tucker_data(case, seed):
    dims = _dims(case)
    g = _gen(seed)
    N = math.prod(dims)
    V = 2 * torch.rand(N, dtype=torch.float64, device="cuda", generator=g) - 1
    W = 2 * torch.rand(N, dtype=torch.float64, device="cuda", generator=g) - 1
    M = [(2 * torch.rand(n * n, dtype=torch.float64, device="cuda", generator=g) - 1) / math.sqrt(n) for n in dims]
    return dims, V, W, M


def _batch_data(case, seed):
    """Sizes, diffusion of v and initial fields of every instance."""
    dims = _batch_dims(case)
    g = _gen(seed)
    dv = (8 + 4 * torch.rand(len(dims), dtype=torch.float64, device="cuda", generator=g)).tolist()
    return dims, dv, [_initial(2, n1 * n2, g) for n1, n2 in dims]


def _grad_data(case, seed):
    dims = _dims(case)
    g = _gen(seed)
    N = math.prod(dims)
    u0 = _initial(case["d"], N, g).reshape(-1)
    return dims, u0, u0 + 0.1 * torch.randn(2 * N, dtype=torch.float64, device="cuda", generator=g)


def _phi_diff(case, seed):
    """The diffusion coefficient: the workload's, varied a little by the seed."""
    return case["stiff"] * (1 + 0.1 * torch.rand(1, dtype=torch.float64, device="cuda", generator=_gen(seed)).item())


# ---- what is measured ---------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "tucker":
        dims, V, W, M = _tucker_data(case, seed)
        return dict(case=case, dims=dims, V=V, W=W, W0=W.clone(), M=M)
    if kind == "step":
        dims = _dims(case)
        diff, g_kind, params, tau = _problem(case["d"])
        A = [[_neumann(n, dc) for n in dims] for dc in diff]
        ctx = setd.Context(dims, A, tau, prec=PREC[case["prec"]])
        u = _initial(case["d"], math.prod(dims), _gen(seed)).reshape(-1)
        return dict(case=case, ctx=ctx, u=u, g_kind=g_kind, params=params)
    if kind == "batch":
        dims, dv, U0 = _batch_data(case, seed)
        A = [[[_neumann(n, dc) for n in dm] for dc in (1.0, dv[b])] for b, dm in enumerate(dims)]
        batch = setd.Batch(dims, A, 1e-3)
        batch.tune()
        u = torch.zeros(batch.total, dtype=torch.float64, device="cuda")
        for b in range(len(dims)):
            for c in range(2):
                batch.field(u, b, c).copy_(U0[b][c])
        return dict(case=case, batch=batch, u=u, params=[SCHNAKENBERG] * len(dims))
    if kind == "grad":
        dims, u0, target = _grad_data(case, seed)
        diff, g_kind, params, tau = _problem(case["d"])
        return dict(case=case, dims=dims, u0=u0.requires_grad_(True), target=target, g_kind=g_kind, tau=tau,
                    D=[[_neumann(n, 1.0) for n in dims] for _ in range(2)],
                    params=torch.tensor(params, dtype=torch.float64, requires_grad=True),
                    diff=torch.tensor(diff, dtype=torch.float64, requires_grad=True))
    return dict(case=case, A=_neumann(case["n"], _phi_diff(case, seed)))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "tucker":
        W = state["W"]
        if case["beta"] != 0.0:
            W.copy_(state["W0"])
        return setd.tucker_apply(state["V"], W, state["dims"], state["M"], beta=case["beta"], prec=PREC[case["prec"]])
    if kind == "step":
        ctx = state["ctx"]
        step = {"etd3": ctx.step, "etd2": ctx.step2, "cplx": ctx.step_cplx}[case["method"]]
        return step(state["u"], case["steps"], state["g_kind"], state["params"])
    if kind == "batch":
        return state["batch"].step(state["u"], case["steps"], setd.G_SCHNAKENBERG, state["params"])
    if kind == "grad":
        u0, params, diff = state["u0"], state["params"], state["diff"]
        uT = setd_autograd.integrate(u0, params, diff, dims=state["dims"], D=state["D"], g_kind=state["g_kind"],
                                     tau=state["tau"], nsteps=case["steps"])
        loss = 0.5 * ((uT - state["target"]) ** 2).sum()
        return (uT.detach(),) + torch.autograd.grad(loss, [u0, params, diff])
    # the matrix of a step of 1e-2
    return setd.phi_matrices(state["A"], 1e-2, case["ell"])


# ---- what a pass cannot do without ------------------------------------------
# Tucker operators of one step per component: split-ETD3 5 split actions of 2
# (2D) or 3 (3D) terms; the complex variant 5 of 2 complex terms (a first real
# product counts 2, the later complex ones 4 and the last, real part only, 2).
def _step_flops(dims, method):
    N, d = math.prod(dims), len(dims)
    if method == "etd2":
        return 2 * 2 * sum(2 * N * n for n in dims)
    if method == "cplx":
        return 2 * 10 * sum(2 * N * n * (2 if k in (0, d - 1) else 4) for k, n in enumerate(dims))
    return 2 * (10 if d == 2 else 15) * sum(2 * N * n for n in dims)


def _cost(case):
    return work(case)["flops"]


def work(case):
    kind = case["kind"]
    if kind == "tucker":
        dims = _dims(case)
        N = math.prod(dims)
        return dict(bytes=8 * (N * (3 if case["beta"] else 2) + sum(n * n for n in dims)),
                    flops=sum(2 * N * n for n in dims))
    if kind == "step":
        dims = _dims(case)
        bank = 8 * 2 * (10 if case["d"] == 2 else 15) * sum(n * n for n in dims)
        return dict(bytes=case["steps"] * (8 * 2 * 2 * math.prod(dims) + bank),
                    flops=case["steps"] * _step_flops(dims, case["method"]))
    if kind == "batch":
        by = fl = 0
        for dims in _batch_dims(case):
            by += case["steps"] * 8 * (4 * math.prod(dims) + 2 * 10 * sum(n * n for n in dims))
            fl += case["steps"] * _step_flops(dims, "etd3")
        return dict(bytes=by, flops=fl)
    if kind == "grad":
        # forward and backward: the step, its transpose and, for the diffusion
        # gradients, 7 products for every 3 (5 for every 2 in 2D) of a step
        dims = _dims(case)
        N, d = math.prod(dims), len(dims)
        return dict(bytes=8 * (2 * N * (3 + 2 * case["steps"])),
                    flops=case["steps"] * _step_flops(dims, "etd3") * (2 + (7 / 3 if d == 3 else 5 / 2)))
    # six powers, the quotient and the recurrence, then ell + 1 products for
    # each of the squarings
    n, ell = case["n"], case["ell"]
    s = max(0, math.ceil(math.log2(4 * _offdiag(n, case["stiff"]) * 1e-2)))
    return dict(bytes=8 * (ell + 2) * n * n, flops=2 * n ** 3 * (8 + ell + s * (ell + 1)))


# ---- reference values in 64 bits --------------------------------------------
# phi-functions of a multiple of D2 from its eigenvectors cos(pi j m/(n-1)):
# entry (j, k) is w_k/(n-1) [c(|j-k|) + c(j+k)], c(s) = sum_m w_m phi(z_m)
# cos(pi s m/(n-1)), w = 1/2 at both ends, z_m = -2 a (1 - cos(pi m/(n-1))).
def _phi_values(z, order):
    """phi_0..phi_order of an array in extended precision."""
    z = np.asarray(z)
    one = z.dtype.type(1)
    small = np.abs(z) < 2
    zs = np.where(small, z, 0)
    zl = np.where(small, one, z)
    out, big = [], np.exp(zl)
    for k in range(order + 1):
        term = one / math.factorial(k) * np.ones_like(zs)
        s = term.copy()
        for j in range(1, 45):
            term = term * zs / (j + k)
            s = s + term
        out.append(np.where(small, s, big))
        big = (big - one / math.factorial(k)) / zl
    return out


class _Spectral:
    def __init__(self, n):
        self.n = n
        r = np.arange(2 * (n - 1)).astype(np.longdouble)
        self.cos = np.cos(r * (np.longdouble("3.14159265358979323846264338327950288") / (n - 1)))
        s, m = np.arange(2 * n - 1), np.arange(n)
        self.table = self.cos[(s[:, None] * m[None, :]) % (2 * (n - 1))]
        self.w = np.ones(n, dtype=np.longdouble)
        self.w[0] = self.w[-1] = 0.5
        self.lam = -2 * (1 - self.cos[:n])
        j, k = np.arange(n)[:, None], np.arange(n)[None, :]
        self.minus, self.plus = np.abs(j - k), j + k

    def matrix(self, f):
        f = self.w * f
        c = self.table @ f.real + (1j * (self.table @ f.imag) if np.iscomplexobj(f) else 0)
        M = (c[self.minus] + c[self.plus]) * (self.w / (self.n - 1))[None, :]
        return torch.from_numpy(M.astype(np.complex128 if np.iscomplexobj(f) else np.float64)).cuda()

    def phi(self, a, ell):
        """phi_ell of the matrix with off-diagonal entry a (real or complex)."""
        a = np.clongdouble(a) if isinstance(a, complex) else np.longdouble(a)
        return self.matrix(_phi_values(a * self.lam, ell)[ell])

    def phi_slope(self, a, ell):
        """d/ds phi_ell(s X) at s = 1, X the matrix with off-diagonal entry a."""
        v = _phi_values(np.longdouble(a) * self.lam, max(ell, 1))
        return self.matrix(v[ell - 1] - ell * v[ell])


def _splitting(ell, d):
    """(phi index, eta, alpha per direction) of every term of a real split action."""
    if d == 2:
        if ell == 1:
            q = math.sqrt(10)
            return [(1, -5 / 4, (4 / 3 + 4 * q / 15, 4 / 3 - 4 * q / 15)), (2, 9.0, (16 / 9 + 2 * q / 9, 16 / 9 - 2 * q / 9))]
        q = math.sqrt(33)
        return [(1, -4 / 3, (9 / 8 + q / 8, 9 / 8 - q / 8)), (2, 22 / 3, (3 / 2 + 3 * q / 22, 3 / 2 - 3 * q / 22))]
    if ell == 1:
        q = math.sqrt(2991111)
        e, x, mid, a2 = 2243 / 1350, 440521 / (675 * q), -12544 / 675, 45 / 28
        a = (3 * (5161 + q) / 15869, 3 * (5161 - q) / 15869)
    else:
        q = math.sqrt(2391)
        e, x, mid, a2 = 19 / 27, 151 / (27 * q), -196 / 27, 9 / 7
        a = (3 * (121 + q) / 490, 3 * (121 - q) / 490)
    return [(1, e + x, (a[0],) * 3), (2, mid, (a2,) * 3), (1, e - x, (a[1],) * 3)]


def _splitting_cplx(ell, d):
    s = 2.0 ** (d - 2)
    if ell == 1:
        q = math.sqrt(2)
        return [(1, 7 / 4 + 1.5j * q, (12 / 11 - 4j * q / 11,) * d), (2, s * (-3 - 6j * q), (4 / 3 - 2j * q / 3,) * d)]
    q = math.sqrt(3)
    return [(1, 2 / 3 + 2j * q / 3, (3 / 4 - 1j * q / 4,) * d), (2, s * (-2 / 3 - 8j * q / 3), (6 / 7 - 3j * q / 7,) * d)]


def _modes(T, mats):
    """T (axes n_d .. n_1) times a matrix along every mode."""
    shape = T.shape
    d = len(shape)
    T = torch.matmul(T.reshape(-1, shape[-1]), mats[0].t()).reshape(shape)
    if d == 3:
        T = torch.matmul(mats[1], T)
    return torch.matmul(mats[d - 1], T.reshape(shape[0], -1)).reshape(shape)


def _reaction(kind, u, v, p):
    if kind == setd.G_SCHNAKENBERG:
        w = u * u * v
        return p[0] * (p[1] - u + w), p[0] * (p[2] - w)
    return u - u * u * u - v, p[0] * (u - p[1] * v - p[2])


class _Plain:
    """The time steps in plain torch, FP64, differentiable in the state, the
    reaction parameters and the diffusion coefficients."""

    def __init__(self, dims, diff, tau, spectral, method="etd3", slopes=False):
        self.dims, self.diff0, self.tau, self.method, self.slopes = dims, diff, tau, method, slopes
        self.sp = spectral
        self.terms, self.cache = {}, {}
        d = len(dims)
        if method == "etd2":
            for ell in (1, 2):
                for c in (0, 1):
                    self.terms[c, 1.0, ell] = [(ell, math.factorial(ell) ** (d - 1), [self._pair(c, mu, tau, ell) for mu in range(d)])]
            return
        for s, ell in ((1 / 3, 1), (2 / 3, 1), (2 / 3, 2), (1.0, 1), (1.0, 2)):
            for c in (0, 1):
                self.terms[c, s, ell] = [
                    (li, eta, [self._pair(c, mu, s * tau * al[mu], li) for mu in range(d)])
                    for li, eta, al in (_splitting_cplx if method == "cplx" else _splitting)(ell, d)]

    def _pair(self, c, mu, z, li):
        key = (c, self.dims[mu], z, li)
        if key not in self.cache:
            a = z * _offdiag(self.dims[mu], self.diff0[c])
            S = self.sp[self.dims[mu]]
            self.cache[key] = (S.phi(a, li), S.phi_slope(a, li) if self.slopes else None)
        return self.cache[key]

    def action(self, c, s, ell, V, diff):
        out = None
        for _, eta, pairs in self.terms[c, s, ell]:
            mats = [P if dP is None else P + (diff[c] / self.diff0[c] - 1) * dP for P, dP in pairs]
            W = _modes(V.to(mats[0].dtype), mats) * eta
            out = W if out is None else out + W
        return out.real if out.is_complex() else out

    def laplace(self, c, V, diff):
        d, out = len(self.dims), 0
        for mu in range(d):
            n = self.dims[mu]
            W = V.movedim(d - 1 - mu, -1)
            r = torch.empty_like(W)
            r = torch.cat([2 * (W[..., 1:2] - W[..., :1]), W[..., :-2] - 2 * W[..., 1:-1] + W[..., 2:],
                           2 * (W[..., -2:-1] - W[..., -1:])], -1)
            out = out + (_offdiag(n, 1.0) * r).movedim(-1, d - 1 - mu)
        return out * diff[c]

    def step(self, U, kind, p, diff):
        tau, act = self.tau, self.action
        G = _reaction(kind, *U, p)
        F = [self.laplace(c, U[c], diff) + G[c] for c in (0, 1)]
        if self.method == "etd2":
            U2 = [U[c] + tau * act(c, 1.0, 1, F[c], diff) for c in (0, 1)]
            g = _reaction(kind, *U2, p)
            return [U2[c] + tau * act(c, 1.0, 2, g[c] - G[c], diff) for c in (0, 1)]
        U2 = [U[c] + tau / 3 * act(c, 1 / 3, 1, F[c], diff) for c in (0, 1)]
        g = _reaction(kind, *U2, p)
        U3 = [U[c] + 2 * tau / 3 * act(c, 2 / 3, 1, F[c], diff) + 4 * tau / 3 * act(c, 2 / 3, 2, g[c] - G[c], diff) for c in (0, 1)]
        g = _reaction(kind, *U3, p)
        return [U[c] + tau * act(c, 1.0, 1, F[c], diff) + 1.5 * tau * act(c, 1.0, 2, g[c] - G[c], diff) for c in (0, 1)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "tucker":
        dims, V, W, M = _tucker_data(case, seed)
        T = _modes(V.reshape(dims[::-1]), [m.reshape(n, n).t() for m, n in zip(M, dims)]).reshape(-1)
        return T + case["beta"] * W if case["beta"] else T
    if kind == "step":
        dims = _dims(case)
        diff, g_kind, params, tau = _problem(case["d"])
        plain = _Plain(dims, diff, tau, {n: _Spectral(n) for n in set(dims)}, case["method"])
        U = list(_initial(case["d"], math.prod(dims), _gen(seed)).reshape((2,) + dims[::-1]))
        for _ in range(case["steps"]):
            U = plain.step(U, g_kind, params, diff)
        return torch.stack(U).reshape(-1)
    if kind == "batch":
        dims, dv, U0 = _batch_data(case, seed)
        sp = {n: _Spectral(n) for n in {n for dm in dims for n in dm}}
        out = []
        for b, dm in enumerate(dims):
            plain = _Plain(dm, (1.0, dv[b]), 1e-3, sp)
            U = list(U0[b].reshape((2,) + dm[::-1]))
            for _ in range(case["steps"]):
                U = plain.step(U, setd.G_SCHNAKENBERG, SCHNAKENBERG, (1.0, dv[b]))
            pad = -(dm[0] * dm[1]) % 8   # each field of the batch's state starts at a multiple of 8
            for u in U:
                out += [u.reshape(-1), torch.zeros(pad, dtype=u.dtype, device=u.device)]
        return torch.cat(out)
    if kind == "grad":
        dims, u0, target = _grad_data(case, seed)
        diff0, g_kind, params, tau = _problem(case["d"])
        plain = _Plain(dims, diff0, tau, {n: _Spectral(n) for n in set(dims)}, slopes=True)
        u0.requires_grad_(True)
        p = torch.tensor(params, dtype=torch.float64, device="cuda", requires_grad=True)
        diff = torch.tensor(diff0, dtype=torch.float64, device="cuda", requires_grad=True)
        U = list(u0.reshape((2,) + dims[::-1]))
        for _ in range(case["steps"]):
            U = plain.step(U, g_kind, p, diff)
        uT = torch.stack(U).reshape(-1)
        gu, gp, gd = torch.autograd.grad(0.5 * ((uT - target) ** 2).sum(), [u0, p, diff])
        return uT.detach(), gu, gp.cpu(), gd.cpu()
    a = 1e-2 * _offdiag(case["n"], _phi_diff(case, seed))
    S = _Spectral(case["n"])
    return torch.stack([S.phi(a, k).t().contiguous().reshape(-1) for k in range(case["ell"] + 1)])
