"""Performance cases of the scattering solver: what its users run, through the
package's public entry points, over the range of sizes they run it at.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``product``   one application of the system matrix (``ori_matvec``): the
  building block of a user's own Krylov method or of a residual check.
* ``solve``     ``ori_load`` + ``ori_solve`` on a context kept by the program:
  one step of a sweep.  With ``sweep`` = "k" (a frequency sweep) every step
  computes the kernel spectrum, with ``sweep`` = "h" (a design loop at one
  frequency) the context keeps it.
* ``batch``     the same for a block of incident directions.
* ``gradient``  ``ori_load`` + ``ori_gradient``: forward and adjoint solve of an
  inverse problem.
* ``autograd``  the differentiable solve under torch.autograd, forward and
  backward, as one step of an optimisation in torch.
* ``group``     ``solve_many``: independent problems of uneven sizes.
* ``field``     post-processing of a solution: charges, scattered field at M
  points outside the body and the far field in M directions.

Inputs follow the paper's Section 4 and workloads.py: the unit cube, N = 1, a
plane wave, impedance -1 + 0.5i with a random spread of 10 %.  Solves run to
the library's default tolerance, 1e-10.
"""

import math

import torch

import paper_1602_04691_amd as ori

TOL = 1e-10
DEV = "cuda"


def listed():
    return [
        # the smallest call: one product on the grid of the parity case; launches and latency
        dict(name="product_n16", kind="product", n=16, k=1.0),
        # an ordinary size that is no power of two (2n = 200)
        dict(name="product_n100", kind="product", n=100, k=5.0),
        # a large ragged size (2n = 600, 27 M unknowns)
        dict(name="product_n300", kind="product", n=300, k=5.0),
        # a small solve inside a design loop: dozens of short kernels and host round trips
        dict(name="solve_n32", kind="solve", n=32, k=5.0, precision="fp64", sweep="h"),
        # a ragged size in mixed precision, one step of a frequency sweep
        dict(name="solve_n200_mixed", kind="solve", n=200, k=5.0, precision="mixed", sweep="k"),
        # the benchmark's workload: 16.8 M unknowns, load and solve in complex128
        dict(name="solve_n256", kind="solve", n=256, k=5.0, precision="fp64", sweep="k"),
        # the largest grid: 134 M unknowns in mixed precision
        dict(name="solve_n512_mixed", kind="solve", n=512, k=10.0, precision="mixed", sweep="h"),
        # one body lit from 32 directions (the batch workload of bench.py)
        dict(name="batch_n64x32_mixed", kind="batch", n=64, k=5.0, nrhs=32, precision="mixed"),
        # one step of an inverse problem (the gradient workload of bench.py)
        dict(name="gradient_n128", kind="gradient", n=128, k=5.0, precision="fp64"),
        # a small differentiable solve in torch, forward and backward
        dict(name="autograd_n48_mixed", kind="autograd", n=48, k=3.0, precision="mixed"),
        # a handful of bodies of different resolution solved together (the uneven workload of bench.py)
        dict(name="group_32_48_64_96_mixed", kind="group", ns="32,48,64,96", k=5.0, precision="mixed"),
        # field and far field of a solution on a sphere of points (the field workload of bench.py)
        dict(name="field_n64_m4096", kind="field", n=64, k=5.0, points=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product", "product", "solve", "solve", "solve", "batch", "gradient", "autograd", "group",
                       "field"])
    precision = rng.choice(["fp64", "mixed"])
    k = round(rng.uniform(1.0, 8.0), 2)
    if kind == "product":
        return dict(kind=kind, n=_log_int(rng, 8, 400), k=k)
    if kind == "solve":
        return dict(kind=kind, n=_log_int(rng, 8, 320), k=k, precision=precision, sweep=rng.choice(["h", "k"]))
    if kind == "batch":
        return dict(kind=kind, n=_log_int(rng, 16, 72), k=k, nrhs=rng.randint(2, 32), precision=precision)
    if kind == "gradient":
        return dict(kind=kind, n=_log_int(rng, 16, 160), k=k, precision=precision)
    if kind == "autograd":
        return dict(kind=kind, n=_log_int(rng, 8, 80), k=k, precision=precision)
    if kind == "group":
        ns = sorted(_log_int(rng, 12, 100) for _ in range(rng.randint(2, 6)))
        return dict(kind=kind, ns=",".join(str(n) for n in ns), k=k, precision=precision)
    return dict(kind=kind, n=_log_int(rng, 16, 72), k=k, points=_log_int(rng, 200, 4096))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _impedance(n, g):
    xi = 2.0 * torch.rand(n ** 3, dtype=torch.float64, device=DEV, generator=g) - 1.0
    return (-1.0 + 0.5j) * (1.0 + 0.1 * xi)


def _direction(g):
    a = torch.randn(3, dtype=torch.float64, device=DEV, generator=g)
    return a / a.norm()


def _plane_wave(n, k, alpha):
    t = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
    e = [torch.polar(torch.ones_like(t), k * alpha[d] * t) for d in range(3)]
    return (e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]).reshape(-1)


def _smooth(n, g):
    """A positive smooth amplitude on the grid (order 1)."""
    t = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
    c = torch.rand(6, dtype=torch.float64, device=DEV, generator=g)
    w = [1.0 + 0.3 * c[d] * torch.cos(2.0 * math.pi * (t + c[3 + d])) for d in range(3)]
    return (w[0][:, None, None] * w[1][None, :, None] * w[2][None, None, :]).reshape(-1)


def _inputs(case, seed):
    """Every tensor of the case, from the seed alone (also what exact() uses)."""
    g, kind, k = _gen(seed), case["kind"], case["k"]
    if kind == "group":
        probs = []
        for n in (int(v) for v in case["ns"].split(",")):
            h = _impedance(n, g)
            probs.append(dict(n=n, k=k, h=h, u0=_plane_wave(n, k, _direction(g))))
        return probs
    n = case["n"]
    s = dict(h=_impedance(n, g), N=torch.ones(n ** 3, dtype=torch.float64, device=DEV))
    if kind == "batch":
        s["u0"] = torch.stack([_plane_wave(n, k, _direction(g)) for _ in range(case["nrhs"])]).reshape(-1)
        return s
    s["u0"] = _plane_wave(n, k, _direction(g))
    if kind == "product":
        s["x"] = s["u0"] * _smooth(n, g)
    if kind in ("gradient", "autograd"):
        # the field asked for: another plane wave of another amplitude
        s["target"] = 0.7 * _plane_wave(n, k, _direction(g))
    if kind == "field":
        s["u"] = s["u0"] * _smooth(n, g)
        d = torch.randn(case["points"], 3, dtype=torch.float64, device=DEV, generator=g)
        s["beta"] = (d / d.norm(dim=1, keepdim=True)).contiguous()
        s["x"] = (0.5 + 2.0 * s["beta"]).contiguous()
    return s


def _precision(case):
    return ori.ORI_MIXED if case.get("precision") == "mixed" else ori.ORI_FP64


def prepare(case, seed):
    kind = case["kind"]
    if kind == "group":
        return dict(case=case, problems=_inputs(case, seed))
    s = _inputs(case, seed)
    n, k = case["n"], case["k"]
    s["case"] = case
    if kind == "autograd":
        return s
    s["ctx"] = ctx = ori.ori_create(n, nrhs=case.get("nrhs", 1))
    if kind in ("product", "field"):
        ori.ori_load(ctx, k, s["h"], s["N"], s["u0"])
    if kind == "product":
        s["y"] = torch.empty_like(s["x"])
    if kind in ("solve", "batch", "gradient"):
        s["u"] = torch.empty_like(s["u0"])
        if case.get("sweep") == "k":
            ori.ori_spectrum_cache(ctx, False)
    if kind == "gradient":
        s["g"] = torch.empty_like(s["u0"])
    return s


def run(s):
    case = s["case"]
    kind, k, prec = case["kind"], case["k"], _precision(case)
    if kind == "group":
        return [u for u, _ in ori.solve_many(s["problems"], tol=TOL, precision=prec)]
    if kind == "product":
        ori.ori_matvec(s["ctx"], s["x"], s["y"])
        return s["y"]
    if kind in ("solve", "batch"):
        ori.ori_load(s["ctx"], k, s["h"], s["N"], s["u0"])
        ori.ori_solve(s["ctx"], s["u"], tol=TOL, precision=prec)
        return s["u"]
    if kind == "gradient":
        ori.ori_load(s["ctx"], k, s["h"], s["N"], s["u0"])
        _, J, _ = ori.ori_gradient(s["ctx"], s["target"], s["u"], s["g"], tol=TOL, precision=prec)
        return dict(J=J, u=s["u"], g=s["g"])
    if kind == "autograd":
        h = s["h"].detach().requires_grad_(True)
        u = ori.OriSolve(h, s["u0"], case["n"], k, N=s["N"], tol=TOL, precision=prec)
        e = torch.view_as_real(u - s["target"])
        J = (e * e).sum()
        (gh,) = torch.autograd.grad(J, h)
        return dict(J=J.detach(), u=u.detach(), g=gh.resolve_conj())
    return dict(q=ori.ori_charges(s["ctx"], s["u"]), v=ori.ori_scattered_field(s["ctx"], s["u"], s["x"]),
                A=ori.ori_far_field(s["ctx"], s["u"], s["beta"]))


# ---------------------------------------------------------------------------
# what one pass cannot do without
# ---------------------------------------------------------------------------
def _product_work(n):
    """One product: x, the diagonal and the result (complex128) and the
    transforms of the padded (2n)^3 grid without the pencils that are zero or
    discarded: 14 n^2 pencils of length 2n, and the spectrum product."""
    L = 2 * n
    return 48.0 * n ** 3, 14.0 * n * n * 5.0 * L * max(1.0, math.log2(L)) + 6.0 * L ** 3


def _solve_work(n, nrhs=1, adjoint=False):
    """h, N, u0 read and u written once; about 15 products at this tolerance,
    each with the update of its vectors (about 60 operations per unknown)."""
    b, f = _product_work(n)
    its = 15.0 * (2.0 if adjoint else 1.0)
    return n ** 3 * (24.0 + nrhs * 32.0) + nrhs * its * b, nrhs * its * (f + 60.0 * n ** 3)


def work(case):
    kind = case["kind"]
    if kind == "product":
        b, f = _product_work(case["n"])
    elif kind in ("solve", "batch"):
        b, f = _solve_work(case["n"], case.get("nrhs", 1))
    elif kind in ("gradient", "autograd"):
        b, f = _solve_work(case["n"], adjoint=True)
        b += 32.0 * case["n"] ** 3  # the target and the gradient
    elif kind == "group":
        b = f = 0.0
        for n in (int(v) for v in case["ns"].split(",")):
            bn, fn = _solve_work(n)
            b, f = b + bn, f + fn
    else:
        P, M = case["n"] ** 3, case["points"]
        # charges: u, D, q.  The sums: u and D again, points and results;
        # operations per pair: distance 8, its square root and reciprocal 2,
        # sine and cosine 2, product 12 (field); a complex multiply-add 8 (far
        # field, whose phase is a product of per-axis phases)
        b, f = 48.0 * P + 2.0 * (32.0 * P + 40.0 * M), 32.0 * P * M
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same results in torch, in 64 bits
# ---------------------------------------------------------------------------
def _smooth_length(m):
    while True:
        r = m
        for p in (2, 3, 5):
            while r % p == 0:
                r //= p
        if r == 1:
            return m
        m += 1


class _Green:
    """y = G0 x on the unit cube's n^3 cell centres by zero-padded FFTs."""

    def __init__(self, n, k):
        self.n = n
        self.L = L = _smooth_length(2 * n)
        d = torch.arange(L, dtype=torch.float64, device=DEV)
        d = torch.where(d < n, d, L - d)  # distances along one axis, periodic
        d = torch.where(d < n, d, torch.full_like(d, n)) / n
        r = (d[:, None, None] ** 2 + d[None, :, None] ** 2 + d[None, None, :] ** 2).sqrt()
        r[0, 0, 0] = 1.0
        G = torch.polar(1.0 / (4.0 * math.pi * r), k * r)
        del r
        G[0, 0, 0] = 0.0
        self.K = torch.fft.fftn(G)

    def __call__(self, x):
        n, L = self.n, self.L
        f = torch.fft.fftn(x.view(n, n, n), s=(L, L, L))
        f *= self.K
        return torch.fft.ifftn(f)[:n, :n, :n].reshape(-1)


def _cocg(apply, b):
    """A w = b for complex-symmetric A, run until the residual stalls at
    rounding."""
    x, r = torch.zeros_like(b), b.clone()
    p = r.clone()
    rho = (r * r).sum()
    stop, best, since = 1e-15 * b.norm().item(), math.inf, 0
    for _ in range(200):
        q = apply(p)
        alpha = rho / (p * q).sum()
        x += alpha * p
        r -= alpha * q
        res = r.norm().item()
        since = 0 if res < 0.9 * best else since + 1
        best = min(best, res)
        if res <= stop or since >= 4:
            break
        rho_new = (r * r).sum()
        p = r + (rho_new / rho) * p
        rho = rho_new
    return x


def _exact_solve(G, h, N, u0):
    """u of the scattering equation; (I + S G0 S) w = S u0, u = w / S."""
    D = (4.0 * math.pi / G.n ** 3) * h * N
    S = D.sqrt()
    w = _cocg(lambda p: p + S * G(S * p), S * u0)
    return w / S


def _exact_gradient(G, h, N, u, t):
    """g with dJ = Re sum g dh for J = sum |u - t|^2: -2 c u G0 lambda,
    (I + D G0) lambda = conj(u - t)."""
    c = (4.0 * math.pi / G.n ** 3) * N
    S = (c * h).sqrt()
    f = torch.conj(u - t).resolve_conj()
    Gf = G(f)
    z = _cocg(lambda p: p + S * G(S * p), S * Gf)
    return -2.0 * c * u * (Gf - G(S * z))


def exact(case, seed):
    s, kind, k = _inputs(case, seed), case["kind"], case["k"]
    if kind == "group":
        return [_exact_solve(_Green(p["n"], k), p["h"], torch.ones_like(p["h"].real), p["u0"]) for p in s]
    n = case["n"]
    D = (4.0 * math.pi / n ** 3) * s["h"] * s["N"]
    if kind == "field":
        t = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
        X = torch.stack(torch.meshgrid(t, t, t, indexing="ij"), dim=-1).reshape(-1, 3)
        q = -D * s["u"]
        v, A = [], []
        step = max(1, 2 ** 25 // n ** 3)
        for m in range(0, case["points"], step):
            y, beta = s["x"][m:m + step], s["beta"][m:m + step]
            r2 = sum((y[:, d, None] - X[None, :, d]) ** 2 for d in range(3))
            r = r2.sqrt()
            v.append((torch.polar(1.0 / (4.0 * math.pi * r), k * r) * q).sum(dim=1))
            ph = -k * sum(beta[:, d, None] * X[None, :, d] for d in range(3))
            A.append((torch.polar(torch.full_like(ph, 1.0 / (4.0 * math.pi)), ph) * q).sum(dim=1))
        return dict(q=q, v=torch.cat(v), A=torch.cat(A))
    G = _Green(n, k)
    if kind == "product":
        return s["x"] + G(D * s["x"])
    if kind == "batch":
        return torch.stack([_exact_solve(G, s["h"], s["N"], b) for b in s["u0"].view(case["nrhs"], -1)]).reshape(-1)
    u = _exact_solve(G, s["h"], s["N"], s["u0"])
    if kind == "solve":
        return u
    e = torch.view_as_real(u - s["target"])
    J = (e * e).sum()
    g = _exact_gradient(G, s["h"], s["N"], u, s["target"])
    if kind == "autograd":  # torch's convention for the gradient of a real loss
        return dict(J=J, u=u, g=torch.conj(g).resolve_conj())
    return dict(J=float(J), u=u, g=g)
