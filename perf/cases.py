"""The calls that a user of this package makes, as measurable cases.

One case is one call (or one short sequence that a program always makes together) through the
public classes of ``paper_2409_07392_amd``: the Hessian product of Lemma 1, the preconditioner
build, the eq. 11 gradient, a Relax iteration, the sampled objective with its autograd backward,
and a Round solve.  Sizes are those of the repository's own configurations (synthdata.CONFIGS, the
batch workload and the studies of bench.py) or lie between them.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same ranges, ``prepare`` what a
program holds before the call, ``run`` the call, ``work`` the bytes and operations it cannot do
without, and ``exact`` its outputs in 64 bits from plain torch.
"""
from __future__ import annotations

import math
import types

import torch

from paper_2409_07392_amd import RelaxContext, RelaxObjective, RoundSolver

LAM = 1e-3          # regulariser of Sigma_z in every configuration
_ROWS = 65536       # rows per slice of the 64-bit evaluation


# ------------------------------------------------------------------------------------- cases
def listed():
    return [
        # The smallest call: one product of the d = 20, c = 5 problem in FP64, the precision that
        # the checks and small studies use.  Latency and launches count.
        dict(name="hvp_small_f64", kind="hvp", prec="f64", n=2000, n_lab=50, d=20, c=5, s=10,
             b=10.0),
        # The product that every PCG iteration of the 50,000-point, 10-class pool runs.
        dict(name="hvp_c10_f32", kind="hvp", prec="f32", n=50000, n_lab=10, d=100, c=10, s=20,
             b=100.0),
        # Odd sizes everywhere: d, c and s that no tile divides, a ragged last row block.
        dict(name="hvp_ragged_f32", kind="hvp", prec="f32", n=30011, n_lab=37, d=203, c=37, s=7,
             b=37.0),
        # The 100-class, d = 256 pool with the split-precision products.
        dict(name="hvp_c100_bf16x3", kind="hvp", prec="bf16x3", n=200000, n_lab=100, d=256, c=100,
             s=32, b=1000.0),
        # The largest call: the product at the ImageNet-1k size (1.28M points, 1000 classes).
        dict(name="hvp_imagenet_f32", kind="hvp", prec="f32", n=1280000, n_lab=2000, d=384, c=1000,
             s=16, b=1000.0),
        # The block-Jacobi preconditioner of one mirror-descent iteration, 100 classes, d = 256.
        dict(name="precond_c100_f32", kind="precond", prec="f32", n=200000, n_lab=100, d=256,
             c=100, s=32, b=1000.0),
        # The per-point gradient of one mirror-descent iteration on the same pool.
        dict(name="grad_c100_f32", kind="grad", prec="f32", n=200000, n_lab=100, d=256, c=100,
             s=32, b=1000.0),
        # A whole Relax iteration of the 50,000-point, 10-class pool: probes, preconditioner, two
        # PCG solves, H_p product, gradient, mirror step.
        dict(name="relax_c10_f32", kind="relax", prec="f32", n=50000, n_lab=10, d=100, c=10, s=20,
             b=100.0, iters=15),
        # A whole Relax iteration at the feature width of the scaling study (d = 383, odd) with
        # many classes: the wide kernels, on a pool that a second fits.
        dict(name="relax_c200_f32", kind="relax", prec="f32", n=60000, n_lab=200, d=383, c=200,
             s=10, b=200.0, iters=10),
        # The objective and its gradient through autograd, split-precision products: the form
        # that a program with its own outer optimiser calls.
        dict(name="objective_c100_bf16x3", kind="objective", prec="bf16x3", n=50000, n_lab=100,
             d=256, c=100, s=16, b=500.0, iters=8),
        # Ten points selected from the 50,000-point, 10-class pool, objective in FP32 (the
        # paper's precision): set-up, rounds, the selection and the scores that follow it.
        dict(name="round_c10_f32", kind="round", prec="f32", n=50000, n_lab=10, d=100, c=10, s=20,
             b=10.0, fp32=True),
        # Ten points selected in the active-learning loop's shape (5000 x 50, 50 classes) in FP64.
        dict(name="round_c50_f64", kind="round", prec="f64", n=5000, n_lab=50, d=50, c=50, s=10,
             b=10.0, fp32=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("hvp", "hvp", "hvp", "precond", "grad", "relax", "objective", "round"))
    prec = rng.choice(("f32", "f32", "bf16x3", "f64"))
    case = dict(kind=kind, prec=prec, n=_log_int(rng, 2000, 400000), n_lab=rng.randint(10, 300),
                d=_log_int(rng, 20, 400), c=_log_int(rng, 5, 1000), s=_log_int(rng, 7, 32))
    if kind in ("relax", "objective"):
        case["iters"] = rng.randint(5, 15)
        case["c"] = min(case["c"], 300)
    if kind == "round":
        case["c"] = min(case["c"], 120)
        case["d"] = min(case["d"], 300)
        case["fp32"] = prec != "f64" and rng.random() < 0.6
    # a drawn case stays within a quarter of the largest listed case's operations (FP64 within a
    # tenth; the Gram sums and scores, at lower rates, within a quarter of that), its probe
    # blocks within 64 MB
    case["s"] = max(1, min(case["s"], (16 << 20) // (case["d"] * case["c"])))
    case["b"] = float(rng.randint(5, 10) if kind == "round" else max(10, case["c"]))
    limit = (3e12 if prec == "f64" else 8e12) / (4.0 if kind in ("round", "precond") else 1.0)
    flops = work(case)["flops"]
    if flops > limit:
        case["n"] = max(2000, int(case["n"] * limit / flops))
    return case


# ------------------------------------------------------------------------------------ inputs
def _dtype(case):
    return torch.float64 if case["prec"] == "f64" else torch.float32


def _problem(case, seed):
    """Feature rows of a unit-variance Gaussian mixture (whitened features), class probabilities
    from a linear model at per-row temperatures (entropies from near-certain to near-uniform),
    relaxed weights b * Dirichlet(1), all drawn in FP32 from the seed."""
    n, N, d, c = case["n"], case["n"] + case["n_lab"], case["d"], case["c"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    f32 = dict(device="cuda", dtype=torch.float32, generator=gen)
    clusters = min(c, 100)
    means = torch.randn(clusters, d, **f32) * 0.8
    lab = torch.randint(0, clusters, (N,), device="cuda", generator=gen)
    X = torch.randn(N, d, **f32).mul_(0.6).add_(means[lab])
    W = torch.randn(d, c, **f32) / math.sqrt(d)
    tau = torch.exp(torch.rand(N, 1, **f32) * math.log(12.0))
    H = torch.softmax((X @ W).mul_(tau), dim=1)
    z = -torch.log(torch.rand(n, **f32).clamp_min_(1e-7)).double()
    z *= case["b"] / z.sum()
    return types.SimpleNamespace(case=case, gen=gen, n=n, N=N, d=d, c=c, s=case["s"],
                                 X=X.to(_dtype(case)).contiguous(),
                                 H=H.to(_dtype(case)).contiguous(), z=z)


def _signs(p, t):
    """Probe block of +-1 entries (the random right-hand sides of Algorithm 2)."""
    r = torch.randint(0, 2, (p.d, p.s, p.c), device="cuda", generator=p.gen)
    return (2 * r - 1).to(t)


def _blocks(p, count):
    """Blocks as PCG holds them: signs at first, then vectors of mixed magnitude."""
    out = []
    for i in range(count):
        B = _signs(p, _dtype(p.case))
        if i > 0:
            B = B * torch.exp(torch.randn(p.d, 1, p.c, device="cuda", generator=p.gen)).to(B.dtype)
        out.append(B)
    return out


def _omega(p):
    return torch.cat([p.z, torch.ones(p.N - p.n, dtype=torch.float64, device="cuda")])


def _eta(p):
    return 8.0 * math.sqrt(p.d * p.c)


def _inputs(case, seed):
    p = _problem(case, seed)
    kind = case["kind"]
    if kind in ("hvp", "precond"):
        p.omega = _omega(p)
    if kind == "hvp":
        p.B = _blocks(p, 2)[1]
    elif kind == "grad":
        p.U, p.W = _blocks(p, 2)
    elif kind == "relax":
        p.w0 = p.z / case["b"]
        p.seed = seed
    elif kind == "objective":
        p.V = _signs(p, _dtype(case))
        p.z.requires_grad_(True)
    return p


def prepare(case, seed):
    p = _inputs(case, seed)
    p.gen = None
    p.ctx = RelaxContext(p.X, p.H, p.n, p.s, case["prec"])
    return p


# -------------------------------------------------------------------------------------- runs
def run(state):
    p, case = state, state.case
    kind = case["kind"]
    if kind == "hvp":
        return p.ctx.hvp(p.B, p.omega, LAM)
    if kind == "precond":
        return p.ctx.build_precond(p.omega, LAM, want_L=False)[1]
    if kind == "grad":
        return p.ctx.grad_z(p.U, p.W)
    if kind == "relax":
        w = p.w0.clone()
        g = torch.empty_like(w)
        # tol = 0: exactly `iters` CG iterations per solve, as the scaling study runs them
        info = p.ctx.relax_step(w, case["b"], LAM, 0.5, p.seed, 1, p.s, 0.0, case["iters"],
                                project=True, g_out=g)
        return dict(w=w, g=g, f_hat=info["f_hat"])
    if kind == "objective":
        f = RelaxObjective.apply(p.z, p.ctx, p.V, LAM, 0.0, case["iters"], True)
        (g,) = torch.autograd.grad(f, p.z)
        return dict(f=f.detach(), g=g)
    if kind == "round":
        b = int(case["b"])
        rs = RoundSolver(p.ctx, p.z, LAM, _eta(p), b, fp32=case["fp32"])
        rs.step(b)
        scores = rs.scores()
        res = rs.result()
        rs.close()
        return dict(selected=res["selected"], nu=res["nu"], score_max=res["score_max"],
                    scores=scores)
    raise ValueError(kind)


# -------------------------------------------------------------------------------------- work
def work(case):
    n, N, d, c, s = case["n"], case["n"] + case["n_lab"], case["d"], case["c"], case["s"]
    e = 8 if case["prec"] == "f64" else 4
    kind = case["kind"]
    rows, block = e * N * (d + c) + 8 * N, e * d * s * c
    hvp = 4 * N * d * c * s
    gram = N * c * d * (d + 1)                     # lower halves, multiply and add
    inv = c * d ** 3                               # symmetric factor and inverse
    if kind == "hvp":
        return dict(bytes=rows + 2 * block, flops=hvp)
    if kind == "precond":
        return dict(bytes=rows + 8 * c * d * d, flops=gram + inv)
    if kind == "grad":
        return dict(bytes=e * n * (d + c) + 2 * block + 8 * n, flops=4 * n * d * c * s)
    if kind in ("relax", "objective"):
        k = 2 * case["iters"]
        return dict(bytes=rows + 8 * 3 * n,
                    flops=gram + inv + (k + 2) * hvp + k * 2 * c * d * d * s)
    if kind == "round":
        b = int(case["b"])
        return dict(bytes=rows + 16 * n,
                    flops=gram + inv + (b + 1) * 2 * n * c * d * d + b * 3 * c * d ** 3)
    raise ValueError(kind)


# ------------------------------------------------------------------------- 64-bit evaluation
def _row_slices(N, width):
    step = max(256, min(_ROWS, (1 << 28) // max(1, width)))
    for r0 in range(0, N, step):
        yield slice(r0, min(N, r0 + step))


def _hvp64(p, omega, B, rows, shift):
    d, s, c = B.shape
    Bm = B.reshape(d, s * c)
    out = shift * Bm
    for sl in _row_slices(rows, s * c):
        X, H = p.X[sl].double(), p.H[sl].double()
        G = (X @ Bm).view(-1, s, c)
        G -= (G * H[:, None, :]).sum(dim=2, keepdim=True)
        G *= H[:, None, :]
        if omega is not None:
            G *= omega[sl][:, None, None]
        out = out + X.T @ G.view(-1, s * c)
        del G
    return out.view(d, s, c)


def _gram64(p, weights, r0, r1):
    P = torch.zeros(p.c, p.d, p.d, dtype=torch.float64, device="cuda")
    for q0 in range(r0, r1, _ROWS):
        sl = slice(q0, min(r1, q0 + _ROWS))
        X, H = p.X[sl].double(), p.H[sl].double()
        U = H * (1.0 - H) * weights[sl][:, None]
        for k in range(p.c):
            P[k] += (X * U[:, k:k + 1]).T @ X
    return P


def _grad64(p, U, W):
    d, s, c = U.shape
    g = torch.empty(p.n, dtype=torch.float64, device="cuda")
    for sl in _row_slices(p.n, 3 * s * c):
        X, H = p.X[sl].double(), p.H[sl].double()[:, None, :]
        A = (X @ U.reshape(d, s * c)).view(-1, s, c)
        Q = (X @ W.reshape(d, s * c)).view(-1, s, c)
        Q -= (Q * H).sum(dim=2, keepdim=True)
        g[sl] = -(A * Q * H).sum(dim=(1, 2)) / s
    return g


def _pcg64(p, omega, Pinv, rhs, iters):
    """`iters` iterations of projected block-Jacobi PCG on all columns from zero."""
    def proj(B):
        return B - B.mean(dim=2, keepdim=True)

    def apply(R):
        return proj(torch.matmul(Pinv, R.permute(2, 0, 1)).permute(1, 2, 0).contiguous())

    def dot(A, B):
        return (A * B).sum(dim=(0, 2))[None, :, None]

    r = proj(rhs)
    x = torch.zeros_like(r)
    z = apply(r)
    q = z.clone()
    rho = dot(r, z)
    for _ in range(iters):
        Aq = _hvp64(p, omega, q, p.N, LAM)
        alpha = rho / dot(q, Aq)
        x += alpha * q
        r = proj(r - alpha * Aq)
        z = apply(r)
        new = dot(r, z)
        q = z + (new / rho) * q
        rho = new
    return x


def _splitmix_signs(seed, t, d, s, c):
    """The documented probe stream: -1 where the top bit of SplitMix64 output number
    ((t - 1) s + j) d c + k d + a is set (64-bit wrap-around arithmetic)."""
    def wrap(v):
        v &= (1 << 64) - 1
        return v - (1 << 64) if v >> 63 else v

    def shr(v, k):
        return (v >> k) & ((1 << (64 - k)) - 1)

    a = torch.arange(d, device="cuda")[:, None, None]
    j = torch.arange(s, device="cuda")[None, :, None]
    k = torch.arange(c, device="cuda")[None, None, :]
    v = ((t - 1) * s + j) * (d * c) + k * d + a
    v = (v + 1) * wrap(0x9E3779B97F4A7C15) + wrap(seed)
    v = (v ^ shr(v, 30)) * wrap(0xBF58476D1CE4E5B9)
    v = (v ^ shr(v, 27)) * wrap(0x94D049BB133111EB)
    v = v ^ shr(v, 31)
    return torch.where(v < 0, -1.0, 1.0).double()


def _inv64(P):
    return torch.linalg.inv(P.cpu()).cuda()


def _precond64(p, omega):
    P = _gram64(p, omega, 0, p.N) + LAM * torch.eye(p.d, dtype=torch.float64, device="cuda")
    return _inv64(P)


def _relax64(p):
    case = p.case
    omega = torch.cat([case["b"] * p.w0, torch.ones(p.N - p.n, dtype=torch.float64,
                                                    device="cuda")])
    V = _splitmix_signs(p.seed, 1, p.d, p.s, p.c)
    Pinv = _precond64(p, omega)
    Y = _hvp64(p, None, _pcg64(p, omega, Pinv, V, case["iters"]), p.n, 0.0)
    f_hat = float((V * Y).sum()) / p.s
    g = _grad64(p, V, _pcg64(p, omega, Pinv, Y, case["iters"]))
    e = torch.log(p.w0) - (0.5 / g.abs().max()) * g
    w = torch.exp(e - e.max())
    return dict(w=w / w.sum(), g=g, f_hat=f_hat)


def _objective64(p):
    omega, V = _omega(p).detach(), p.V.double()
    Pinv = _precond64(p, omega)
    U = _pcg64(p, omega, Pinv, V, p.case["iters"])
    Y = _hvp64(p, None, V, p.n, 0.0)
    f = (U * Y).sum() / p.s
    return dict(f=f, g=_grad64(p, U, _pcg64(p, omega, Pinv, Y, p.case["iters"])))


def _nu64(lam, eta):
    lo = 1.0 - eta * float(lam.min())
    hi = math.sqrt(lam.numel()) - eta * float(lam.min())
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        if mid <= lo or mid >= hi:
            break
        if float(((mid + eta * lam) ** -2).sum()) > 1.0:
            lo = mid
        else:
            hi = mid
    return 0.5 * (lo + hi)


def _round64(p):
    b, eta = int(p.case["b"]), _eta(p)
    omega = _omega(p)
    Ho = _gram64(p, omega, p.n, p.N)
    Sig = _gram64(p, omega, 0, p.n) + Ho
    Sig += LAM * torch.eye(p.d, dtype=torch.float64, device="cuda")
    Linv = torch.linalg.inv(torch.linalg.cholesky(Sig.cpu()))
    X, H = p.X[:p.n].double(), p.H[:p.n].double()
    G = H * (1.0 - H)
    taken = torch.zeros(p.n, dtype=torch.bool, device="cuda")

    def scores(Binv):
        r = torch.zeros(p.n, dtype=torch.float64, device="cuda")
        for k in range(p.c):
            Y = X @ Binv[k]
            q1, q2 = (Y * X).sum(dim=1), ((Y @ Sig[k]) * Y).sum(dim=1)
            r += G[:, k] * q2 / (1.0 + eta * G[:, k] * q1)
        return r.masked_fill_(taken, -math.inf)

    Hk = torch.zeros_like(Sig)
    nus, best = [math.sqrt(p.d * p.c)], []
    Binv = _inv64(nus[0] * Sig + (eta / b) * Ho)
    for _ in range(b):
        r = scores(Binv)
        i = int(torch.argmax(r))
        best.append(float(r[i]))
        taken[i] = True
        Hk += Ho / b + G[i][:, None, None] * torch.outer(X[i], X[i])
        lam = torch.linalg.eigvalsh(torch.matmul(torch.matmul(Linv, Hk.cpu()),
                                                 Linv.transpose(1, 2).contiguous()))
        nus.append(_nu64(lam, eta))
        Binv = _inv64(nus[-1] * Sig + eta * Hk + (eta / b) * Ho)
    return dict(selected=None, nu=torch.tensor(nus, dtype=torch.float64).numpy(),
                score_max=torch.tensor(best, dtype=torch.float64).numpy(), scores=scores(Binv))


def exact(case, seed):
    # the 64-bit PCG, Gram and eigenvalue loops of the larger draws would take too long
    if case["kind"] != "hvp" and case["c"] * case["d"] ** 2 > 3e7:
        return None
    if work(case)["flops"] > (4e13 if case["kind"] == "hvp" else 6e12):
        return None
    with torch.no_grad():
        p = _inputs(case, seed)
        kind = case["kind"]
        if kind == "hvp":
            return _hvp64(p, p.omega, p.B.double(), p.N, LAM)
        if kind == "precond":
            return _precond64(p, p.omega)
        if kind == "grad":
            return _grad64(p, p.U.double(), p.W.double())
        if kind == "relax":
            return _relax64(p)
        if kind == "objective":
            return _objective64(p)
        if kind == "round":
            return _round64(p)
    raise ValueError(kind)
