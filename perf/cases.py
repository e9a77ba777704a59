"""What a user of the library has it do, as a list of measurable cases.

A case is one call sequence through the public binding (``paper_2602_03067_amd.binding``) at one size:

  update      one f- and one g-half-step from given potentials (a user's own schedule)
  solve       the annealed alternating solve from zero potentials
  symmetric   the averaged schedule, then the gradient with respect to x (forward and backward)
  step        solve, dual value and gradient with respect to x: one training step of an OT loss
  transport   the plan of given potentials applied to a value matrix in both directions
  grad        the gradient with respect to x at given potentials
  divergence  the debiased loss (three solves inside the library)
  hvp         one Hessian-vector product

Point clouds are drawn on the GPU from the seed; given potentials come from plain float64 Sinkhorn half-steps
(against all points of a small problem, against a sample of a large one).
"""
from __future__ import annotations

import math

import torch

from paper_2602_03067_amd import binding

# What each listed case stands for:
#  update_1000_d3        the smallest call: two half-steps on a ragged point set, bound by launches and the prologue
#  tiny_1024_d3          the benchmark's smallest solve: fifty iterations that are launches more than work
#  step_50k_d3           shape matching at ordinary size: loss value and gradient on two ragged 3-d clouds
#  anneal_262k_d3        the benchmark's headline shape, the annealing in four stages instead of twenty
#  symmetric_20k_d10     forward and backward with the averaged schedule on unit-cube data in ten dimensions
#  divergence_10k_d64    the forward size of the paper's tables (n = 10000, d = 64, unit cube), as a debiased loss
#  transport_16k_d64     the benchmark's transport workload: shifted Gaussians at d = 64, ten iterations, gradient
#  step_d128_ragged      the paper's forward + backward dimension on ragged sizes, random weights
#  hvp_8k_d64            second-order use: one Hessian-vector product at d = 64
#  image_70k_d784        the benchmark's image-shaped clouds in bf16 mode
#  embed_50k_20k_d1024   the benchmark's embedding clouds: bf16 storage, unbalanced sizes, Dirichlet weights, P V and P^T U
#  grad_image_d784       the gradient at image dimension in bf16 mode: as many value columns as coordinates
_LISTED = [
    dict(name="update_1000_d3", op="update", n=1000, m=777, d=3, dist="normal", eps=0.1, compute="fp32", weights="random"),
    dict(name="tiny_1024_d3", op="solve", n=1024, m=1024, d=3, dist="normal", eps=0.1, stages=1, iters=50, compute="fp32",
         weights="uniform"),
    dict(name="step_50k_d3", op="step", n=50021, m=40013, d=3, dist="cube", eps=0.05, stages=1, iters=10, compute="fp32",
         weights="uniform"),
    dict(name="anneal_262k_d3", op="solve", n=262144, m=262144, d=3, dist="mixture", eps=0.01, eps_start=1.0, stages=4, iters=1,
         compute="fp32", weights="uniform"),
    dict(name="symmetric_20k_d10", op="symmetric", n=20011, m=20011, d=10, dist="cube", eps=0.1, iters=10, compute="fp32",
         weights="uniform"),
    dict(name="divergence_10k_d64", op="divergence", n=10000, m=10000, d=64, dist="cube", eps=0.1, iters=10, compute="fp32",
         weights="uniform"),
    dict(name="transport_16k_d64", op="step", n=16384, m=16384, d=64, dist="shifted", eps=0.1, stages=1, iters=10, compute="fp32",
         weights="uniform"),
    dict(name="step_d128_ragged", op="step", n=9973, m=12007, d=128, dist="cube", eps=0.1, stages=1, iters=10, compute="fp32",
         weights="random"),
    dict(name="hvp_8k_d64", op="hvp", n=8192, m=8000, d=64, dist="cube", eps=0.25, cg=20, compute="fp32", weights="uniform"),
    dict(name="image_70k_d784", op="solve", n=70000, m=70000, d=784, dist="beta", eps=3.5828559, stages=1, iters=4,
         compute="bf16", weights="uniform"),
    dict(name="embed_50k_20k_d1024", op="transport", n=50000, m=20000, d=1024, dist="sphere", eps=0.05, p=64, compute="bf16",
         storage="bf16", weights="random"),
    dict(name="grad_image_d784", op="grad", n=40009, m=30011, d=784, dist="beta", eps=3.5828559, compute="bf16", weights="uniform"),
]


def listed():
    return [dict(c) for c in _LISTED]


def _size(rng, lo, hi):
    """A size spread evenly over its logarithm; half of them odd."""
    k = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, k | 1 if rng.random() < 0.5 else k))


def draw(rng):
    kind = rng.choice(["small", "lowd", "middle", "fp32", "fp32", "bf16", "bf16"])
    weights = rng.choice(["uniform", "random"])
    if kind == "small":       # launches and prologue
        n, m = _size(rng, 200, 6000), _size(rng, 200, 6000)
        if rng.random() < 0.5:
            return dict(op="update", n=n, m=m, d=rng.choice([1, 2, 3, 5, 16, 24, 64]), dist="normal", eps=rng.choice([0.1, 0.3, 1.0]),
                        compute="fp32", weights=weights)
        return dict(op="solve", n=n, m=m, d=rng.choice([2, 3]), dist="normal", eps=0.1, stages=1, iters=rng.randint(10, 50),
                    compute="fp32", weights=weights)
    if kind == "lowd":
        n, m = _size(rng, 10000, 150000), _size(rng, 10000, 150000)
        d = rng.choice([2, 3])
        if rng.random() < 0.5:
            return dict(op="solve", n=n, m=m, d=d, dist="mixture", eps=0.01, eps_start=1.0, stages=rng.randint(2, 8), iters=1,
                        compute="fp32", weights=weights)
        return dict(op="step", n=n, m=m, d=d, dist="cube", eps=rng.choice([0.03, 0.05, 0.1]), stages=1, iters=rng.randint(3, 10),
                    compute="fp32", weights=weights)
    if kind == "middle":
        return dict(op=rng.choice(["symmetric", "step"]), n=_size(rng, 2000, 30000), m=_size(rng, 2000, 30000), d=rng.randint(4, 16),
                    dist="cube", eps=rng.choice([0.1, 0.2]), stages=1, iters=rng.randint(3, 10), compute="fp32", weights=weights)
    if kind == "fp32":
        d = _size(rng, 17, 256)
        op = rng.choice(["step", "step", "divergence", "transport", "hvp"])
        if op == "hvp":
            return dict(op=op, n=_size(rng, 1000, 8000), m=_size(rng, 1000, 8000), d=min(d, 128), dist="cube", eps=0.25, cg=20,
                        compute="fp32", weights="uniform")
        hi = 16000 if d <= 128 else 10000
        c = dict(op=op, n=_size(rng, 1500, hi), m=_size(rng, 1500, hi), d=d, dist=rng.choice(["cube", "shifted"]) if op != "divergence" else "cube",
                 eps=rng.choice([0.1, 0.25]), compute="fp32", weights=weights)
        if op == "transport":
            return dict(c, p=_size(rng, 1, 128))
        return dict(c, stages=1, iters=rng.randint(3, 10))
    d = _size(rng, 64, 1024)
    dist = rng.choice(["beta", "sphere"])
    c = dict(n=_size(rng, 4000, 50000), m=_size(rng, 4000, 50000), d=d, dist=dist, eps=0.05 if dist == "sphere" else 0.05 * 0.0914 * d,
             compute="bf16", storage=rng.choice(["f32", "bf16"]), weights=weights)
    op = rng.choice(["solve", "transport", "grad"])
    if op == "solve":
        return dict(c, op=op, stages=1, iters=rng.randint(1, 4))
    if op == "transport":
        return dict(c, op=op, p=_size(rng, 1, 128))
    return dict(c, op=op)


# ---- inputs ------------------------------------------------------------------------------------------------------
def _cloud(gen, kind, k, d, target):
    dev = "cuda:0"

    def normal(*s):
        return torch.randn(*s, generator=gen, device=dev, dtype=torch.float32)

    def uniform(*s):
        return torch.rand(*s, generator=gen, device=dev, dtype=torch.float32)

    if kind == "normal":
        return normal(k, d) + (0.5 if target else 0.0)
    if kind == "shifted":
        return normal(k, d) + (1.0 if target else 0.0)
    if kind == "cube":
        return uniform(k, d)
    if kind == "mixture":
        if not target:
            return uniform(k, d)
        means = uniform(8, d)
        return means[torch.randint(0, 8, (k,), generator=gen, device=dev)] + 0.05 * normal(k, d)
    if kind == "beta":       # Beta(1/2, 2) = G1 / (G1 + G2), G1 ~ Gamma(1/2), G2 ~ Gamma(2)
        g1 = normal(k, d).square_().mul_(0.5)
        g2 = -(uniform(k, d).clamp_(min=1e-12).log_() + uniform(k, d).clamp_(min=1e-12).log_())
        return g1 / (g1 + g2)
    v = normal(k, d)         # "sphere": unit rows
    return v / v.norm(dim=1, keepdim=True)


def _weights(gen, kind, k):
    if kind == "uniform":
        return torch.full((k,), 1.0 / k, device="cuda:0", dtype=torch.float32)
    e = -torch.rand(k, generator=gen, device="cuda:0", dtype=torch.float64).clamp_(min=1e-12).log_()
    return (e / e.sum()).to(torch.float32)


def _used(t, case):
    """The points as the mode sees them, in float64 (bf16 mode rounds them to bf16)."""
    return (t.to(torch.bfloat16) if case["compute"] == "bf16" else t).to(torch.float64)


def _half_step(x, y, pot, logw, eps):
    """-eps LSE_j[(pot_j - |x_i - y_j|^2)/eps + logw_j], float64, in row blocks."""
    out = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
    bias = (pot - (y * y).sum(1)) / eps + logw
    rows = max(1, (1 << 28) // y.shape[0])
    for i in range(0, x.shape[0], rows):
        xi = x[i:i + rows]
        s = torch.addmm(bias.unsqueeze(0), xi, y.t(), alpha=2.0 / eps)
        mx = s.max(dim=1).values
        s.sub_(mx.unsqueeze(1)).exp_()
        out[i:i + rows] = (xi * xi).sum(1) - eps * (mx + s.sum(1).log_())
    return out


def _potentials(x, y, a, b, case):
    """Potentials a program would hold: ten half-steps on all points (small) or two on a sample of the points (large)."""
    eps = _eps(case)
    x, y = _used(x, case), _used(y, case)
    la, lb = a.to(torch.float64).log(), b.to(torch.float64).log()
    g = torch.zeros(y.shape[0], dtype=torch.float64, device=y.device)
    if x.shape[0] * y.shape[0] <= 150_000_000:
        for _ in range(5):
            f = _half_step(x, y, g, lb, eps)
            g = _half_step(y, x, f, la, eps)
    else:
        k = 2048
        f0 = torch.zeros(k, dtype=torch.float64, device=x.device)
        uni = torch.full((k,), -math.log(k), dtype=torch.float64, device=x.device)
        g = _half_step(y, x[:k], f0, uni, eps)
        f = _half_step(x, y[:k], g[:k], uni, eps)
    return f.to(torch.float32), g.to(torch.float32)


def _eps(case):
    return float(torch.tensor(case["eps"], dtype=torch.float32))


def _inputs(case, seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    n, m, d = case["n"], case["m"], case["d"]
    x, y = _cloud(gen, case["dist"], n, d, False), _cloud(gen, case["dist"], m, d, True)
    if case.get("storage") == "bf16":
        x, y = x.to(torch.bfloat16), y.to(torch.bfloat16)
    a, b = _weights(gen, case["weights"], n), _weights(gen, case["weights"], m)
    op = case["op"]
    s = dict(x=x, y=y, a=a, b=b)
    if op in ("update", "transport", "grad", "hvp"):
        s["f"], s["g"] = _potentials(x, y, a, b, case)
    if op == "transport":
        s["V"] = torch.randn(m, case["p"], generator=gen, device="cuda:0")
        s["U"] = torch.randn(n, case["p"], generator=gen, device="cuda:0")
    if op == "hvp":
        s["A"] = torch.randn(n, d, generator=gen, device="cuda:0")
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = dict(case)
    s["ctx"] = binding.Context(0)
    s["prob"] = binding.Problem(s["x"], s["y"], s["a"], s["b"],
                                binding.FS_COMPUTE_BF16_MFMA if case["compute"] == "bf16" else binding.FS_COMPUTE_FP32)
    return s


# ---- one pass ----------------------------------------------------------------------------------------------------
def run(s):
    case, ctx, prob = s["case"], s["ctx"], s["prob"]
    op, eps = case["op"], _eps(case)
    if op == "update":
        return dict(f=ctx.fs_update_f(prob, eps, s["g"]), g=ctx.fs_update_g(prob, eps, s["f"]))
    if op == "transport":
        PV, r = ctx.fs_apply_plan(prob, eps, s["f"], s["g"], s["V"], want_mass=True)
        PtU, c = ctx.fs_apply_plan_T(prob, eps, s["f"], s["g"], s["U"], want_mass=True)
        return dict(PV=PV, r=r, PtU=PtU, c=c)
    if op == "grad":
        return dict(gx=ctx.fs_grad_x(prob, eps, s["f"], s["g"], 2))
    if op == "hvp":
        return dict(G=ctx.fs_hvp(prob, eps, s["f"], s["g"], s["A"], 1e-5, 1e-6, case["cg"])[0])
    if op == "divergence":
        value, terms, f, g = ctx.fs_divergence(prob, eps, case["iters"])
        return dict(value=value, terms=torch.tensor(terms, dtype=torch.float64), f=f, g=g)
    f = torch.zeros(prob.n, device="cuda:0")
    g = torch.zeros(prob.m, device="cuda:0")
    if op == "symmetric":
        ctx.fs_solve_symmetric(prob, eps, case["iters"], f, g)
        return dict(f=f, g=g, gx=ctx.fs_grad_x(prob, eps, f, g, 2))
    ctx.fs_solve(prob, case.get("eps_start", eps), eps, case["stages"], case["iters"], f, g)
    if op == "solve":
        return dict(f=f, g=g)
    return dict(f=f, g=g, value=ctx.fs_ot_value(prob, eps, f, g), gx=ctx.fs_grad_x(prob, eps, f, g, 2))


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def work(case):
    n, m, d, op = case["n"], case["m"], case["d"], case["op"]
    pair = float(n) * m
    it = case.get("iters", 1) * case.get("stages", 1)
    el = 2 if case.get("storage") == "bf16" else 4
    pts, pots = (n + m) * d * el, (n + m) * 4
    half = pair * (2 * d + 4)              # contraction, bias, subtraction, exponential, sum
    apply_p = lambda p: pair * (2 * d + 4 + 2 * p)
    if op == "update":
        return dict(bytes=pts + 3 * pots, flops=2 * half)
    if op == "solve":
        return dict(bytes=pts + 2 * pots, flops=2 * it * half)
    if op == "transport":
        return dict(bytes=pts + 3 * pots + 2 * (n + m) * case["p"] * 4, flops=2 * apply_p(case["p"]))
    if op == "grad":
        return dict(bytes=pts + 2 * pots + n * d * 4, flops=apply_p(d))
    if op == "divergence":
        cubes = pair + float(n) * n + float(m) * m
        return dict(bytes=pts + 2 * pots, flops=cubes * (2 * d + 4) * (2 * it + 1))
    if op == "hvp":
        return dict(bytes=pts + 2 * pots + 2 * n * d * 4, flops=3 * apply_p(d) + pair * (6 * d + 4) + 2 * case["cg"] * apply_p(1))
    extra = half if op == "step" else 0.0  # the dual value costs one pass
    return dict(bytes=pts + 2 * pots + n * d * 4, flops=2 * it * half + extra + apply_p(d))


def tolerance(case):
    """About four times the distance from ``exact`` that each kind of output shows.

    Gradients are differences of nearby points and inherit what the iterations amplify in the potentials (2e-5 at d = 64, where the
    plan is close to an assignment); bf16 plan entries and values leave 2e-3 of an application."""
    if case["compute"] == "bf16":
        return {"solve": {"rel": 2e-6}, "transport": {"rel": 1e-2, "max": 0.2}, "grad": {"rel": 1e-3}}[case["op"]]
    return {"rel": {"update": 1e-6, "solve": 2e-6, "divergence": 2e-6, "transport": 2e-5, "hvp": 1e-4}.get(case["op"], 1e-4)}


# ---- the same in plain float64 -----------------------------------------------------------------------------------
def _plan_rows(x, y, a, b, f, g, eps, rows):
    """Row blocks of P_ij = a_i b_j exp((f_i + g_j - |x_i - y_j|^2)/eps)."""
    bias = (g - (y * y).sum(1)) / eps + b.log()
    for i in range(0, x.shape[0], rows):
        xi = x[i:i + rows]
        s = torch.addmm(bias.unsqueeze(0), xi, y.t(), alpha=2.0 / eps)
        s += ((f[i:i + rows] - (xi * xi).sum(1)) / eps + a[i:i + rows].log()).unsqueeze(1)
        yield i, s.exp_()


def _solve(x, y, la, lb, epss, iters):
    g = torch.zeros(y.shape[0], dtype=torch.float64, device=y.device)
    f = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
    for eps in epss:
        for _ in range(iters):
            f = _half_step(x, y, g, lb, eps)
            g = _half_step(y, x, f, la, eps)
    return f, g


def _value(x, y, a, b, f, g, eps):
    mass = sum(p.sum() for _, p in _plan_rows(x, y, a, b, f, g, eps, max(1, (1 << 28) // y.shape[0])))
    return float((a * f).sum() + (b * g).sum() - eps * (mass - a.sum() * b.sum()))


def _apply(x, y, a, b, f, g, eps, V):
    out = torch.empty(x.shape[0], V.shape[1], dtype=torch.float64, device=x.device)
    mass = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
    for i, p in _plan_rows(x, y, a, b, f, g, eps, max(1, (1 << 28) // y.shape[0])):
        out[i:i + p.shape[0]] = p @ V
        mass[i:i + p.shape[0]] = p.sum(1)
    return out, mass


def _hvp(x, y, a, b, f, g, eps, A, tau, eta, max_cg):
    P = torch.cat([p.clone() for _, p in _plan_rows(x, y, a, b, f, g, eps, 4096)])
    r, c = P.sum(1), P.sum(0)
    PY = P @ y
    u, up = (x * A).sum(1), (PY * A).sum(1)
    B5 = (P * (A @ y.t())) @ y
    EA = 2 * r[:, None] * A - (4 / eps) * ((r * u)[:, None] * x - u[:, None] * PY - up[:, None] * x + B5)
    r1 = 2 * (r * u - up)
    r2 = 2 * (P.t() @ u - ((P.t() @ A) * y).sum(1))
    rhs = r2 - P.t() @ (r1 / r)
    w2 = torch.zeros_like(rhs)
    res, q = rhs.clone(), rhs.clone()
    rr = rr0 = float(res @ res)
    for _ in range(max_cg):
        if not rr > 0 or math.sqrt(rr) <= eta * math.sqrt(rr0):
            break
        Sq = c * q - P.t() @ ((P @ q) / r) + tau * q
        al = rr / float(q @ Sq)
        w2 += al * q
        res -= al * Sq
        new = float(res @ res)
        q = res + (new / rr) * q
        rr = new
    pw = P @ w2
    w1 = (r1 - pw) / r
    return 2 * ((r * w1)[:, None] * x - w1[:, None] * PY + pw[:, None] * x - P @ (w2[:, None] * y)) / eps + EA


def exact(case, seed):
    s = _inputs(case, seed)
    eps, op = _eps(case), case["op"]
    x, y = _used(s["x"], case), _used(s["y"], case)
    a, b = s["a"].to(torch.float64), s["b"].to(torch.float64)
    la, lb = a.log(), b.log()
    if op in ("update", "transport", "grad", "hvp"):
        f, g = s["f"].to(torch.float64), s["g"].to(torch.float64)
    if op == "update":
        return dict(f=_half_step(x, y, g, lb, eps), g=_half_step(y, x, f, la, eps))
    if op == "transport":
        PV, r = _apply(x, y, a, b, f, g, eps, s["V"].to(torch.float64))
        PtU, c = _apply(y, x, b, a, g, f, eps, s["U"].to(torch.float64))
        return dict(PV=PV, r=r, PtU=PtU, c=c)
    if op == "hvp":
        return dict(G=_hvp(x, y, a, b, f, g, eps, s["A"].to(torch.float64), 1e-5, 1e-6, case["cg"]))
    xg, yg = s["x"].to(torch.float64), s["y"].to(torch.float64)   # the points a gradient is assembled from
    if op == "grad":
        return dict(gx=xg - _apply(x, y, a, b, f, g, eps, yg)[0] / a[:, None])
    if op == "divergence":
        out = []
        for u, v, wu, wv in ((x, y, a, b), (x, x, a, a), (y, y, b, b)):
            fu, gv = _solve(u, v, wu.log(), wv.log(), [eps], case["iters"])
            out.append((_value(u, v, wu, wv, fu, gv, eps), fu, gv))
        t = torch.tensor([o[0] for o in out], dtype=torch.float64)
        return dict(value=float(t[0] - 0.5 * t[1] - 0.5 * t[2]), terms=t, f=out[0][1], g=out[0][2])
    if op == "symmetric":
        f = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
        g = torch.zeros(y.shape[0], dtype=torch.float64, device=y.device)
        for _ in range(case["iters"]):
            f, g = 0.5 * f + 0.5 * _half_step(x, y, g, lb, eps), 0.5 * g + 0.5 * _half_step(y, x, f, la, eps)
        return dict(f=f, g=g, gx=xg - _apply(x, y, a, b, f, g, eps, yg)[0] / a[:, None])
    st = case["stages"]
    e0 = float(torch.tensor(case.get("eps_start", eps), dtype=torch.float32))
    epss = [eps if k >= st - 1 else e0 if k == 0 else float(torch.tensor(e0 * (eps / e0) ** (k / (st - 1)), dtype=torch.float32))
            for k in range(st)]
    f, g = _solve(x, y, la, lb, epss, case["iters"])
    if op == "solve":
        return dict(f=f, g=g)
    return dict(f=f, g=g, value=_value(x, y, a, b, f, g, eps), gx=xg - _apply(x, y, a, b, f, g, eps, yg)[0] / a[:, None])
