"""GPU parity of the half-steps and gradients through cell moments (d <= 3) against the float64 oracle, where they are left out, and
what they hold.

The passes are mostly forced with the context's "lowd_moments" switch, so that small clouds reach every part of them: cells of several
blocks, more streamed cells than one segment, several launches, ragged groups of rows, empty cells, one-cell clouds.

Tolerance of a half-step in units of eps (= relative error of a row sum): the series of e^t is off by 3e-8, monomials, weights and
moments are kept to 2^-22, and a row in a corner of its cell can lose e^(2 tau) = 14 of that to cancellation: 14 (3e-8 + 3 2^-22) =
1.1e-5; the float output adds |f| 2^-24 / eps.  The exponents are floats as well: up to 18 between the points of a cell and 36 between
its rows and a cell in the clouds of this file, which adds up to 54 ln2 2^-24 = 2e-6 where one term makes a row and is left to the slack
of the bound above (they may reach 48 and 96, with the scores: fp32 scores of that size round as much).
"""
import numpy as np
import pytest
import torch

from paper_2602_03067_amd import binding, workloads
from tests._gpu_common import dev, host, make_problem, max_err_over_eps, say

pytestmark = pytest.mark.gpu

TOL = 1.1e-5


def _tol(f, eps):
    return TOL + float(np.max(np.abs(f))) * 2.0 ** -24 / eps


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    c.fs_debug_set("lowd_moments", 1)
    yield c
    c.close()


def _cloud(rng, kind, n, d):
    if kind == "cube":
        x = rng.random((n, d))
    elif kind == "clusters":      # most points in a few cells
        x = 0.5 + 0.002 * rng.standard_normal((n, d))
        x[: n // 10] = rng.random((n // 10, d))
    elif kind == "flat":          # no extent in the last coordinate
        x = rng.random((n, d))
        x[:, -1] = 0.25
    else:                         # one point, n times
        x = np.full((n, d), 0.3)
    return x.astype(np.float32)


def _weights(rng, n, zeros=False):
    a = rng.random(n) + 0.1
    if zeros:
        a[rng.random(n) < 0.3] = 0.0
        a[0] = 0.5
    return (a / a.sum()).astype(np.float32)


# one point, ragged tiles of 32 rows and points, cells of more than 256 rows and of several blocks, every kind of expansion (it
# follows from d and eps), more than 1024 cells (two segments, several launches)
@pytest.mark.parametrize("n,m,d,eps,kind", [
    (1, 1, 3, 0.1, "cube"), (5, 3, 1, 0.05, "cube"), (255, 257, 2, 0.05, "cube"), (1000, 777, 3, 0.1, "cube"),
    (700, 3000, 3, 3.0, "cube"), (2049, 513, 3, 0.05, "cube"), (900, 1100, 3, 0.6, "cube"), (5000, 4000, 3, 0.3, "clusters"),
    (1500, 9000, 2, 0.1, "clusters"), (3000, 6000, 1, 0.2, "clusters"), (4000, 3000, 3, 0.012, "cube"), (3000, 2500, 2, 0.003, "cube"),
    (800, 900, 3, 0.1, "flat"), (300, 500, 2, 0.2, "point")])
@pytest.mark.parametrize("pot", ["zero", "smooth", "rough"])
def test_half_steps(ctx, oracle, n, m, d, eps, kind, pot):
    rng = np.random.default_rng(n + 7 * m + d)
    x, y = _cloud(rng, "cube" if kind == "clusters" else kind, n, d), _cloud(rng, kind, m, d)
    a, b = _weights(rng, n), _weights(rng, m, zeros=pot == "rough")
    eps = float(np.float32(eps))
    g = np.zeros(m, np.float32)
    f = np.zeros(n, np.float32)
    if pot == "smooth":
        g, f = (y ** 2).sum(1) - 0.3 * y[:, 0], (x ** 2).sum(1) + 0.2 * x[:, -1]
    elif pot == "rough":
        g, f = 8.0 * eps * rng.standard_normal(m), 8.0 * eps * rng.standard_normal(n)
    g, f = g.astype(np.float32), f.astype(np.float32)
    say("moments n=%d m=%d d=%d eps=%g %s %s" % (n, m, d, eps, kind, pot))
    prob = make_problem(x, y, a, b)
    f1 = host(ctx.fs_update_f(prob, eps, dev(g)))
    g1 = host(ctx.fs_update_g(prob, eps, dev(f)))
    fw, gw = oracle.update_f(x, y, b, eps, g), oracle.update_g(x, y, a, eps, f)
    assert max_err_over_eps(f1, fw, eps) <= _tol(fw, eps)
    assert max_err_over_eps(g1, gw, eps) <= _tol(gw, eps)
    # a fixed order of every sum
    assert np.array_equal(f1, host(ctx.fs_update_f(prob, eps, dev(g))))


# the rows' kernel is compiled per kind of expansion: the one between the least and the largest in two dimensions, and full, ragged and
# single groups of rows for it
@pytest.mark.parametrize("n,m,eps", [(600, 500, 0.01), (3000, 2500, 0.006), (3000, 2500, 0.01), (2561, 2049, 0.008)])
def test_middle_expansion_in_two_dimensions(ctx, oracle, n, m, eps):
    test_half_steps(ctx, oracle, n, m, 2, eps, "cube", "smooth")
    assert ctx.fs_debug_get("moment_kind") == 5


# Every kind of expansion, forced: rows that fill a group of a cell but for one, it and one row more (and one row, all in one cell), and
# several cells with ragged and full groups each; the widest cells that a kind allows have 2, 4 or 7 tiles of moments to themselves
@pytest.mark.parametrize("kind", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n,m,extent", [(1, 300, 0.1), (255, 40, 0.1), (256, 33, 0.1), (257, 300, 0.1), (513, 1, 0.1), (900, 1500, 1.0),
                                        (3000, 2049, 1.0)])
def test_every_kind_of_expansion(oracle, kind, n, m, extent):
    d = {1: 3, 2: 3, 3: 3, 4: 2, 5: 2, 6: 2, 7: 1}[kind]
    rng = np.random.default_rng(n + m + kind)
    x, y = ((extent * rng.random((k, d))).astype(np.float32) for k in (n, m))
    a, b = _weights(rng, n), _weights(rng, m)
    eps = float(np.float32(0.1))
    g, f = ((0.3 * rng.standard_normal(1) * v[:, 0] + eps * rng.standard_normal(len(v))).astype(np.float32) for v in (y, x))
    c = binding.Context(0)
    c.fs_debug_set("lowd_moments", 1)
    c.fs_debug_set("moment_kind", kind)
    assert c.fs_debug_get("moment_kind") == 0
    say("moments kind %d n=%d m=%d extent=%g" % (kind, n, m, extent))
    prob = make_problem(x, y, a, b)
    f1 = host(c.fs_update_f(prob, eps, dev(g)))
    assert c.fs_debug_get("moment_kind") == kind
    g1 = host(c.fs_update_g(prob, eps, dev(f)))
    fw, gw = oracle.update_f(x, y, b, eps, g), oracle.update_g(x, y, a, eps, f)
    assert max_err_over_eps(f1, fw, eps) <= _tol(fw, eps)
    assert max_err_over_eps(g1, gw, eps) <= _tol(gw, eps)
    c.close()


def test_runs_through_moments_and_falls_back(oracle):
    """Forced and left out the results differ (they are other sums); where the cells would be too many both run over the pairs."""
    rng = np.random.default_rng(3)
    n, m, eps = 1500, 1300, float(np.float32(0.1))
    for spread, differs in ((1.0, True), (40.0, False)):
        x, y = _cloud(rng, "cube", n, 3) * spread, _cloud(rng, "cube", m, 3) * spread
        a, b = _weights(rng, n), _weights(rng, m)
        g = rng.standard_normal(m).astype(np.float32) * eps
        out = []
        for mode in (1, 2):
            c = binding.Context(0)
            c.fs_debug_set("lowd_moments", mode)
            say("moments mode %d spread %g" % (mode, spread))
            out.append(host(c.fs_update_f(make_problem(x, y, a, b), eps, dev(g))))
            c.close()
        assert np.array_equal(out[0], out[1]) != differs
        assert max_err_over_eps(out[0], oracle.update_f(x, y, b, eps, g), eps) <= 1e-4


@pytest.mark.parametrize("where", ["nan", "inf", "-inf", "all -inf"])
def test_potentials_that_are_not_finite(oracle, where):
    """The same rows are NaN or infinite as over the pairs."""
    rng = np.random.default_rng(5)
    n, m, eps = 900, 800, float(np.float32(0.1))
    x, y = _cloud(rng, "cube", n, 3), _cloud(rng, "cube", m, 3)
    g = np.zeros(m, np.float32)
    g[:: 1 if where == "all -inf" else 97] = {"nan": np.nan, "inf": np.inf}.get(where, -np.inf)
    out = []
    for mode in (1, 2):
        c = binding.Context(0)
        c.fs_debug_set("lowd_moments", mode)
        say("moments mode %d potentials %s" % (mode, where))
        out.append(host(c.fs_update_f(make_problem(x, y, None, None), eps, dev(g))))
        c.close()
    same = np.isnan(out[0]) == np.isnan(out[1])
    assert same.all() and (np.isposinf(out[0]) == np.isposinf(out[1])).all() and (np.isneginf(out[0]) == np.isneginf(out[1])).all()
    ok = np.isfinite(out[0])
    if ok.any():
        assert np.max(np.abs(out[0][ok] - out[1][ok])) <= 1e-4 * eps


def test_strides_and_bf16_storage(ctx, oracle):
    rng = np.random.default_rng(9)
    n, m, eps = 1200, 1100, float(np.float32(0.05))
    x, y = workloads.to_bf16_round(_cloud(rng, "cube", n, 3)), workloads.to_bf16_round(_cloud(rng, "cube", m, 3))
    g = (0.1 * rng.standard_normal(m)).astype(np.float32)
    want = oracle.update_f(x, y, np.full(m, 1.0 / m), eps, g)
    xt = torch.zeros(n, 5, device="cuda:0", dtype=torch.bfloat16)
    xt[:, :3] = dev(x, torch.bfloat16)
    say("moments bf16 storage, strided")
    f = host(ctx.fs_update_f(binding.Problem(xt[:, :3], dev(y, torch.bfloat16), None, None), eps, dev(g)))
    assert max_err_over_eps(f, want, eps) <= _tol(want, eps) + 1e-6   # (uniform weights: log(1/m) in float64 on both sides)


@pytest.mark.parametrize("n,m,d,eps,kind", [(1100, 900, 3, 0.1, "cube"), (3000, 5000, 3, 0.3, "clusters"), (700, 600, 2, 0.05, "cube"),
                                            (400, 500, 1, 0.05, "cube"), (900, 800, 3, 0.1, "flat")])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_gradients(ctx, oracle, n, m, d, eps, kind, mode):
    """Gradients run the plan application of the other cloud's points through moments of their own."""
    rng = np.random.default_rng(n + m + d + mode)
    x, y = _cloud(rng, "cube" if kind == "clusters" else kind, n, d) - 0.5, _cloud(rng, kind, m, d) - 0.4
    a, b = _weights(rng, n), _weights(rng, m)
    eps = float(np.float32(eps))
    f, g = oracle.solve(x, y, a, b, eps, eps, 1, 5)
    f, g = f.astype(np.float32), g.astype(np.float32)
    say("moments gradient n=%d m=%d d=%d mode=%d" % (n, m, d, mode))
    prob = make_problem(x, y, a, b)
    for wrt_y in (False, True):
        z, o, w = (y, x, b) if wrt_y else (x, y, a)
        apply = oracle.apply_plan_T if wrt_y else oracle.apply_plan
        T = apply(x, y, a, b, eps, f, g, o)
        ones = apply(x, y, a, b, eps, f, g, np.ones((len(o), 1), np.float32))
        want = 2 * (w[:, None] * z - T) if mode == 0 else 2 * (ones * z - T) if mode == 1 else z - T / w[:, None]
        got = host((ctx.fs_grad_y if wrt_y else ctx.fs_grad_x)(prob, eps, dev(f), dev(g), mode))
        # sums of |entries| times |values| bound the error of T; the row factor adds the float potentials' share, which the
        # oracle has as well
        scale = np.abs(ones) * np.abs(o).max() * (2.0 if mode < 2 else 1.0 / w[:, None])
        assert np.max(np.abs(got - want) / scale) <= 2 * TOL


def test_annealed_solve(ctx, oracle):
    rng = np.random.default_rng(11)
    n, m = 2000, 1700
    x, y = _cloud(rng, "cube", n, 3), _cloud(rng, "clusters", m, 3) * 0.5 + 0.2
    a, b = _weights(rng, n), _weights(rng, m)
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    say("moments annealed solve")
    prob = make_problem(x, y.astype(np.float32), a, b)
    ctx.fs_solve(prob, 1.0, 0.03, 4, 5, f, g)
    fo, go = oracle.solve(x, y.astype(np.float32), a, b, 1.0, 0.03, 4, 5)
    eps = float(np.float32(0.03))
    assert max_err_over_eps(host(f), fo, eps) <= 1e-4 and max_err_over_eps(host(g), go, eps) <= 1e-4
    # kept copies of the clouds change nothing
    ctx.fs_points_keep(prob)
    for _ in range(2):
        f2, g2 = torch.zeros_like(f), torch.zeros_like(g)
        ctx.fs_solve(prob, 1.0, 0.03, 4, 5, f2, g2)
        assert torch.equal(f, f2) and torch.equal(g, g2)
    ctx.fs_points_release()
    err_r, err_c = ctx.fs_marginal_err(prob, eps, f, g)
    wr, wc = oracle.marginal_err(x, y.astype(np.float32), a, b, eps, host(f), host(g))
    assert abs(err_r - wr) <= 1e-5 and abs(err_c - wc) <= 1e-5


def test_large_clouds_take_moments_by_themselves():
    """Sampled rows of a half-step at a size where the library chooses, against float64 sums over all points."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(2)
    n, m = 70001, 60007
    x = torch.rand(n, 3, generator=gen, device="cuda:0")
    y = torch.rand(m, 3, generator=gen, device="cuda:0") * 0.9
    g = 0.05 * torch.randn(m, generator=gen, device="cuda:0")
    eps = float(np.float32(0.1))
    prob = binding.Problem(x, y, None, None)
    out = []
    for mode in (0, 2):
        c = binding.Context(0)
        c.fs_debug_set("lowd_moments", mode)
        say("moments by themselves, mode %d" % mode)
        out.append(c.fs_update_f(prob, eps, g))
        torch.cuda.synchronize()
        c.close()
    assert not torch.equal(out[0], out[1])
    rows = torch.arange(0, n, 97, device="cuda:0")
    xs, ys = x[rows].double(), y.double()
    s = ((g.double() - (ys * ys).sum(1)) / eps)[None, :] + 2.0 / eps * xs @ ys.t()
    want = (xs * xs).sum(1) - eps * (torch.logsumexp(s, 1) - np.log(m))
    assert float((out[0][rows].double() - want).abs().max()) / eps <= TOL + float(want.abs().max()) * 2.0 ** -24 / eps


def _gradient_error(ctx, oracle, x, y, a, b, eps, f, g, mode, wrt_y):
    """Largest error of a gradient against the oracle, in units of the sums of |entries| times the largest |coordinate|."""
    z, o, w = (y, x, b) if wrt_y else (x, y, a)
    apply = oracle.apply_plan_T if wrt_y else oracle.apply_plan
    T = apply(x, y, a, b, eps, f, g, o)
    ones = apply(x, y, a, b, eps, f, g, np.ones((len(o), 1), np.float32))
    want = 2 * (w[:, None] * z - T) if mode == 0 else 2 * (ones * z - T) if mode == 1 else z - T / w[:, None]
    got = host((ctx.fs_grad_y if wrt_y else ctx.fs_grad_x)(make_problem(x, y, a, b), eps, dev(f), dev(g), mode))
    assert np.isfinite(got).all()
    # (the weighted row itself is a term of the difference)
    scale = (np.abs(ones) + (w[:, None] if mode != 1 else 0)) * max(np.abs(o).max(), np.abs(z).max()) * (2.0 if mode < 2 else 1.0 / w[:, None])
    return float(np.max(np.abs(got - want) / scale))


@pytest.mark.parametrize("shift", [(10.0, -10.0, 3.0), (300.0, 300.0, 300.0), (1000.0, -1000.0, 0.0), (1.0e4, 1.0, -1.0e4)])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("rough", [False, True])
def test_gradients_away_from_the_origin(ctx, oracle, shift, mode, rough):
    """The values of a gradient's application are coordinates of any size, of one sign or both; rough potentials spread the weights of
    a block over e^(+-24).  2 TOL as in test_gradients, and the float result's own 2^-24."""
    rng = np.random.default_rng(21)
    n, m, eps = 900, 1100, float(np.float32(0.1))
    x = (_cloud(rng, "cube", n, 3) + np.array(shift)).astype(np.float32)
    y = (_cloud(rng, "clusters", m, 3) + np.array(shift)).astype(np.float32)
    a, b = _weights(rng, n), _weights(rng, m)
    f, g = oracle.solve(x, y, a, b, eps, eps, 1, 5)
    if rough:
        f, g = f + 8.0 * eps * rng.standard_normal(n), g + 8.0 * eps * rng.standard_normal(m)
    f, g = f.astype(np.float32), g.astype(np.float32)
    say("moments gradient shifted by %s mode=%d rough=%d" % (shift, mode, rough))
    for wrt_y in (False, True):
        assert _gradient_error(ctx, oracle, x, y, a, b, eps, f, g, mode, wrt_y) <= 2 * TOL + 2.0 ** -23


@pytest.mark.parametrize("d", [1, 2, 3])
def test_gradients_do_not_depend_on_the_scale_of_the_points(ctx, oracle, d):
    """Points times 2^k at eps times 4^k: the same gradient times 2^k, bit for bit (every scale on the way is a power of two)."""
    rng = np.random.default_rng(d)
    n, m, eps = 700, 800, 0.1
    x, y = _cloud(rng, "cube", n, d) - np.float32(0.5), _cloud(rng, "clusters", m, d) - np.float32(0.4)
    a, b = _weights(rng, n), _weights(rng, m)
    eps = float(np.float32(eps))
    f, g = oracle.solve(x, y, a, b, eps, eps, 1, 5)
    f, g = f.astype(np.float32), g.astype(np.float32)
    want = None
    for k in (0, -31, -20, 10, 20):
        s = np.float32(2.0 ** k)
        say("moments gradient d=%d points times 2^%d" % (d, k))
        got = host(ctx.fs_grad_x(make_problem(x * s, y * s, a, b), eps * 4.0 ** k, dev(f * s * s), dev(g * s * s), 2))
        if want is None:
            want = got
            assert _gradient_error(ctx, oracle, x, y, a, b, eps, f, g, 2, False) <= 2 * TOL
        else:
            assert np.array_equal(got, want * 2.0 ** k)


def test_gradients_with_values_only_where_there_is_no_weight(ctx):
    """Points at the origin that hold the weight, and others of the same cell with 2^-128 of it: what these add is nothing."""
    n, m, eps = 300, 256, float(np.float32(0.1))
    x = np.linspace(0.0, 0.02, n, dtype=np.float32).reshape(n, 1).copy()
    y = np.zeros((m, 1), np.float32)
    y[::4, 0] = np.linspace(0.005, 0.01, m // 4, dtype=np.float32)
    g = np.where(y[:, 0] > 0, -128.0 * np.log(2.0) * eps, 0.0).astype(np.float32)
    prob = make_problem(x, y, None, None)
    f = ctx.fs_update_f(prob, eps, dev(g))
    say("moments gradient, values without weight")
    got = host(ctx.fs_grad_x(prob, eps, f, dev(g), 2))
    assert np.max(np.abs(got - x)) <= 2.0 ** -30


def test_large_gradients_away_from_the_origin_take_moments_by_themselves():
    """At a size where the library chooses: the same gradient as over the pairs, whose application keeps exponentials to 2^-17, in
    units of the coordinates' size."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(4)
    n, m, eps = 70001, 60007, float(np.float32(0.1))
    x = torch.rand(n, 3, generator=gen, device="cuda:0") + 1000.0
    y = torch.rand(m, 3, generator=gen, device="cuda:0") * 0.9 + 1000.0
    prob = binding.Problem(x, y, None, None)
    out = []
    for mode in (0, 2):
        c = binding.Context(0)
        c.fs_debug_set("lowd_moments", mode)
        say("moments gradient by themselves, mode %d" % mode)
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
        c.fs_solve(prob, eps, eps, 1, 3, f, g)
        out.append(c.fs_grad_x(prob, eps, f, g, 2))
        torch.cuda.synchronize()
        c.close()
    assert bool(torch.isfinite(out[0]).all()) and not torch.equal(out[0], out[1])
    assert float((out[0] - out[1]).abs().max()) <= 1001.0 * 2.0 ** -17


def test_float64_grade_scores_stay_over_the_pairs():
    """Measurements (marginal error, dual value), small eps and many iterations ask for float64-grade scores; moments, which a few
    iterations of the same problem take, do not stand in for those: the results are those of the passes over the pairs, bit for bit."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(6)
    n, m, eps = 50021, 40013, float(np.float32(0.05))
    x, y = torch.rand(n, 3, generator=gen, device="cuda:0"), torch.rand(m, 3, generator=gen, device="cuda:0")
    x[0], y[0] = 0.0, 1.0     # |x|^2 = 0.75 after centring in both corners: scores of 2 log2(e) / 0.05 * 0.75 = 43
    prob = binding.Problem(x, y, None, None)
    zero = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")

    def both(what, call):
        out = []
        for mode in (0, 2):
            c = binding.Context(0)
            c.fs_debug_set("lowd_moments", mode)
            say("moments mode %d: %s" % (mode, what))
            out.append([float(v) if not torch.is_tensor(v) else v.clone() for v in call(c)])
            torch.cuda.synchronize()
            c.close()
        return all(torch.equal(u, v) if torch.is_tensor(u) else u == v for u, v in zip(*out)), out[0]

    def solve(c, iters):
        f, g = zero[0].clone(), zero[1].clone()
        c.fs_solve(prob, eps, eps, 1, iters, f, g)
        return f, g

    same, (f, g) = both("five iterations", lambda c: solve(c, 5))
    assert not same
    assert both("marginal errors", lambda c: c.fs_marginal_err(prob, eps, f, g))[0]
    assert both("dual value", lambda c: [c.fs_ot_value(prob, eps, f, g)])[0]
    # 140 half-steps at scores of 43 ask for float64-grade ones (Mag T > 5000), and so do scores beyond 480
    assert both("seventy iterations", lambda c: solve(c, 70))[0]
    small = float(np.float32(0.004))
    assert both("half-step at small eps", lambda c: [c.fs_update_f(prob, small, g)])[0]
    # potentials are given up to a constant, and a large one is a large score
    assert both("large potentials", lambda c: [c.fs_update_f(prob, eps, g + 300.0)])[0]


def test_cloud_narrower_than_a_float_at_its_distance(ctx, oracle):
    """Points 2e-9 apart at a distance of 0.5 from the common mean, where floats are 3e-8 apart: their potentials differ by 4e-4 eps."""
    rng = np.random.default_rng(8)
    n, m, eps = 300, 280, float(np.float32(1e-5))
    x = (2e-9 * rng.random((n, 1))).astype(np.float32)
    y = (1.0 + 5e-4 * rng.random((m, 1))).astype(np.float32)
    a, b = _weights(rng, n), _weights(rng, m)
    g = (y[:, 0].astype(np.float64) ** 2).astype(np.float32)   # (takes the cost out: f is of the size of eps)
    say("moments narrow cloud")
    got, want = host(ctx.fs_update_f(make_problem(x, y, a, b), eps, dev(g))), oracle.update_f(x, y, b, eps, g)
    assert np.ptp(want) >= 1e-4 * eps
    assert max_err_over_eps(got, want, eps) <= _tol(want, eps)


def _large(seed, n=20011, m=16001):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    x, y = torch.rand(n, 3, generator=gen, device="cuda:0"), torch.rand(m, 3, generator=gen, device="cuda:0")
    return binding.Problem(x, y, None, None)


def _taken(call, **switches):
    """What `call` returns on a new context with these switches, and how much device memory the context holds behind it."""
    c = binding.Context(0)
    for k, v in switches.items():
        c.fs_debug_set(k, v)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    out = call(c)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    c.close()
    return out, held


def test_moment_buffers_only_where_they_are_used():
    """Calls that never run through moments hold what they hold without them, and so do those that are too short for them; a solve
    holds the buffers."""
    prob, eps = _large(12), float(np.float32(0.1))
    f, g = torch.zeros(prob.n, device="cuda:0"), torch.zeros(prob.m, device="cuda:0")
    V, A = torch.rand(prob.m, 2, device="cuda:0"), torch.rand(prob.n, 3, device="cuda:0")
    calls = dict(
        symmetric=lambda c: c.fs_solve_symmetric(prob, eps, 1, f.clone(), g.clone()),
        apply=lambda c: c.fs_apply_plan(prob, eps, f, g, V),
        update=lambda c: c.fs_update_f(prob, eps, g),
        hadamard=lambda c: c.fs_apply_plan_hadamard(prob, eps, f, g, A, V),
        hvp=lambda c: c.fs_hvp(prob, eps, f, g, A, 1e-3, 1e-2, 1),
        marginals=lambda c: c.fs_marginal_err(prob, eps, f, g),
        value=lambda c: c.fs_ot_value(prob, eps, f, g))
    for name, call in calls.items():
        _taken(call)   # (what torch keeps for the outputs)
        say("moment buffers: %s" % name)
        assert _taken(call, lowd_moments=0)[1] == _taken(call, lowd_moments=2)[1]
    call = lambda c: c.fs_solve(prob, eps, eps, 1, 10, f.clone(), g.clone())
    assert _taken(call, lowd_moments=0)[1] >= _taken(call, lowd_moments=2)[1] + (64 << 20)


def test_without_memory_for_the_buffers_passes_run_over_the_pairs():
    prob, eps = _large(13), float(np.float32(0.1))

    def solve(c):
        f, g = torch.zeros(prob.n, device="cuda:0"), torch.zeros(prob.m, device="cuda:0")
        c.fs_solve(prob, eps, eps, 1, 2, f, g)
        return f, g, c.fs_grad_x(prob, eps, f, g, 2)

    _taken(solve)   # (what torch keeps for the outputs)
    say("moment buffers: none")
    pairs, held = _taken(solve, lowd_moments=2)
    forced, _ = _taken(solve, lowd_moments=1)
    assert not torch.equal(forced[0], pairs[0])
    denied, held_denied = _taken(lambda c: solve(c) and solve(c), lowd_moments=1, ws_limit=held + (1 << 20))
    assert all(torch.equal(u, v) for u, v in zip(denied, pairs)) and held_denied == held
    # what does not fit without the buffers either is still an error
    c = binding.Context(0)
    c.fs_debug_set("ws_limit", 1 << 20)
    with pytest.raises(binding.FlashSinkError):
        solve(c)
    c.fs_debug_set("ws_limit", 0)
    assert torch.equal(solve(c)[0], _taken(solve, lowd_moments=0)[0][0])
    c.close()


def test_kept_points_with_and_without_bounds():
    """Copies kept by a call without moments have no bounds of the clouds: the next half-step makes them, and results stay the same."""
    prob, eps = _large(14), float(np.float32(0.1))
    g, V = 0.01 * torch.ones(prob.m, device="cuda:0"), torch.rand(prob.m, 2, device="cuda:0")
    f = torch.zeros(prob.n, device="cuda:0")
    say("moments, kept points")
    want = _taken(lambda c: c.fs_update_f(prob, eps, g), lowd_moments=1)[0]
    plan = _taken(lambda c: c.fs_apply_plan(prob, eps, f, g, V), lowd_moments=1)[0]
    c = binding.Context(0)
    c.fs_debug_set("lowd_moments", 1)
    c.fs_points_keep(prob)
    for _ in range(3):
        assert torch.equal(c.fs_apply_plan(prob, eps, f, g, V), plan)
        assert torch.equal(c.fs_update_f(prob, eps, g), want)
    c.fs_points_release()
    c.close()


def test_profile_says_what_ran():
    """Half-steps through moments are booked as launches that evaluate no pairs, half-steps over the pairs with their pairs."""
    prob, eps = _large(15), float(np.float32(0.1))
    f, g = torch.zeros(prob.n, device="cuda:0"), torch.zeros(prob.m, device="cuda:0")
    for mode, pairs in ((1, 0.0), (2, float(prob.n) * prob.m)):
        c = binding.Context(0)
        c.fs_debug_set("lowd_moments", mode)
        c.fs_profile_enable(True)
        say("moments profile, mode %d" % mode)
        c.fs_solve(prob, eps, eps, 1, 3, f, g)
        avg, launches, per_launch = c.fs_profile_read()
        assert avg > 0.0 and launches == 6 and per_launch == pairs
        c.close()
