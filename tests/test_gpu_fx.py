"""GPU parity of the fixed-point kernels (16 < d <= 128, fp32 accuracy) against the float64 oracle, at the sizes where
they can go wrong: edges of their tiles (32 points, 128 resident rows) and k-steps (32 coordinates), both sides of the
gate that chooses between them and the fp64 kernels, tiles that take the float64 epilogue (padding,
potentials far away) or the mask (zero weights), and values and potentials that are not finite.

Tolerances: potentials to 1e-6 eps (scores are off by 2^-23 base-2 units rms at most, sums by a few 1e-8) plus the rounding of a
float output, 2^-24 |f|; applications to 1e-6 of the largest value (float values in three bf16 pieces, sums of 16
products in fp32: a few 1e-7)."""
import numpy as np
import pytest
import torch

from paper_2602_03067_amd import binding
from tests._gpu_common import dev, host, make_problem, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    c.fs_debug_set("fx_any_size", 1)   # the library itself takes small problems to the fp64 kernels
    yield c
    c.close()


def _problem(seed, n, m, d, scale=1.0):
    rng = np.random.default_rng(seed)
    x = (rng.random((n, d)) * scale).astype(np.float32)
    y = ((rng.random((m, d)) * 0.9 + 0.1) * scale).astype(np.float32)
    a = rng.random(n) + 0.1
    b = rng.random(m) + 0.1
    return rng, x, y, (a / a.sum()).astype(np.float32), (b / b.sum()).astype(np.float32)


def _check_pot(got, want, eps):
    assert np.all(np.abs(host(got) - want) <= 1e-6 * eps + 2.0 ** -24 * np.abs(want) * 1.01)


def _check_values(got, want):
    assert np.abs(host(got) - want).max() <= 1e-6 * max(np.abs(want).max(), 1e-300)


# (n, m, d): tile and row-block edges, k-step edges, the last dimension of the path and the first beyond it
SHAPES = [(1, 1, 17), (31, 33, 32), (32, 64, 33), (33, 31, 64), (127, 129, 65), (128, 96, 96), (129, 1, 97), (257, 300, 128), (65, 200, 129)]


@pytest.mark.parametrize("n,m,d", SHAPES)
# unit-cube data: thirteen products, ten, ten at the lower end of the window (2.885 / eps >= 1/2), the fp64 kernels below it
@pytest.mark.parametrize("eps", [0.02, 0.5, 5.0, 30.0])
def test_updates_and_applications(ctx, oracle, n, m, d, eps):
    eps = float(np.float32(eps))
    rng, x, y, a, b = _problem(n + 7 * m + d, n, m, d)
    prob = make_problem(x, y, a, b)
    say("fx n=%d m=%d d=%d eps=%g" % (n, m, d, eps))
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    f = oracle.update_f(x, y, b, eps, g).astype(np.float32)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), oracle.update_f(x, y, b, eps, g), eps)
    _check_pot(ctx.fs_update_g(prob, eps, dev(f)), oracle.update_g(x, y, a, eps, f), eps)
    for p in (1, 4, 5, 33, 97):
        V = rng.standard_normal((m, p)).astype(np.float32)
        U = rng.standard_normal((n, p)).astype(np.float32)
        _check_values(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))
        _check_values(ctx.fs_apply_plan_T(prob, eps, dev(f), dev(g), dev(U)), oracle.apply_plan_T(x, y, a, b, eps, f, g, U))


@pytest.mark.parametrize("scale,eps", [(1e-3, 1.0), (1.0, 0.3), (15.0, 0.1), (16.0, 0.1), (60.0, 0.3), (300.0, 0.3), (1e-30, 1e-6)])
def test_both_sides_of_the_gate(ctx, oracle, scale, eps):
    """scale^2 / eps from far below to far above the window of the fixed-point scores."""
    eps = float(np.float32(eps))
    n, m, d = 150, 190, 40
    rng, x, y, a, b = _problem(3, n, m, d, scale)
    prob = make_problem(x, y, a, b)
    say("fx gate scale=%g eps=%g" % (scale, eps))
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    want = oracle.update_f(x, y, b, eps, g)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), want, eps)
    f = want.astype(np.float32)
    V = rng.standard_normal((m, 3)).astype(np.float32)
    _check_values(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))


@pytest.mark.parametrize("offset", [0.0, 3e3, -3e3, 1e8])
def test_far_potentials_and_zero_weights(ctx, oracle, offset):
    """Biases beyond the records (a whole side, or single points of it) and points that never contribute."""
    eps = float(np.float32(0.3))
    n, m, d = 100, 400, 48
    rng, x, y, a, b = _problem(11, n, m, d)
    b[5] = b[200:264] = 0.0
    prob = make_problem(x, y, a, b)
    say("fx far potentials offset=%g" % offset)
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    g[300:] += np.float32(offset)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), oracle.update_f(x, y, b, eps, g), eps)
    g = (g + np.float32(offset)).astype(np.float32)
    f = oracle.update_f(x, y, b, eps, g).astype(np.float32)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), oracle.update_f(x, y, b, eps, g), eps)
    if offset < 1e6:   # (an offset of 1e8 leaves nothing of a float potential's difference)
        V = rng.standard_normal((m, 2)).astype(np.float32)
        _check_values(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))
        V = rng.standard_normal((m, 40)).astype(np.float32)
        _check_values(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))


def test_values_that_are_not_finite(ctx):
    """A column with an infinite or NaN value is infinite or NaN in every row it reaches, its neighbours are untouched."""
    eps = float(np.float32(1.0))
    n, m, d = 70, 90, 33
    rng, x, y, a, b = _problem(5, n, m, d)
    prob = make_problem(x, y, a, b)
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    say("fx values that are not finite")
    for p in (3, 40):
        V = rng.standard_normal((m, p)).astype(np.float32)
        clean = host(ctx.fs_apply_plan(prob, eps, f, g, dev(V)))
        V[m - 1, 0], V[40, 1], V[3, 2] = np.inf, -np.inf, np.nan
        out = host(ctx.fs_apply_plan(prob, eps, f, g, dev(V)))
        assert np.all(out[:, 0] == np.inf) and np.all(out[:, 1] == -np.inf) and np.all(np.isnan(out[:, 2]))
        assert np.array_equal(out[:, 3:], clean[:, 3:])
    # a point that is not finite turns the gate off: the fp64 kernels propagate it
    x[7, 2] = np.nan
    fu = host(ctx.fs_update_f(make_problem(x, y, a, b), eps, g))
    assert np.isnan(fu[7]) and np.isfinite(np.delete(fu, 7)).all()


@pytest.mark.parametrize("point", [66, 5])   # one in each half of a wave: bit 2 of the number within a tile
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_potentials_that_are_not_finite(ctx, point, value):
    """A NaN or +inf potential of one streamed point leaves no finite entry in any row, whatever form the product takes."""
    eps = float(np.float32(1.0))
    n, m, d = 70, 90, 33
    rng, x, y, a, b = _problem(6, n, m, d)
    prob = make_problem(x, y, a, b)
    f, g = np.zeros(n, dtype=np.float32), np.zeros(m, dtype=np.float32)
    g[point] = value
    say("fx potential %g at %d" % (value, point))
    assert not np.isfinite(host(ctx.fs_update_f(prob, eps, dev(g)))).any()
    for p in (3, 40):
        V = rng.standard_normal((m, p)).astype(np.float32)
        assert not np.isfinite(host(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)))).any()
        A = rng.standard_normal((n, d)).astype(np.float32)
        assert not np.isfinite(host(ctx.fs_apply_plan_hadamard(prob, eps, dev(f), dev(g), dev(A), dev(V)))).any()


@pytest.mark.parametrize("n,m,d", [(40, 70, 24), (130, 97, 64), (33, 129, 128)])
def test_hadamard_weights(ctx, n, m, d):
    """Rows of A of very different sizes, a zero row, columns beyond one block of 32."""
    eps = float(np.float32(0.5))
    rng, x, y, a, b = _problem(9, n, m, d)
    prob = make_problem(x, y, a, b)
    say("fx hadamard n=%d m=%d d=%d" % (n, m, d))
    A = (rng.standard_normal((n, d)) * np.exp(rng.uniform(-8, 8, (n, 1)))).astype(np.float32)
    A[1] = 0.0
    g = np.zeros(m, dtype=np.float32)
    f = host(ctx.fs_update_f(prob, eps, dev(g))).astype(np.float32)
    X, Y = x.astype(np.float64), y.astype(np.float64)
    C = ((X[:, None, :] - Y[None, :, :]) ** 2).sum(2)
    e = np.float64(eps)
    P = a[:, None].astype(np.float64) * b[None, :].astype(np.float64) * np.exp((f[:, None].astype(np.float64) + g[None, :] - C) / e)
    W = P * (A.astype(np.float64) @ Y.T)
    for p in (2, 70):
        V = rng.standard_normal((m, p)).astype(np.float32)
        got = host(ctx.fs_apply_plan_hadamard(prob, eps, dev(f), dev(g), dev(A), dev(V)))
        want = W @ V.astype(np.float64)
        # per row: the weights of a row share its scale
        scale = np.abs(W).sum(1, keepdims=True) * np.abs(V).max() + 1e-300
        assert (np.abs(got - want) / scale).max() <= 1e-6
        assert np.all(got[1] == 0.0)


# Streams of many tiles through one workgroup: what the small shapes above, where every workgroup has one tile, never reach
# (slots of the LDS ring used again, the max lifted with sums in hand, tiles with and without the float64 epilogue in turn,
# the alternating sign of the second product).
PROFILES = ["flat", "rise", "steep", "fall", "mixed", "none"]


def _stream(rng, m, eps, profile):
    """Potentials of the streamed points in units of eps, and the points without weight."""
    t = np.arange(m) // 32
    g = rng.standard_normal(m)
    dead = np.zeros(m, dtype=bool)
    if profile == "rise":        # by more than the 4 base-2 units that a running max may lag behind, every tile
        g += 8.0 * t
    elif profile == "steep":     # by more than 2^10, beyond the bias records for the later tiles
        g += 1000.0 * t
    elif profile == "fall":
        g -= 700.0 * t
    elif profile == "mixed":
        dead[[0, 3, 37]] = True                    # the first tile, and a tile after one that is whole
        dead[6 * 32:8 * 32] = True                 # tiles without any weight
        g[5 * 32 + 9] += 1.0e5                     # far above, in the middle
        g[9 * 32:9 * 32 + 3] -= 1.0e5              # far below
        g[m - 1] += 1.0e5 + 3.0                    # the last, ragged tile
        dead[10 * 32 + 5] = True                   # in a tile of its own kind after those far away
    elif profile == "none":      # nothing seen for two tiles, then in one half of the lanes only, then rising
        dead[:2 * 32] = True
        dead[[2 * 32 + i for i in range(32) if not i & 4]] = True
        dead[7 * 32 + 1::64] = True
        g += 8.0 * t
        g[4 * 32 + 6] = -np.inf
    return (g * eps).astype(np.float32), dead


@pytest.mark.parametrize("d", [20, 50, 90, 128])
@pytest.mark.parametrize("eps", [0.5, 0.03])       # ten and thirteen digit products
@pytest.mark.parametrize("splits", [1, 2])
def test_many_tiles_per_workgroup(oracle, d, eps, splits):
    n, m = 140, 13 * 32 + 7
    eps = float(np.float32(eps))
    c = binding.Context(0)
    c.fs_debug_set("fx_any_size", 1)
    c.fs_debug_set("fx_splits", splits)
    for k, profile in enumerate(PROFILES):
        rng, x, y, a, b = _problem(100 * d + k, n, m, d)
        g, dead = _stream(rng, m, eps, profile)
        b[dead] = 0.0
        prob = make_problem(x, y, a, b)
        say("fx many tiles d=%d eps=%g splits=%d %s" % (d, eps, splits, profile))
        want = oracle.update_f(x, y, b, eps, g)
        _check_pot(c.fs_update_f(prob, eps, dev(g)), want, eps)
        f = want.astype(np.float32)
        for p in (3, 40):
            V = rng.standard_normal((m, p)).astype(np.float32)
            _check_values(c.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))
        # Hadamard weights: per row, since a row's weights share a scale
        A = (rng.standard_normal((n, d)) * np.exp(rng.uniform(-3, 3, (n, 1)))).astype(np.float32)
        V = rng.standard_normal((m, 2)).astype(np.float32)
        X, Y = x.astype(np.float64), y.astype(np.float64)
        cost = ((X[:, None, :] - Y[None, :, :]) ** 2).sum(2)
        with np.errstate(over="ignore"):
            P = a[:, None].astype(np.float64) * b[None, :] * np.exp((f[:, None].astype(np.float64) + g[None, :] - cost) / np.float64(eps))
        W = P * (A.astype(np.float64) @ Y.T)
        got = host(c.fs_apply_plan_hadamard(prob, eps, dev(f), dev(g), dev(A), dev(V)))
        scale = np.abs(W).sum(1, keepdims=True) * np.abs(V).max() + 1e-300
        assert (np.abs(got - W @ V.astype(np.float64)) / scale).max() <= 1e-6
    c.close()


@pytest.mark.parametrize("n,m,d", [(140, 423, 20), (300, 97, 50), (33, 700, 90), (260, 500, 128)])
@pytest.mark.parametrize("splits", [0, 1])
def test_paired_passes(oracle, n, m, d, splits):
    """Both passes of an averaged iteration in one launch."""
    eps = float(np.float32(0.2))
    rng, x, y, a, b = _problem(n + m + d, n, m, d)
    c = binding.Context(0)
    c.fs_debug_set("fx_any_size", 1)
    c.fs_debug_set("fx_splits", splits)
    prob = make_problem(x, y, a, b)
    say("fx paired passes n=%d m=%d d=%d splits=%d" % (n, m, d, splits))
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    c.fs_solve_symmetric(prob, eps, 7, f, g)
    fo, go = oracle.solve_symmetric(x, y, a, b, eps, 7)
    for got, want in ((f, fo), (g, go)):   # (seven iterations, each adding at most its own error)
        assert np.all(np.abs(host(got) - want) <= 7e-6 * eps + 2.0 ** -24 * np.abs(want) * 1.01)
    c.close()


@pytest.mark.parametrize("d", [20, 64, 70, 128])
@pytest.mark.parametrize("kind", ["cube", "cube fine", "wide", "clusters", "no weight"])
def test_long_passes_of_a_solve(oracle, d, kind):
    """Passes of 24 tiles and more per workgroup: the running max starts at a point the last pass found, and tiles that cannot
    count are left at their leading products (how many: the tests below)."""
    n, m = 900, 35 * 32 + 5
    rng, x, y, a, b = _problem(d + len(kind), n, m, d)
    e0 = e1 = {"cube": 0.5, "cube fine": 0.03, "wide": 0.1, "clusters": 0.1, "no weight": 0.1}[kind]
    stages, iters = 1, 4
    if kind in ("wide", "no weight"):
        x = (rng.standard_normal((n, d)) * 1.5).astype(np.float32)
        y = (rng.standard_normal((m, d)) * 1.5 + 0.5).astype(np.float32)
    if kind == "clusters":      # consecutive points in one cluster of six, and stages of eps over ten and thirteen products
        centres = rng.standard_normal((6, d))
        x = (centres[np.arange(n) * 6 // n] + 0.05 * rng.standard_normal((n, d))).astype(np.float32)
        y = (centres[np.arange(m) * 6 // m] + 0.05 * rng.standard_normal((m, d))).astype(np.float32)
        e0, stages, iters = 2.0, 3, 2
    if kind == "no weight":
        b[:70] = 0.0
        b[200::7] = 0.0
        a[5 * 32:9 * 32] = 0.0
        a, b = (a / a.sum(dtype=np.float64)).astype(np.float32), (b / b.sum(dtype=np.float64)).astype(np.float32)
    e0, e1 = float(np.float32(e0)), float(np.float32(e1))
    c = binding.Context(0)
    c.fs_debug_set("fx_any_size", 1)
    c.fs_debug_set("fx_splits", 1)
    prob = make_problem(x, y, a, b)
    say("fx long passes d=%d %s" % (d, kind))
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    c.fs_solve(prob, e0, e1, stages, iters, f, g)
    fo, go = oracle.solve(x, y, a, b, e0, e1, stages, iters)
    # each half-step adds at most 1e-6 of its eps and passes on no more than it gets
    steps = 2 * iters * sum(e0 * (e1 / e0) ** (s / max(1, stages - 1)) for s in range(stages))
    for got, want in ((f, fo), (g, go)):
        err = np.abs(host(got) - want)
        say("  %.2e of %.2e" % (err.max(), 1e-6 * steps))
        assert np.all(err <= 1e-6 * steps + 2.0 ** -24 * np.abs(want) * 1.01)
    if stages == 1:
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
        c.fs_solve_symmetric(prob, e1, iters, f, g)
        fo, go = oracle.solve_symmetric(x, y, a, b, e1, iters)
        for got, want in ((f, fo), (g, go)):
            assert np.all(np.abs(host(got) - want) <= 1e-6 * steps + 2.0 ** -24 * np.abs(want) * 1.01)
    c.close()


def test_annealing_across_the_gate(ctx, oracle):
    """eps from where the weights no longer fit the bias records to where the scale is too large: the stages run on the
    fp64 kernels, on ten and on thirteen digit products, and on the fp64 kernels again."""
    n, m, d = 150, 210, 40
    rng, x, y, a, b = _problem(8, n, m, d)
    prob = make_problem(x, y, a, b)
    say("fx annealing across the gate")
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    e0, e1 = float(np.float32(200.0)), float(np.float32(2e-4))
    ctx.fs_solve(prob, e0, e1, 12, 3, f, g)
    fo, go = oracle.solve(x, y, a, b, e0, e1, 12, 3)
    # What an early half-step leaves is common to all points, (f + t, g - t), and not damped: at most 1e-6 of its eps each
    # (measured: 1.6e-8 of the first eps).  The rest is damped by the half-steps after it.
    t = float(np.median(host(f) - fo))
    steps = 6 * sum(e0 * (e1 / e0) ** (s / 11) for s in range(12))
    say("  common shift %.2e" % t)
    assert abs(t) <= 1e-6 * steps
    ulp = 2.0 ** -23 * max(np.abs(fo).max(), np.abs(go).max()) * 1.01   # of the potential itself, and of those t is taken from
    for got, want, sign in ((f, fo, 1.0), (g, go, -1.0)):
        assert np.abs(host(got) - sign * t - want).max() <= 1e-5 * e1 + ulp


def _borrowed():
    from tests import test_gpu_edge as e, test_gpu_f64 as q, test_gpu_grad as r, test_gpu_hadamard as h, test_gpu_hvp as w
    from tests import test_gpu_labels as l, test_gpu_schedules as s, test_gpu_value as v
    return {
        "half steps": (q.test_single_half_steps, (300, 500, 64)),
        "half steps d=33": (q.test_single_half_steps, (129, 1000, 33)),
        "bf16 storage": (q.test_bf16_storage_in_fp32_mode, ()),
        "trajectory": (q.test_transport_grad_trajectory_scaled_down, ()),
        "apply": (q.test_apply_shapes, (257, 190, 40, 70)),
        "apply wide": (q.test_apply_shapes, (150, 333, 100, 200)),
        "gradients": (r.test_gradients_all_modes, (200, 333, 64, "fp32")),
        "strides": (e.test_row_strides_larger_than_the_rows, (40, "fp32", 1e-4)),
        "one context": (e.test_one_context_many_problems, ()),
        "kept copies": (e.test_kept_derived_copies_change_nothing, (40, "fp32")),
        "hadamard": (h.test_hadamard_transport_matches_dense_oracle, (150, 260, 64, 7, 6.0, 10, 0.2)),
        "hvp": (w.test_hvp_matches_dense_oracle, (150, 260, 64, 6.0, 30)),
        "labels": (l.test_labeled_cost_matches_dense_sinkhorn_on_the_explicit_cost, (200, 330, 40, 10, "fp32", 0.5, 0.5)),
        "tolerance": (s.test_solve_tol_stops_where_the_oracle_does, (300, 260, 40, 0.15)),
        "few rows": (s.test_few_rows_many_columns, (64, "fp32")),
        "value": (v.test_value_matches_oracle_dual, (130, 257, 64, 1.0, 5)),
        "divergence": (v.test_divergence_entry_point, (180, 410, 24, 0.5, 15)),
    }


@pytest.mark.parametrize("name", ["half steps", "half steps d=33", "bf16 storage", "trajectory", "apply", "apply wide", "gradients",
                                  "strides", "one context", "kept copies", "hadamard", "hvp", "labels", "tolerance", "few rows",
                                  "value", "divergence"])
def test_entry_points_on_fixed_point_scores(ctx, oracle, monkeypatch, name):
    """Tests of the other files, whose problems are small enough for the fp64 kernels, on the fixed-point ones."""
    import inspect
    make = binding.Context

    def with_switch(*args, **kw):
        c = make(*args, **kw)
        c.fs_debug_set("fx_any_size", 1)
        return c

    monkeypatch.setattr(binding, "Context", with_switch)
    fn, args = _borrowed()[name]
    names = list(inspect.signature(fn).parameters)
    given = [{"ctx": ctx, "oracle": oracle}[k] for k in names if k in ("ctx", "oracle")]
    fn(*given, *args)


def test_noalloc_without_room_for_digits():
    """A solve whose digit images do not fit the static scratch array runs on the fp64 kernels there."""
    n, d = 20000, 64
    eps = float(np.float32(0.1))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    x, y = torch.rand(n, d, generator=gen, device="cuda:0"), torch.rand(n, d, generator=gen, device="cuda:0")
    c = binding.Context(0)
    prob = binding.Problem(x, y)
    say("fx noalloc n=m=%d d=%d" % (n, d))
    out = []
    for solve in (c.fs_solve, c.fs_solve_noalloc):
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0")
        solve(prob, eps, eps, 1, 2, f, g)
        out.append((host(f), host(g)))
    c.close()
    for u, v in zip(*out):   # four half-steps on either side, and the rounding of two float outputs
        assert np.all(np.abs(u - v) <= 8e-6 * eps + 2.0 ** -23 * np.abs(u) * 1.01)


@pytest.mark.parametrize("offset", [-5.0, 40.0, 1000.0])
@pytest.mark.parametrize("eps", [0.3, 0.01])   # fixed point, and beyond the gate
def test_clouds_far_from_the_origin(ctx, oracle, offset, eps):
    """The digits are those of the shifted points: potentials, applications and, where the points themselves enter, Hadamard
    weights, whose rows sum to nearly nothing here so that the shift's share of a weight is large and cancels."""
    eps = float(np.float32(eps))
    n, m, d = 130, 170, 40
    rng, x, y, a, b = _problem(17, n, m, d, 4.0)
    x, y = (x + np.float32(offset)).astype(np.float32), (y + np.float32(offset)).astype(np.float32)
    prob = make_problem(x, y, a, b)
    say("fx offset %g eps=%g" % (offset, eps))
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    want = oracle.update_f(x, y, b, eps, g)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), want, eps)
    f = want.astype(np.float32)
    V = rng.standard_normal((m, 9)).astype(np.float32)
    _check_values(ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V)), oracle.apply_plan(x, y, a, b, eps, f, g, V))
    A = rng.standard_normal((n, d)).astype(np.float32)
    A -= A.mean(1, keepdims=True)
    X, Y = x.astype(np.float64), y.astype(np.float64)
    cost = ((X[:, None, :] - Y[None, :, :]) ** 2).sum(2)
    W = a[:, None].astype(np.float64) * b[None, :] * np.exp((f[:, None].astype(np.float64) + g[None, :] - cost) / np.float64(eps))
    W *= A.astype(np.float64) @ Y.T
    got = host(ctx.fs_apply_plan_hadamard(prob, eps, dev(f), dev(g), dev(A), dev(V)))
    scale = np.abs(W).sum(1, keepdims=True) * np.abs(V).max()
    assert (np.abs(got - W @ V.astype(np.float64)) / scale).max() <= 1e-6


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["pixels", "two values", "one direction", "normal"])
def test_plan_sums_of_data_with_regular_digits(ctx, oracle, d, kind):
    """Coordinates whose base-256 digits repeat (k / 255, a single constant): the digit products left out add up instead of
    averaging out.  Plan sums at the upper end of ten products, a little above it, and at the upper end of the gate stay at
    what the fp64 kernels leave (4e-8 to 4e-7 for these).  Points along one direction are the exception: a point within
    2^-7 of the range from the origin, one in 64, has all its d coordinates rounded the same way, by at most 2^-32 of the
    scale, which against a point at the far end is d 2^-31 v base-2 units of a score."""
    n, m = 200, 333
    rng = np.random.default_rng(d)

    def cloud(k):
        if kind == "pixels":
            return rng.integers(0, 256, (k, d)) / 255.0
        if kind == "two values":
            return 0.7 * rng.integers(0, 2, (k, d))
        if kind == "one direction":
            return np.ones((k, d)) * rng.random((k, 1))
        return rng.standard_normal((k, d))

    x, y = cloud(n).astype(np.float32), cloud(m).astype(np.float32)
    half = 0.5 * (max(x.max(), y.max()) - min(x.min(), y.min()))
    r2 = 2.0 ** np.frexp(half * 128 / 126.99)[1]
    a, b = np.full(n, 1.0 / n, dtype=np.float32), np.full(m, 1.0 / m, dtype=np.float32)
    for v in (30.0, 40.0, 2000.0):
        eps = float(np.float32(2.0 / np.log(2.0) * r2 * r2 / v))
        fo, go = oracle.solve(x, y, a, b, eps, eps, 1, 3)
        f, g = fo.astype(np.float32), go.astype(np.float32)
        prob = make_problem(x, y, a, b)
        say("fx digits %s d=%d v=%g eps=%.4g" % (kind, d, v, eps))
        for p in (1, 5):
            got, mass = ctx.fs_apply_plan(prob, eps, dev(f), dev(g), torch.ones(m, p, device="cuda:0"), want_mass=True)
            want = oracle.apply_plan(x, y, a, b, eps, f, g, np.ones((m, p), dtype=np.float32))
            e = [np.linalg.norm(host(got) - want) / np.linalg.norm(want), np.linalg.norm(host(mass) - want[:, 0]) / np.linalg.norm(want[:, 0])]
            say("  p=%d sums %.2e mass %.2e" % (p, *e))
            assert max(e) <= 2.5e-7 + (np.log(2.0) * d * 2.0 ** -31 * v / 64 if kind == "one direction" else 0.0)


@pytest.mark.parametrize("p", [1, 4, 70])
def test_merge_of_an_application_beyond_the_gate(ctx, oracle, p):
    """The fp64 kernel's accumulator rows are longer than those the merge's grid is made for; more rows than one round of it."""
    n, m, d = 9001, 40, 20
    eps = float(np.float32(1e-4))
    rng, x, y, a, b = _problem(23, n, m, d)
    prob = make_problem(x, y, a, b)
    say("fx merge beyond the gate p=%d" % p)
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    f = oracle.update_f(x, y, b, eps, g).astype(np.float32)
    V = rng.standard_normal((m, p)).astype(np.float32)
    got, mass = ctx.fs_apply_plan(prob, eps, dev(f), dev(g), dev(V), want_mass=True)
    want, r = oracle.apply_plan(x, y, a, b, eps, f, g, V, return_mass=True)
    _check_values(got, want)
    _check_values(mass, r)


def test_half_steps_beyond_the_gate_with_many_row_blocks(ctx, oracle):
    """More (row block, split) pairs than the fp64 kernel beside the fixed-point one has workgroups: each takes several."""
    n, m, d = 40003, 70, 20
    eps = float(np.float32(1e-4))
    rng, x, y, a, b = _problem(29, n, m, d)
    prob = make_problem(x, y, a, b)
    say("fx many row blocks beyond the gate")
    g = (rng.standard_normal(m) * eps).astype(np.float32)
    f = oracle.update_f(x, y, b, eps, g)
    _check_pot(ctx.fs_update_f(prob, eps, dev(g)), f, eps)
    _check_pot(ctx.fs_update_g(prob, eps, dev(f.astype(np.float32))), oracle.update_g(x, y, a, eps, f.astype(np.float32)), eps)
    fs, gs = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    ctx.fs_solve_symmetric(prob, eps, 3, fs, gs)
    fo, go = oracle.solve_symmetric(x, y, a, b, eps, 3)
    for got, want in ((fs, fo), (gs, go)):
        assert np.all(np.abs(host(got) - want) <= 3e-6 * eps + 2.0 ** -24 * np.abs(want) * 1.01)


@pytest.mark.parametrize("n,m,d", [(300, 4000, 24), (2000, 700, 100)])
def test_workspace_covers_every_pass_of_a_wide_application(ctx, n, m, d):
    """The passes of one call differ in width, workgroups per CU and so in splits; the buffer is sized from the first and
    the last.  Column by column the same as one column at a time (to rounding: those run on the vector ALU)."""
    eps = float(np.float32(0.5))
    rng, x, y, a, b = _problem(31, n, m, d)
    prob = make_problem(x, y, a, b)
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    f = ctx.fs_update_f(prob, eps, g)
    V, A = rng.standard_normal((m, 333)).astype(np.float32), dev(rng.standard_normal((n, d)).astype(np.float32))
    one = host(ctx.fs_apply_plan(prob, eps, f, g, dev(V[:, :3].copy())))
    for p in (5, 33, 64, 65, 96, 97, 127, 128, 129, 132, 133, 160, 192, 193, 200, 256, 257, 333):
        say("fx wide application n=%d m=%d d=%d p=%d" % (n, m, d, p))
        out = host(ctx.fs_apply_plan(prob, eps, f, g, dev(V[:, :p].copy())))
        assert np.abs(out[:, :3] - one).max() <= 1e-6 * np.abs(one).max()
        assert np.isfinite(out).all()
        assert np.isfinite(host(ctx.fs_apply_plan_hadamard(prob, eps, f, g, A, dev(V[:, :p].copy())))).all()


def _long_context(stream=None):
    """Half-steps of 24 tiles and more a workgroup at small sizes."""
    c = binding.Context(0, stream)
    c.fs_debug_set("fx_any_size", 1)
    c.fs_debug_set("fx_splits", 1)
    return c


def _check_solve(got, want, eps, iters):
    """Each half-step adds at most 1e-6 of its eps and passes on no more than it gets."""
    for u, v in zip(got, want):
        assert np.all(np.abs(host(u) - v) <= 2e-6 * iters * eps + 2.0 ** -24 * np.abs(v) * 1.01)


def _long_clouds(kind, n, m, d):
    """Clouds, weights and eps by what a long half-step may leave of them."""
    rng, x, y, a, b = _problem(d + len(kind), n, m, d)
    e0 = e1 = {"cube": 0.5, "cube fine": 0.03}.get(kind, 0.1)
    if kind == "wide":
        x = (rng.standard_normal((n, d)) * 1.5).astype(np.float32)
        y = (rng.standard_normal((m, d)) * 1.5 + 0.5).astype(np.float32)
    if kind == "clusters":
        centres = rng.standard_normal((6, d))
        x = (centres[np.arange(n) * 6 // n] + 0.05 * rng.standard_normal((n, d))).astype(np.float32)
        y = (centres[np.arange(m) * 6 // m] + 0.05 * rng.standard_normal((m, d))).astype(np.float32)
    return x, y, a, b, float(np.float32(e1))


# three splits of 25 tiles a side; 14 splits of a few rows (more than the twelve that are looked through at once), against one or two
# tiles a workgroup of the other side
@pytest.mark.parametrize("n,m,splits", [(2400, 2390, 3), (200, 14 * 24 * 32 + 5, 14)])
@pytest.mark.parametrize("d", [20, 64, 70, 128])
@pytest.mark.parametrize("kind", ["cube", "cube fine", "wide", "clusters"])
def test_long_passes_over_several_splits(oracle, n, m, splits, d, kind):
    """The best of several splits' starts, from either lane half and from the first pass's own: solves of both schedules at the bounds of
    one split, and how many tiles are left early: none of a cube's, some of wide clouds', and of clusters in a row most of those out of
    reach."""
    iters = 3
    x, y, a, b, eps = _long_clouds(kind, n, m, d)
    c = binding.Context(0)
    c.fs_debug_set("fx_any_size", 1)
    c.fs_debug_set("fx_long", 1)
    c.fs_debug_set("fx_splits", splits)
    c.fs_debug_set("fx_count", 1)
    prob = make_problem(x, y, a, b)
    say("fx long passes n=%d m=%d splits=%d d=%d %s" % (n, m, splits, d, kind))
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    c.fs_solve(prob, eps, eps, 1, iters, f, g)
    tiles, left = c.fs_debug_get("fx_tiles"), c.fs_debug_get("fx_tiles_left")
    rows = [-(-k // 128) * 4 for k in (n, m)]
    assert tiles == iters * (rows[0] * -(-m // 32) + rows[1] * -(-n // 32))
    say("  %.3f of the tiles left" % (left / tiles))
    if kind == "cube":
        assert left == 0
    if kind == "wide":
        assert left > 0
    if kind == "clusters":   # (from the second pass over a side on; a tile of rows or points may lie in two clusters)
        assert left >= (iters - 1) / iters * (5 / 6 - 0.35) * tiles
    _check_solve((f, g), oracle.solve(x, y, a, b, eps, eps, 1, iters), eps, iters)
    f.zero_()
    g.zero_()
    c.fs_debug_set("fx_count", 0)
    c.fs_solve_symmetric(prob, eps, iters, f, g)
    _check_solve((f, g), oracle.solve_symmetric(x, y, a, b, eps, iters), eps, iters)
    c.close()


def test_early_tiles_change_nothing_that_is_seen():
    """Clouds many of whose tiles are left early, against passes that leave none: the same to the rounding of the potentials."""
    n, m, d, iters = 900, 35 * 32 + 5, 64, 4
    for kind in ("wide", "clusters"):
        x, y, a, b, eps = _long_clouds(kind, n, m, d)
        out = []
        for long in (1, 2):
            c = _long_context()
            c.fs_debug_set("fx_long", long)
            c.fs_debug_set("fx_count", 1)
            say("fx long=%d %s" % (long, kind))
            f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
            c.fs_solve(make_problem(x, y, a, b), eps, eps, 1, iters, f, g)
            tiles, left = c.fs_debug_get("fx_tiles"), c.fs_debug_get("fx_tiles_left")
            say("  %d of %d tiles left" % (left, tiles))
            assert (left > 0.05 * tiles) if long == 1 else tiles == 0
            out.append((host(f), host(g)))
            c.close()
        for u, v in zip(*out):
            assert np.all(np.abs(u - v) <= 4e-6 * iters * eps + 2.0 ** -23 * np.abs(u) * 1.01)


def test_long_passes_across_the_gate(oracle):
    """Stages of eps on the fp64 kernels, on ten and on thirteen products and on the fp64 kernels again, in long half-steps: starts that a
    pass on the other kernels left behind are none."""
    n, m, d = 900, 35 * 32 + 5, 40
    rng, x, y, a, b = _problem(8, n, m, d)
    prob = make_problem(x, y, a, b)
    e0, e1, stages, iters = float(np.float32(200.0)), float(np.float32(2e-4)), 12, 2
    fo, go = oracle.solve(x, y, a, b, e0, e1, stages, iters)
    steps = 2 * iters * sum(e0 * (e1 / e0) ** (s / (stages - 1)) for s in range(stages))
    ulp = 2.0 ** -23 * max(np.abs(fo).max(), np.abs(go).max()) * 1.01
    for splits in (1, 2):
        c = _long_context()
        c.fs_debug_set("fx_splits", splits)
        c.fs_debug_set("fx_long", 1)
        say("fx long passes across the gate, splits=%d" % splits)
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
        c.fs_solve(prob, e0, e1, stages, iters, f, g)
        t = float(np.median(host(f) - fo))   # (common to all points and not damped, see test_annealing_across_the_gate)
        say("  common shift %.2e" % t)
        assert abs(t) <= 1e-6 * steps
        for got, want, sign in ((f, fo, 1.0), (g, go, -1.0)):
            assert np.abs(host(got) - sign * t - want).max() <= 1e-5 * e1 + ulp
        c.close()


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("where", ["nan", "inf", "-inf", "all -inf", "far"])
def test_long_passes_with_potentials_that_are_not_finite(where, splits):
    """Half-steps and solves from such potentials: what is not finite is what it is in short half-steps, the rest agrees."""
    n, m, d, iters = 900, 35 * 32 + 5, 40, 3
    x, y, a, b, eps = _long_clouds("wide", n, m, d)
    g0 = np.zeros(m, np.float32)
    if where == "all -inf":
        g0[:] = -np.inf
    else:
        g0[[5, 700, m - 1]] = {"nan": np.nan, "inf": np.inf, "-inf": -np.inf, "far": -3e6}[where]
    prob = make_problem(x, y, a, b)
    out = []
    for long in (1, 2):
        c = _long_context()
        c.fs_debug_set("fx_splits", splits)
        c.fs_debug_set("fx_long", long)
        say("fx long=%d %s splits=%d" % (long, where, splits))
        f, g = torch.zeros(n, device="cuda:0"), dev(g0)
        one = host(c.fs_update_f(prob, eps, g))
        c.fs_solve(prob, eps, eps, 1, iters, f, g)
        out.append((one, host(f), host(g)))
        c.close()
    for u, v in zip(*out):
        assert np.array_equal(np.isnan(u), np.isnan(v)) and np.array_equal(np.isposinf(u), np.isposinf(v))
        assert np.array_equal(np.isneginf(u), np.isneginf(v))
        ok = np.isfinite(u)
        assert np.all(np.abs(u[ok] - v[ok]) <= 4e-6 * iters * eps + 2.0 ** -23 * np.abs(u[ok]) * 1.01)


@pytest.mark.parametrize("splits", [1, 2])
def test_long_passes_with_early_stopping(oracle, splits):
    """fs_solve_tol looks at the error between half-steps of one call: the iterations and potentials of the oracle."""
    n, m, d, iters = 900, 35 * 32 + 5, 40, 5
    for kind in ("cube", "clusters"):
        x, y, a, b, eps = _long_clouds(kind, n, m, d)
        c = _long_context()
        c.fs_debug_set("fx_splits", splits)
        c.fs_debug_set("fx_long", 1)
        say("fx long passes, early stopping, %s splits=%d" % (kind, splits))
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
        done, err = c.fs_solve_tol(make_problem(x, y, a, b), eps, iters, 2, 0.0, f, g)
        want = oracle.solve(x, y, a, b, eps, eps, 1, iters)
        assert done == iters and abs(err - oracle.marginal_err(x, y, a, b, eps, *want)[0]) <= 1e-5
        _check_solve((f, g), want, eps, iters)
        c.close()


def test_recorded_solve_after_other_calls(oracle):
    """A solve that is recorded into a graph runs in the workspace that other calls on the problem have left: what it would hold beside
    (starts of the running max) is not worth an allocation that cannot be made then."""
    n, m, d, eps, iters = 900, 35 * 32 + 5, 40, float(np.float32(0.1)), 3
    rng, x, y, a, b = _problem(3, n, m, d)
    stream = torch.cuda.Stream()
    c = _long_context(stream)
    prob = make_problem(x, y, a, b)
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    torch.cuda.synchronize()
    say("fx recorded solve")
    c.fs_update_f(prob, eps, g)
    c.fs_update_g(prob, eps, f)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        c.fs_solve(prob, eps, eps, 1, iters, f, g)
    want = oracle.solve(x, y, a, b, eps, eps, 1, iters)
    first = None
    for k in range(4):
        say("  replay %d" % k)
        f.fill_(float(k))
        g.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _check_solve((f, g), want, eps, iters)
        first = (host(f), host(g)) if first is None else first
        assert np.array_equal(host(f), first[0]) and np.array_equal(host(g), first[1])
    del graph
    c.close()


def test_solves_where_there_is_no_memory_for_starts(oracle):
    """Without memory for the starts of the running max a solve takes as much workspace as a half-step and leaves what there is alone:
    the kept copies of the clouds survive it, the first time and afterwards."""
    n, m, d, eps, iters = 900, 35 * 32 + 5, 40, float(np.float32(0.1)), 3
    rng, x, y, a, b = _problem(4, n, m, d)
    xd, yd = dev(x), dev(y)
    prob = binding.Problem(xd, yd, dev(a), dev(b))
    g0 = torch.zeros(m, device="cuda:0")

    def fits(limit):
        c = _long_context()
        c.fs_debug_set("ws_limit", limit)
        try:
            c.fs_update_f(prob, eps, g0)
            return True
        except binding.FlashSinkError as e:
            assert e.status == 6
            return False
        finally:
            c.close()

    lo, hi = 0, 1 << 28
    while hi - lo > 256:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid) else (mid, hi)
    say("fx solves in %d bytes" % hi)
    c = _long_context()
    c.fs_debug_set("ws_limit", hi)
    c.fs_points_keep(prob)
    old = host(c.fs_update_f(prob, eps, g0))
    want = oracle.solve(x, y, a, b, eps, eps, 1, iters)
    xd.mul_(2.0)
    for k in range(2):   # (from the copies of the old coordinates)
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
        c.fs_solve(prob, eps, eps, 1, iters, f, g)
        _check_solve((f, g), want, eps, iters)
    assert np.array_equal(host(c.fs_update_f(prob, eps, g0)), old)
    xd.mul_(0.5)
    c.fs_points_release()
    c.fs_debug_set("ws_limit", 0)
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    c.fs_solve(prob, eps, eps, 1, iters, f, g)
    _check_solve((f, g), want, eps, iters)
    c.close()


def test_starts_of_many_row_blocks_and_splits():
    """The starts of the running max are there at every launch shape: where many row blocks meet many splits (13 here), most tiles of
    clouds of consecutive clusters are left early, and the result is that of passes that leave none."""
    n, d, eps, iters = 30000, 32, float(np.float32(0.1)), 3
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    centres = torch.randn(8, d, generator=gen, device="cuda:0")
    x, y = (centres[torch.arange(n, device="cuda:0") * 8 // n] + 0.05 * torch.randn(n, d, generator=gen, device="cuda:0") for _ in range(2))
    prob = binding.Problem(x, y)
    say("fx starts of many splits n=m=%d" % n)
    out = []
    for long in (0, 2):
        c = binding.Context(0)
        c.fs_debug_set("fx_long", long)
        c.fs_debug_set("fx_count", 1)
        f, g = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0")
        c.fs_solve(prob, eps, eps, 1, iters, f, g)
        tiles, left = c.fs_debug_get("fx_tiles"), c.fs_debug_get("fx_tiles_left")
        say("  %d of %d tiles left" % (left, tiles))
        if long == 0:
            assert tiles == 2 * iters * 940 * 938   # (235 row blocks of four waves, 938 tiles)
            # (seven clusters of eight are out of reach from the second pass over a side on)
            assert left >= 0.8 * (iters - 1) / iters * 7 / 8 * tiles
        else:
            assert tiles == 0
        out.append((f, g))
        c.close()
    for u, v in zip(*out):
        assert float((u - v).abs().max()) <= 2 * 2e-6 * iters * eps + 2.0 ** -23 * float(u.abs().max()) * 1.01


@pytest.mark.parametrize("d,n,m", [(30, 9000, 8923), (100, 9000, 8923), (100, 7000, 6923), (128, 15000, 14923), (100, 25000, 6000)])
def test_every_form_of_long_half_steps_by_itself(d, n, m):
    """Sizes at which the library chooses each form of its own accord (three and two workgroups per CU, none, alone, in solves and in pairs),
    against forced short half-steps: the same to the rounding of the potentials."""
    eps, iters = float(np.float32(0.1)), 3
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n + d)
    x, y = torch.randn(n, d, generator=gen, device="cuda:0"), torch.randn(m, d, generator=gen, device="cuda:0") + 0.5
    prob = binding.Problem(x, y)
    say("fx forms n=%d m=%d d=%d" % (n, m, d))
    out = []
    for long in (0, 2):
        c = binding.Context(0)
        c.fs_debug_set("fx_long", long)
        f, g = torch.zeros(prob.n, device="cuda:0"), torch.zeros(prob.m, device="cuda:0")
        got = [c.fs_update_f(prob, eps, g), c.fs_update_g(prob, eps, f)]
        for solve in (lambda: c.fs_solve(prob, eps, eps, 1, iters, f, g), lambda: c.fs_solve_symmetric(prob, eps, iters, f, g)):
            f.zero_()
            g.zero_()
            solve()
            got += [f.clone(), g.clone()]
        out.append([host(v) for v in got])
        c.close()
    for u, v in zip(*out):
        assert np.all(np.abs(u - v) <= 4e-6 * iters * eps + 2.0 ** -23 * np.abs(u) * 1.01)
