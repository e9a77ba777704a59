"""fs_solve_noalloc (the entry point for callers that cannot allocate device memory) against fs_solve and
the float64 oracle, through the C ABI: two calls in a row on one context, the second on a smaller problem, so
that the second runs in a static scratch array that still holds the first call's data."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2602_03067_amd import binding, workloads
from tests._gpu_common import host, max_err_over_eps, say

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _solve(lib, h, name, prob, w, f, g):
    fn = getattr(lib, name)
    st = fn(h, ctypes.byref(prob.c), ctypes.c_float(w.eps_start), ctypes.c_float(w.eps_end), w.n_stages, w.iters,
            ctypes.c_void_p(f.data_ptr()), ctypes.c_void_p(g.data_ptr()))
    assert st == 0, (name, st, lib.fs_last_error(h))
    torch.cuda.synchronize()


def test_noalloc_solve_matches_solve_twice_in_a_row(oracle):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = binding.Context(0)
    lib, h = ctx.lib, ctx.h
    # annealed low-dimension problem (several stages, both score arithmetics), then a smaller fixed-eps one
    cases = [workloads.make("lowdim_anneal", n=3000, m=2600, iters=3), workloads.make("tiny", n=700, m=900, iters=12)]
    for k, w in enumerate(cases):
        prob = binding.problem_from_workload(w)
        f0, g0 = torch.zeros(w.n, device="cuda:0"), torch.zeros(w.m, device="cuda:0")
        f1, g1 = torch.zeros(w.n, device="cuda:0"), torch.zeros(w.m, device="cuda:0")
        say("fs_solve_noalloc call %d: %s n=%d m=%d d=%d stages=%d iters=%d" % (k + 1, w.name, w.n, w.m, w.d, w.n_stages, w.iters))
        _solve(lib, h, "fs_solve_noalloc", prob, w, f1, g1)
        _solve(lib, h, "fs_solve", prob, w, f0, g0)
        eps = float(np.float32(w.eps_end))
        ef = max_err_over_eps(host(f1), host(f0), eps)
        eg = max_err_over_eps(host(g1), host(g0), eps)
        fo, go = oracle.solve(w.x, w.y, w.a, w.b, w.eps_start, w.eps_end, w.n_stages, w.iters)
        of = max_err_over_eps(host(f1), fo, eps)
        og = max_err_over_eps(host(g1), go, eps)
        say("  against fs_solve: max|df|/eps=%.3e max|dg|/eps=%.3e; against the oracle: %.3e %.3e" % (ef, eg, of, og))
        assert ef <= TOL and eg <= TOL
        assert of <= TOL and og <= TOL
    ctx.close()


def test_noalloc_solve_refuses_what_does_not_fit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = binding.Context(0)
    n = 70000                      # beyond the static scratch at d = 3
    x = torch.rand(n, 3, device="cuda:0")
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0")
    prob = binding.Problem(x, x.clone())
    say("fs_solve_noalloc refuses n=m=%d, d=3" % n)
    with pytest.raises(binding.FlashSinkError) as ei:
        ctx.fs_solve_noalloc(prob, 0.1, 0.1, 1, 1, f, g)
    assert ei.value.status == 2 and "fs_solve_noalloc" in str(ei.value)
    assert float(f.abs().max()) == 0.0 and float(g.abs().max()) == 0.0     # nothing was launched
    ctx.close()


def test_graph_of_a_noalloc_solve_outlives_its_context(oracle):
    """A recorded fs_solve_noalloc refers to the caller's tensors and the static scratch array only, so its graph may be replayed after
    the context is gone, on whatever the tensors hold then: every replay is the eager call bit for bit."""
    rng = np.random.default_rng(11)
    n, m, d = 700, 900, 40
    eps = float(np.float32(0.3))
    stream = torch.cuda.Stream()
    x, y = torch.empty(n, d, device="cuda:0"), torch.empty(m, d, device="cuda:0")
    f, g = torch.zeros(n, device="cuda:0"), torch.zeros(m, device="cuda:0")
    prob = binding.Problem(x, y)
    clouds = [(rng.random((n, d)).astype(np.float32), rng.random((m, d)).astype(np.float32)) for _ in range(3)]

    def fill(k):
        x.copy_(torch.from_numpy(clouds[k][0]))
        y.copy_(torch.from_numpy(clouds[k][1]))
        f.zero_()
        g.zero_()
        torch.cuda.synchronize()

    say("graph of fs_solve_noalloc n=%d m=%d d=%d" % (n, m, d))
    ctx = binding.Context(0, stream)
    ctx.fs_debug_set("fx_any_size", 1)
    want = []
    for k in range(3):
        fill(k)
        ctx.fs_solve_noalloc(prob, eps, eps, 1, 3, f, g)
        torch.cuda.synchronize()
        want.append((host(f), host(g)))
    fo, go = oracle.solve(clouds[2][0], clouds[2][1], np.full(n, 1.0 / n), np.full(m, 1.0 / m), eps, eps, 1, 3)
    assert max_err_over_eps(want[2][0], fo, eps) <= TOL and max_err_over_eps(want[2][1], go, eps) <= TOL
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.fs_solve_noalloc(prob, eps, eps, 1, 3, f, g)
    ctx.close()
    for k in (0, 1, 2, 0):
        say("  replay on clouds %d" % k)
        fill(k)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(f), want[k][0]) and np.array_equal(host(g), want[k][1])


def test_contexts_share_the_words_of_the_static_scratch():
    """The scalars that come to the host in fs_solve_noalloc pass through one pinned box a GPU: calls of two contexts in turn, with
    ordinary calls (whose box is the context's own) between them, give what they give alone."""
    rng = np.random.default_rng(12)
    ctxs = [binding.Context(0) for _ in range(2)]
    cases = []
    for n, m, d in ((300, 200, 3), (250, 310, 40)):
        x, y = (torch.from_numpy(rng.random((k, d)).astype(np.float32)).to("cuda:0") for k in (n, m))
        cases.append(binding.Problem(x, y))
    for c in ctxs:
        c.fs_debug_set("fx_any_size", 1)

    def solve(c, prob, name):
        f, g = torch.zeros(prob.n, device="cuda:0"), torch.zeros(prob.m, device="cuda:0")
        getattr(c, name)(prob, 0.3, 0.3, 1, 3, f, g)
        return host(f), host(g)

    say("shared pinned box")
    want = [solve(ctxs[0], p, "fs_solve_noalloc") for p in cases]
    for k in range(12):
        p = (k + k // 4) % 2
        got = solve(ctxs[k % 2], cases[p], ("fs_solve", "fs_solve_noalloc", "fs_solve_noalloc")[k % 3])
        assert max(np.abs(u - v).max() for u, v in zip(got, want[p])) <= (0.0 if k % 3 else 1e-5)
    for c in ctxs:
        c.close()


def test_a_context_costs_next_to_nothing():
    """fs_create and fs_destroy take no memory of the GPU's or pinned: 1.3 us together, 20 with a pinned page."""
    import time
    lib, stream = binding.load_library(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    took = []
    say("contexts made and destroyed")
    for _ in range(300):
        h = ctypes.c_void_p()
        t0 = time.perf_counter()
        assert lib.fs_create(ctypes.byref(h), 0, stream) == 0 and lib.fs_destroy(h) == 0
        took.append(time.perf_counter() - t0)
    say("  %.2f us" % (np.median(took) * 1e6))
    assert np.median(took) <= 8e-6
