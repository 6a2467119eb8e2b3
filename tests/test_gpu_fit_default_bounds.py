"""cat_fit on matrices large enough for its loop to leave rows out by distance bounds (from 64 MB on; 32 MB with two launches
per pass), against the loop that runs every pass over every row.

Centroids, assignments and counts are the same bit for bit.  The objective of the plain loop is a sum of float32 terms
|x|^2 + score (relative error of a term up to about 1e-4 |x||c| over the distance, far less in the sum); cat_fit has it from
double sums from pass 3 on, and the two agree to 1e-5 here."""
import numpy as np
import pytest
import torch

from paper_2509_26277_amd import binding, cat_fit, cat_fit_restarts

from parity_util import full_loop

pytestmark = pytest.mark.gpu


def _rows(seed, N, D, C, dt, spread):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    mu = r(C, D) * spread
    y = mu[torch.randint(0, C, (N,), generator=g, device="cuda")] + r(N, D)
    x = y * (0.6 + 0.8 * torch.rand(D, generator=g, device="cuda")) + 0.2 * r(N, D)
    t = torch.bfloat16 if dt == "bf16" else torch.float32
    return x.to(t).contiguous(), y.to(t).contiguous()


def _same(a, b, what=""):
    for key in ("centroids", "assignments", "counts"):
        assert torch.equal(a[key], b[key]), (what, key)
    for key in ("gamma", "beta"):  # statistics are summed with atomics
        torch.testing.assert_close(a[key], b[key], rtol=1e-5, atol=1e-6)
    ja, jb = a["inertia"].cpu().numpy(), b["inertia"].cpu().numpy()
    np.testing.assert_allclose(ja, jb, rtol=1e-5)


def _full(*args, **kw):
    with full_loop():
        return cat_fit(*args, **kw)


SHAPES = [
    (68000, 256, 9, 8, "f32", 1.0),
    (130000, 130, 31, 6, "f32", 0.5),    # not a whole number of 16-byte groups: the loop runs on a padded copy
    (17000, 1000, 48, 9, "f32", 0.3),     # chunked operand, overlapping components: rows keep moving
    (33000, 1024, 64, 7, "bf16", 0.5),
    (264000, 64, 17, 4, "f32", 1.0),     # one pass over listed rows before the last
    (264000, 64, 5, 3, "f32", 1.0),      # too few iterations: the plain loop
    (33000, 256, 150, 7, "f32", 0.4),    # two launches per pass
    (9100, 1001, 200, 6, "f32", 0.3),    # two launches per pass, on a padded copy
    (20000, 840, 256, 5, "bf16", 0.3),
    (66000, 256, 1, 5, "f32", 1.0),      # one cluster
    (264000, 64, 250, 5, "f32", 0.5),    # 16 cluster tiles in one launch
]


@pytest.mark.parametrize("N,D,K,iters,dt,spread", SHAPES)
def test_same_outputs_as_the_loop_that_reads_every_row(N, D, K, iters, dt, spread):
    x, y = _rows(N + D, N, D, max(K // 2, 2), dt, spread)
    a = cat_fit(x, y, K, iters, seed=5)
    _same(a, _full(x, y, K, iters, seed=5))
    _same(a, cat_fit(x, y, K, iters, seed=5, early_stop=True))
    assert int(a["counts"].sum()) == N
    assert torch.equal(a["counts"].long(), torch.bincount(a["assignments"].long(), minlength=K))
    # the last entry of the objective against its definition in double (float32 terms where no row was left out)
    d = sum(float((xc.double() - a["centroids"].double()[ac.long()]).square().sum())
            for xc, ac in zip(x.split(20000), a["assignments"].split(20000)))
    np.testing.assert_allclose(float(a["inertia"][-1]), d, rtol=2e-5)


@pytest.mark.parametrize("D,K,points,init", [
    (256, 24, 40, False), (256, 24, 24, True),
    (255, 24, 40, False),                       # on the padded copy
    (256, 150, 200, False), (256, 150, 150, True),  # two launches per pass
])
def test_objective_of_repeated_rows_far_from_the_origin(D, K, points, init):
    """Rows 300 from the origin in every channel, a hundredth apart: the objective is 1e-9 of the sums it is the difference of.
    Double sums leave it with a few hundred roundings of that size; it is never negative, and zero where every row is a centroid
    (started from the points themselves)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(D + K)
    base = 300.0 + 0.01 * torch.randn(points, D, generator=g, device="cuda")
    x = base[torch.randint(0, points, (70000,), generator=g, device="cuda")].contiguous()
    r = cat_fit(x, 2 * x, K, 8, seed=4, init_centroids=base.contiguous() if init else None)
    total = float(x.double().square().sum())
    d = float((x.double() - r["centroids"].double()[r["assignments"].long()]).square().sum())
    j = r["inertia"].cpu().numpy()
    assert (j >= 0.0).all()
    assert abs(j[-1] - d) <= 512 * 2.0 ** -53 * total
    if init:
        assert d == 0.0


def test_duplicates_empty_clusters_and_exact_ties():
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    base = torch.randint(-3, 4, (8, 64), generator=g, device="cuda").float()
    x = base.repeat_interleave(34000, 0).contiguous()
    y = (x * 1.5 + 0.25).contiguous()
    for K in (3, 20, 140):
        _same(cat_fit(x, y, K, 6, seed=K), _full(x, y, K, 6, seed=K), K)


@pytest.mark.parametrize("N,D,K,dt", [(68000, 256, 9, "f32"), (33000, 1024, 64, "bf16"), (33000, 256, 150, "f32")])
def test_results_do_not_depend_on_the_list_and_queue_capacities(N, D, K, dt):
    x, y = _rows(11, N, D, max(2, K // 3), dt, 0.3)
    want = cat_fit(x, y, K, 7, seed=2)
    try:
        for q, l in ((-1, 0), (1, 1), (7, 3)):
            binding.debug_rerank_queue(q)
            binding.debug_list_capacity(l)
            _same(cat_fit(x, y, K, 7, seed=2), want, (q, l))
    finally:
        binding.debug_rerank_queue(0)
        binding.debug_list_capacity(0)


def test_restarts():
    x, y = _rows(4, 68000, 256, 6, "f32", 0.5)
    r = cat_fit_restarts(x, y, 9, 8, seed=3, restarts=3)
    best = int(r["best_run"])
    _same(r, _full(x, y, 9, 8, seed=3 + best))
    with full_loop():
        assert int(cat_fit_restarts(x, y, 9, 8, seed=3, restarts=3)["best_run"]) == best


@pytest.mark.parametrize("N,D,K", [(68000, 256, 9), (33000, 256, 150), (130000, 130, 31)])
def test_a_workspace_without_the_scratch_of_the_bounds_is_enough(N, D, K):
    """Single passes never use it; cat_fit then reads every row in every pass.  (12 bytes per row are less than that scratch.)"""
    x, y = _rows(2, N, D, 5, "f32", 1.0)
    full = binding.cat_fit_workspace_bytes(N, D, K)
    ws = torch.empty(full - 12 * N, dtype=torch.uint8, device="cuda")
    want = cat_fit(x, y, K, 6, seed=1)
    _same(cat_fit(x, y, K, 6, seed=1, workspace=ws), want)
    _same(cat_fit(x, y, K, 6, seed=1, workspace=ws, early_stop=True), want)
    a, counts, _ = binding.cat_assign(x, want["centroids"], workspace=ws)
    assert torch.equal(a, want["assignments"]) and torch.equal(counts, want["counts"])
    cent, _ = binding.cat_update(x, a, want["centroids"], workspace=ws)
    assert torch.isfinite(cent).all()
    g, b = binding.cat_stats(x, y, a, K, centroids=want["centroids"], workspace=ws)[:2]
    torch.testing.assert_close(g, want["gamma"], rtol=1e-5, atol=1e-6)
    with pytest.raises(binding.CatError):
        cat_fit(x, y, K, 6, seed=1, workspace=torch.empty((full - 12 * N) // 2, dtype=torch.uint8, device="cuda"))


def test_captures_into_a_hip_graph_and_replays():
    """which rows a pass evaluates is decided on the device: one graph, different inputs"""
    N, D, K, iters = 68000, 256, 9, 6
    x, y = _rows(1, N, D, 4, "f32", 0.5)
    ws = torch.empty(binding.cat_fit_workspace_bytes(N, D, K), dtype=torch.uint8, device="cuda")
    cat_fit(x, y, K, iters, seed=1, workspace=ws)  # kernels loaded before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = cat_fit(x, y, K, iters, seed=1, workspace=ws)
    for seed in (1, 2, 3):
        xs, ys = _rows(seed, N, D, 3 + seed, "f32", 0.5)
        x.copy_(xs)
        y.copy_(ys)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _same({k: v.clone() for k, v in out.items()}, _full(xs, ys, K, iters, seed=1), seed)


def test_non_finite_rows_leave_the_others_alone():
    x, y = _rows(9, 68000, 256, 5, "f32", 2.0)
    x[100] = float("nan")
    x[20000, 7] = float("inf")
    r = cat_fit(x, y, 6, 6, seed=1)
    torch.cuda.synchronize()
    a = r["assignments"]
    assert int(a.min()) >= 0 and int(a.max()) < 6 and int(r["counts"].sum()) == 68000
