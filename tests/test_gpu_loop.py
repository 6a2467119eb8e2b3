"""Lloyd loops in one launch (cat_loop.hip): the fits of up to 64 MB whose centroids fit LDS.

Compared with the loop of two launches a pass, which the oracle tests pin, and with the oracle itself.  Both sides rank the rows
exactly and keep their sums in double precision, in another order: centroids agree to a rounding of fp32, and a row may only
differ where its two nearest centroids do to that rounding.  The objective's terms are fp32 (|x|^2 + score, see cat_fit)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_26277_amd import binding, cat_fit

from test_gpu_pca_grid import _stream_with
from parity_util import CENTROID_RTOL, check_assignments_lazy, check_values, dev_matrix, f32_round, host_matrix

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _defaults():
    yield
    binding.debug_loop(0)


def _rows(N, D, comps, dtype, seed, spread=2.0):
    rng = np.random.default_rng(seed)
    mu = rng.standard_normal((comps, D)) * spread
    x = mu[rng.integers(0, comps, N)] + rng.standard_normal((N, D))
    y = 1.1 * x + 0.3 + 0.05 * rng.standard_normal((N, D))
    if dtype == "bf16":
        x, y = (torch.from_numpy(a).bfloat16().float().numpy() for a in (x, y))
    return x.astype(np.float32), y.astype(np.float32)


ALL = 256  # the most workgroups a loop has: waits for all of them, and every shape that fits runs in one launch


def _fit_on(members, lq, fp, K, iters, **kw):
    """cat_fit with the hook set, and how many workgroups shared its last pass (0: two launches a pass)"""
    N, D = lq.shape
    dt = binding.CAT_BF16 if lq.dtype == torch.bfloat16 else binding.CAT_F32
    ws = torch.zeros(binding.cat_fit_workspace_bytes(N, D, K, dt), dtype=torch.uint8, device="cuda")
    binding.debug_loop(members)
    r = cat_fit(lq, fp, K, iters, seed=5, workspace=ws, **kw)
    binding.debug_loop(0)
    return r, binding.debug_loop_members(N, D, K, dt, ws)


def _fits(x, y, K, iters, dtype, members=ALL, **kw):
    lq, fp = dev_matrix(x, dtype), dev_matrix(y, dtype)
    got, shared = _fit_on(members, lq, fp, K, iters, **kw)
    want, none = _fit_on(-1, lq, fp, K, iters, **kw)
    assert shared > 0 and none == 0
    return got, want


def _same(got, want, x, dtype):
    cent = host_matrix(want["centroids"])
    differ = check_assignments_lazy(got["assignments"].cpu().numpy(),
                                    oracle.assign(x, f32_round(cent)) if (got["assignments"] != want["assignments"]).any()
                                    else got["assignments"].cpu().numpy(), x, f32_round(cent), "labels")
    counts = torch.bincount(got["assignments"].long(), minlength=cent.shape[0])
    assert (counts == got["counts"]).all()
    np.testing.assert_allclose(got["inertia"].cpu().numpy(), want["inertia"].cpu().numpy(), rtol=1e-4)
    if differ == 0:
        check_values(host_matrix(got["centroids"]), cent, CENTROID_RTOL, "centroids")
        for name in ("gamma", "beta"):
            check_values(host_matrix(got[name]), host_matrix(want[name]), 1e-5, name)
    if "passes_skipped" in got and differ == 0:
        assert int(got["passes_skipped"].item()) == int(want["passes_skipped"].item())


SHAPES = [
    # N, D, K, iterations, type: fewest rows, one channel group, one cluster
    (256, 4, 1, 3, "f32"), (256, 8, 3, 5, "bf16"),
    # remainders of tiles and of clusters, both sides of each cluster tile count
    (1000, 28, 15, 8, "f32"), (2049, 36, 16, 8, "f32"), (2047, 36, 17, 8, "f32"), (3001, 64, 32, 6, "bf16"),
    (3001, 64, 33, 6, "f32"), (4099, 60, 65, 6, "f32"), (5000, 128, 128, 5, "f32"), (5000, 120, 127, 5, "bf16"),
    # long rows: two, four and eight waves share the channels of a tile, the panel takes part of the channels
    (300, 1000, 16, 6, "f32"), (2500, 1024, 16, 5, "f32"), (5000, 512, 30, 5, "f32"), (9001, 520, 9, 5, "bf16"), (600, 1000, 3, 9, "bf16"),
    # more tiles than waves on the chip, rows that are not whole 16-byte groups
    (70000, 32, 7, 6, "f32"), (40000, 45, 2, 6, "f32"),
    # one iteration; a loop that settles
    (900, 40, 6, 1, "f32"), (4096, 64, 4, 40, "f32"),
]


@pytest.mark.parametrize("N,D,K,iters,dtype", SHAPES)
def test_same_outputs_as_two_launches_a_pass(N, D, K, iters, dtype):
    x, y = _rows(N, D, max(2, K - 1), dtype, N + D)
    got, want = _fits(x, y, K, iters, dtype)
    _same(got, want, x, dtype)


@pytest.mark.parametrize("members", [ALL, 3])
@pytest.mark.parametrize("N,D,K,iters,dtype", [(70001, 240, 5, 9, "f32"), (66003, 512, 17, 6, "bf16"), (131101, 128, 128, 5, "f32"),
                                               (17001, 1000, 16, 12, "f32"), (280001, 60, 1, 4, "f32"), (400031, 45, 33, 8, "f32")])
def test_passes_that_leave_rows_out(N, D, K, iters, dtype, members):
    """from 64 MB on: the bounds of two launches a pass, which test_gpu_fit_default_bounds compares with the full loop"""
    _bounded(N, D, K, iters, dtype, members)


@pytest.mark.parametrize("N,D,K,iters,dtype", [
    # bf16, each number of cluster tiles, whole 16-byte groups and not
    (150001, 256, 5, 7, "bf16"), (300001, 128, 17, 6, "bf16"), (400003, 90, 33, 6, "bf16"), (420001, 80, 100, 6, "bf16"),
    # fp32, two tiles of clusters; long rows, whose channels four or eight waves share
    (200003, 100, 20, 6, "f32"), (33001, 600, 8, 20, "f32"), (17001, 1000, 5, 20, "f32"),
    # the panel takes part of the channels at a time, two and eight parts
    (90001, 192, 50, 8, "f32"), (150001, 128, 119, 12, "f32")])
def test_shapes_that_are_dispatched_there(N, D, K, iters, dtype):
    _bounded(N, D, K, iters, dtype, 0)


@pytest.mark.parametrize("N,D,K,iters,dtype", [(636254, 144, 91, 5, "bf16"), (477132, 192, 57, 5, "bf16"), (349631, 96, 117, 7, "f32"), (135001, 128, 5, 4, "f32"), (40000, 1000, 5, 10, "f32"), (80000, 1000, 5, 30, "bf16")])
def test_fits_that_two_launches_a_pass_are_faster_for(N, D, K, iters, dtype):
    """channels taken in parts; a single pass in between; long rows with few iterations or of bf16"""
    lq = torch.randn(N, D, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    assert _fit_on(0, lq, lq, K, iters)[1] == 0
    assert _fit_on(ALL, lq, lq, K, iters)[1] > 0


def _bounded(N, D, K, iters, dtype, members):
    g = torch.Generator(device="cuda").manual_seed(N)
    mu = torch.randn(max(2, K - 1), D, generator=g, device="cuda") * 0.7
    lq = mu[torch.randint(0, mu.shape[0], (N,), generator=g, device="cuda")] + torch.randn(N, D, generator=g, device="cuda")
    lq = lq.to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()
    fp = (lq * 1.1).contiguous()
    got, shared = _fit_on(members, lq, fp, K, iters)
    want, none = _fit_on(-1, lq, fp, K, iters)
    assert shared > 0 and none == 0
    # both rank exactly against centroids that agree to a rounding: a handful of rows between two of them may differ
    assert int((got["assignments"] != want["assignments"]).sum()) <= 3
    assert (torch.bincount(got["assignments"].long(), minlength=K) == got["counts"]).all()
    np.testing.assert_allclose(got["inertia"].cpu().numpy(), want["inertia"].cpu().numpy(), rtol=1e-9)
    check_values(host_matrix(got["centroids"]), host_matrix(want["centroids"]), 1e-4, "centroids")


@pytest.mark.parametrize("members", [1, 2, 5, ALL])
def test_any_number_of_workgroups(members):
    """the rows are shared out over the workgroups that are there when the first one closes the door, and anew (the hook: over up to four times
    as many) when others have come"""
    x, y = _rows(9000, 96, 12, "f32", 3, spread=0.5)
    got, want = _fits(x, y, 20, 12, "f32", members=members, early_stop=True)
    _same(got, want, x, "f32")


@pytest.mark.parametrize("N,D,K,iters,dtype", [(9000, 96, 20, 12, "f32"), (5003, 520, 30, 9, "f32"), (30001, 40, 128, 9, "bf16"), (12000, 64, 5, 10, "bf16"),
                                               (50001, 1000, 5, 20, "f32"), (300001, 128, 17, 12, "bf16"), (420001, 80, 100, 12, "bf16")])
def test_workgroups_that_come_later_join(N, D, K, iters, dtype):
    """a loop that begins with one workgroup (others hold the chip) is shared by all before its last pass"""
    g = torch.Generator(device="cuda").manual_seed(N)
    mu = torch.randn(max(2, K - 1), D, generator=g, device="cuda") * 0.3
    lq = mu[torch.randint(0, mu.shape[0], (N,), generator=g, device="cuda")] + torch.randn(N, D, generator=g, device="cuda")
    lq = lq.to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()
    fp = (lq * 1.1).contiguous()
    (got, shared), (want, every) = _fit_on(1, lq, fp, K, iters), _fit_on(ALL, lq, fp, K, iters)
    assert shared == every
    # both rank exactly against centroids that agree to a rounding: a handful of rows between two of them may differ
    assert int((got["assignments"] != want["assignments"]).sum()) <= 3
    assert (torch.bincount(got["assignments"].long(), minlength=K) == got["counts"]).all()
    np.testing.assert_allclose(got["inertia"].cpu().numpy(), want["inertia"].cpu().numpy(), rtol=1e-9)
    check_values(host_matrix(got["centroids"]), host_matrix(want["centroids"]), 1e-4, "centroids")


@pytest.mark.parametrize("N,D,K,dtype", [(30037, 480, 16, "f32"), (400031, 64, 33, "f32")])
def test_a_fit_begun_beside_another_kernel_gets_the_whole_chip(N, D, K, dtype):
    """the second of two fits begins with what the first one leaves of the chip, and is shared by all workgroups once that has ended"""
    g = torch.Generator(device="cuda").manual_seed(N)
    mu = torch.randn(K, D, generator=g, device="cuda") * 0.1
    lq = mu[torch.randint(0, K, (N,), generator=g, device="cuda")] + torch.randn(N, D, generator=g, device="cuda")
    fp = (lq * 1.1).contiguous()
    want, every = _fit_on(ALL, lq, fp, K, 60)
    assert every > 200
    at = binding.cat_fit_workspace_bytes(N, D, K, binding.CAT_F32)
    ws = [torch.zeros(at, dtype=torch.uint8, device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    binding.debug_loop(ALL)
    for _ in range(3):  # (the first calls on a stream take long)
        ws[1].zero_()
        go = torch.cuda.Event()
        torch.cuda._sleep(3000000)  # both are queued when they start
        go.record()
        got = []
        for s, w, iters in zip(streams, ws, (15, 60)):
            s.wait_event(go)
            with torch.cuda.stream(s):
                got.append(cat_fit(lq, fp, K, iters, seed=5, workspace=w))
        torch.cuda.synchronize()
        assert binding.debug_loop_members(N, D, K, binding.CAT_F32, ws[1]) == every
    assert int((got[1]["assignments"] != want["assignments"]).sum()) <= N // 1000
    np.testing.assert_allclose(got[1]["inertia"].cpu().numpy(), want["inertia"].cpu().numpy(), rtol=1e-4)


@pytest.mark.parametrize("cus", [64, 128])
def test_a_stream_with_some_of_the_cus(cus):
    """the workgroups that have no place there never come while the loop runs; those that are there do all of it (LDS: one a CU)"""
    g = torch.Generator(device="cuda").manual_seed(cus)
    mu = torch.randn(100, 128, generator=g, device="cuda") * 0.5
    lq = mu[torch.randint(0, 100, (40000,), generator=g, device="cuda")] + torch.randn(40000, 128, generator=g, device="cuda")
    fp = (lq * 1.1).contiguous()
    want, every = _fit_on(ALL, lq, fp, 100, 6)
    with _stream_with(cus) as s, torch.cuda.stream(s):
        got, shared = _fit_on(ALL, lq, fp, 100, 6)
    assert every == 256 and 0 < shared <= cus
    assert int((got["assignments"] != want["assignments"]).sum()) <= 3
    check_values(host_matrix(got["centroids"]), host_matrix(want["centroids"]), 1e-4, "centroids")


def test_ties_and_empty_clusters():
    """integer rows on few points: exact ties between centroids, clusters without rows (they keep their centroid)"""
    rng = np.random.default_rng(1)
    pts = rng.integers(-3, 4, (6, 32)).astype(np.float32)
    x = pts[rng.integers(0, 6, 3000)]
    y = (x * 2 + 1).astype(np.float32)
    o = oracle.fit(x, y, 9, iters=6, seed=5)
    got, _ = _fits(x, y, 9, 6, "f32")
    assert (got["assignments"].cpu().numpy() == o["assignments"]).all()
    assert (got["counts"].cpu().numpy() == 0).any()
    check_values(host_matrix(got["centroids"]), o["centroids"], CENTROID_RTOL, "centroids")


def test_given_centroids_far_from_the_rows():
    """all rows in one cluster first, the others empty; |x| large beside the spread (most rows measured exactly)"""
    x, y = _rows(3000, 64, 5, "f32", 9)
    x = (x + 100.0).astype(np.float32)
    init = torch.from_numpy(np.concatenate([x[:1], x[:4] + 1000.0]).astype(np.float32)).cuda()
    got, want = _fits(x, y, 5, 7, "f32", init_centroids=init)
    _same(got, want, x, "f32")


@pytest.mark.parametrize("members", [ALL, 1])
def test_rows_of_very_different_magnitude(members):
    """a few rows 1e17 times as long as the others leave those rows' clusters after pass 0: nothing of them may stay in the sums
    (pass 1 makes them afresh then, as two launches a pass always do)"""
    rng = np.random.default_rng(2)
    u = rng.standard_normal(64)
    x = rng.standard_normal((3000, 64)) + 2.0
    for i, far in ((100, 1.0e17), (200, -1.0e17)):  # (the two groups all but cancel: the short rows keep their cluster)
        x[i:i + 20] = far * u
        x[i + 20:i + 80] = 1.8 * far * u
        x[i + 80:i + 84] = 3.0 * far * u
    x = x.astype(np.float32)
    y = (0.5 * x + 1.0).astype(np.float32)
    init = np.stack([np.zeros(64), 3.0e17 * u, -3.0e17 * u]).astype(np.float32)
    # what the case is about, by the oracle: the long rows lie with the short ones in pass 0 and leave them in pass 1
    first = oracle.assign(x, init)
    second = oracle.assign(x, oracle.fit(x, y, 3, 1, init_centroids=init)["centroids"])
    assert (first[100:120] == 0).all() and (second[100:120] == 1).all() and (second == 0).sum() == 2832
    want = oracle.fit(x, y, 3, 6, init_centroids=init)
    got, two = _fits(x, y, 3, 6, "f32", members=members, init_centroids=torch.from_numpy(init).cuda())
    for r in (two, got):
        assert (r["assignments"].cpu().numpy() == want["assignments"]).all()
        for k in range(3):
            check_values(host_matrix(r["centroids"])[k], want["centroids"][k], CENTROID_RTOL, f"centroid {k}")


def test_calls_side_by_side_on_streams():
    """loops of several streams share the chip: each with the members that were there in time"""
    cases = [(_rows(n, d, 8, "f32", n), k) for n, d, k in ((20000, 64, 9), (33000, 80, 37), (5000, 600, 8), (12000, 100, 64))]
    want = []
    for (x, y), k in cases:
        binding.debug_loop(-1)
        want.append(cat_fit(dev_matrix(x, "f32"), dev_matrix(y, "f32"), k, 10, seed=5))
    binding.debug_loop(ALL)
    ins = [(dev_matrix(x, "f32"), dev_matrix(y, "f32"), k) for (x, y), k in cases]
    streams = [torch.cuda.Stream() for _ in cases]
    torch.cuda.synchronize()
    for _ in range(5):
        got = []
        for s, (lq, fp, k) in zip(streams, ins):
            with torch.cuda.stream(s):
                got.append(cat_fit(lq, fp, k, 10, seed=5))
        torch.cuda.synchronize()
        for g, w, ((x, _), _) in zip(got, want, cases):
            _same(g, w, x, "f32")


def test_replayed_from_a_graph():
    x, y = _rows(8000, 72, 10, "f32", 4, spread=0.7)
    lq, fp = dev_matrix(x, "f32"), dev_matrix(y, "f32")
    ws = torch.empty(binding.cat_fit_workspace_bytes(8000, 72, 12, binding.CAT_F32), dtype=torch.uint8, device="cuda")
    binding.debug_loop(ALL)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cat_fit(lq, fp, 12, 8, seed=5, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = cat_fit(lq, fp, 12, 8, seed=5, workspace=ws)
    for scale in (1.0, 0.5, 2.0):
        lq.copy_(dev_matrix((x * scale).astype(np.float32), "f32"))
        graph.replay()
        torch.cuda.synchronize()
        binding.debug_loop(-1)
        want = cat_fit(lq, fp, 12, 8, seed=5)
        _same(got, want, (x * scale).astype(np.float32), "f32")


@pytest.mark.parametrize("N,D,K,iters,dtype,one", [
    # measured on both sides: where the additions of all workgroups, channels taken in parts or bf16 rows outweigh the launches saved
    (28835, 1000, 16, 4, "bf16", False), (60074, 480, 16, 10, "bf16", False), (14417, 1000, 16, 4, "f32", False), (1715, 136, 98, 2, "bf16", False),
    (30037, 480, 16, 10, "f32", True), (6291, 1000, 3, 10, "bf16", True), (4096, 64, 4, 20, "f32", True), (33816, 80, 37, 30, "f32", True), (89422, 296, 1, 5, "bf16", True), (25269, 230, 37, 7, "bf16", True)])
def test_small_fits_take_the_faster_way(N, D, K, iters, dtype, one):
    x, y = _rows(N, D, K, dtype, 1)
    _, shared = _fit_on(0, dev_matrix(x, dtype), dev_matrix(y, dtype), K, iters)
    assert (shared > 0) == one
