"""Tridiagonalisation in one launch whose workgroups pass their products on through memory: sizes on either side of its range and
of its numbers of rows and columns per workgroup and thread, the one workgroup that does the work when a wait is given up,
captured graphs, and calls on several streams at once.  Each says by which of the ways its columns went.

Bounds: an eigenvalue is within a few D eps |C| (the covariance is summed in double); a row of the result satisfies
C v = lambda v to the rounding of its float32 entries (6e-8 |C|) and the rows are at right angles to the same."""
import contextlib
import ctypes
import time

import numpy as np
import pytest
import torch

from paper_2509_26277_amd import binding, cat_pca_fit

pytestmark = pytest.mark.gpu


def _rows(D, seed, N=None):
    rng = np.random.default_rng(seed)
    N = N or max(300, D // 2)  # wide rows: a covariance of less than full rank
    x = rng.standard_normal((N, D)) * np.exp(-3.0 * np.arange(D) / D) + rng.standard_normal((N, 4)) @ rng.standard_normal((4, D))
    return np.ascontiguousarray(x, dtype=np.float32)


def _fit(t, p, **kw):
    """cat_pca_fit with a workspace of its own; the way its columns went, and its outputs"""
    N, D = t.shape
    ws = torch.empty(binding.load_library().cat_pca_workspace_bytes(N, D, p, binding.CAT_F32), dtype=torch.uint8, device="cuda")
    out = cat_pca_fit(t, p, workspace=ws, **kw)
    return binding.debug_pca_route(ws, N, D, p), out


def _check(x, mean, comps, evals):
    D, p = x.shape[1], len(comps)
    xd = x.astype(np.float64) - x.astype(np.float64).mean(0)
    C = xd.T @ xd / len(x)
    w = np.linalg.eigvalsh(C)[::-1]
    v, lam = comps.cpu().numpy().astype(np.float64), evals.cpu().numpy()
    norm = np.abs(w).max()
    slack = 30 * D * np.finfo(np.float64).eps * norm
    assert np.isfinite(v).all()
    assert np.abs(lam - w[:p]).max() <= slack
    assert np.abs(v @ v.T - np.eye(p)).max() <= 1e-6
    assert np.linalg.norm(v @ C - lam[:, None] * v, axis=1).max() <= 3e-7 * norm + slack


@pytest.mark.parametrize("D", [63, 64, 65, 127, 128, 129, 255, 256, 257, 383, 511, 512, 513, 769, 1000, 1023, 1024, 1025])
def test_sizes(D):
    x = _rows(D, D)
    route, out = _fit(torch.from_numpy(x).cuda(), min(D, 20))
    assert route == ("grid" if 64 <= D <= 1024 else "columns")
    _check(x, *out)


@pytest.mark.parametrize("N", [2, 15, 17, 63, 64, 65, 71, 72, 73, 129, 2049, 70001])
@pytest.mark.parametrize("D", [64, 65, 130])
def test_rows_of_the_covariance(N, D):
    """remainders of the rows that a wave takes at once, in turn and in all, and one or several ranges of rows"""
    x = _rows(D, N + D, N)
    _check(x, *cat_pca_fit(torch.from_numpy(x).cuda(), 8))


@pytest.mark.parametrize("D", [64, 200, 300, 1001])
def test_a_wait_given_up(D):
    x = _rows(D, D + 1)
    t = torch.from_numpy(x).cuda()
    route, want = _fit(t, 16)
    assert route == "grid"
    binding.debug_pca_patience(-1)
    try:
        route, got = _fit(t, 16)
    finally:
        binding.debug_pca_patience(binding.CAT_PCA_PATIENCE)
    assert route == "alone"
    _check(x, *got)
    # the covariance is summed with atomics, in another order from call to call
    assert (got[2] - want[2]).abs().max() <= 60 * D * np.finfo(np.float64).eps * want[2].max()


def test_values_that_are_no_numbers_end():
    x = _rows(130, 3)
    x[5, 7] = np.nan
    route, (_, comps, evals) = _fit(torch.from_numpy(x).cuda(), 4)
    assert route == "grid" and comps.shape == (4, 130)  # (values that are none of a number are passed on like others)


def test_a_constant_matrix():
    x = torch.full((100, 96), 2.5, device="cuda")
    _, comps, evals = cat_pca_fit(x, 5)
    assert evals.abs().max().item() == 0.0
    v = comps.double()
    assert (v @ v.T - torch.eye(5, device="cuda", dtype=torch.float64)).abs().max().item() <= 1e-6


def test_captures_into_a_hip_graph_and_replays():
    D, p, N = 320, 12, 2000
    xs = [_rows(D, s, N) for s in (11, 12, 13)]
    buf = torch.from_numpy(xs[0]).cuda()
    ws = torch.empty(binding.load_library().cat_pca_workspace_bytes(N, D, p, binding.CAT_F32), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cat_pca_fit(buf, p, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = cat_pca_fit(buf, p, workspace=ws)
    for x in xs:
        buf.copy_(torch.from_numpy(x))
        graph.replay()
        torch.cuda.synchronize()
        assert binding.debug_pca_route(ws, N, D, p) == "grid"
        _check(x, *out)


def test_calls_on_several_streams_at_once():
    D, p = 1000, 8
    xs = [_rows(D, 20 + s, 600) for s in range(4)]
    ts = [torch.from_numpy(x).cuda() for x in xs]
    ws = [torch.empty(binding.load_library().cat_pca_workspace_bytes(600, D, p, binding.CAT_F32), dtype=torch.uint8, device="cuda")
          for _ in xs]
    streams = [torch.cuda.Stream() for _ in xs]
    torch.cuda.synchronize()
    outs = [None] * 4
    for _ in range(3):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[i] = cat_pca_fit(ts[i], p, workspace=ws[i])
    torch.cuda.synchronize()
    for x, o, w in zip(xs, outs, ws):
        assert binding.debug_pca_route(w, 600, D, p) == "grid"  # four times 128 workgroups were resident together, or in turn
        _check(x, *o)


def _hip():
    """the HIP runtime that torch and the library have loaded"""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return ctypes.CDLL(path)


@contextlib.contextmanager
def _stream_with(cus):
    """a stream with the first ``cus`` CUs (a multiple of 32: as many of every shader engine of every XCD)"""
    hip, words = _hip(), torch.cuda.get_device_properties(0).multi_processor_count // 32
    mask = (ctypes.c_uint32 * words)(*[0xFFFFFFFF if 32 * (i + 1) <= cus else 0 for i in range(words)])
    handle = ctypes.c_void_p()
    torch.cuda.synchronize()
    if hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), words, mask) != 0:
        pytest.skip("no streams with a CU mask here")
    try:
        yield torch.cuda.ExternalStream(handle.value)
        torch.cuda.synchronize()
    finally:
        assert hip.hipStreamDestroy(handle) == 0


@pytest.mark.parametrize("cus", [64, 128, 224])
def test_a_stream_with_some_of_the_cus_takes_a_launch_per_column(cus):
    x = _rows(200, 31)
    t = torch.from_numpy(x).cuda()
    with _stream_with(cus) as s, torch.cuda.stream(s):
        route, out = _fit(t, 8)
    assert route == "columns"
    _check(x, *out)
    assert _fit(t, 8)[0] == "grid"  # and the default stream as before


def test_workgroups_that_cannot_all_be_resident_give_up_soon():
    """a graph captured with the whole device and replayed where half of the workgroups have no place: they wait some 20 ms, one
    workgroup does the columns (some 6 ms at this size)"""
    N, D, p = 600, 300, 8
    x = _rows(D, 33, N)
    t = torch.from_numpy(x).cuda()
    ws = torch.empty(binding.load_library().cat_pca_workspace_bytes(N, D, p, binding.CAT_F32), dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = cat_pca_fit(t, p, workspace=ws)
    graph.replay()
    torch.cuda.synchronize()
    assert binding.debug_pca_route(ws, N, D, p) == "grid"
    with _stream_with(32) as s:
        with torch.cuda.stream(s):
            start = time.perf_counter()
            graph.replay()
            torch.cuda.synchronize()
            took = time.perf_counter() - start
    assert binding.debug_pca_route(ws, N, D, p) == "alone"
    assert 0.015 <= took < 0.3
    _check(x, *out)


def test_the_default_streams_take_the_grid():
    x = _rows(100, 32)
    t = torch.from_numpy(x).cuda()
    mean, comps, evals = torch.empty(100, device="cuda"), torch.empty((5, 100), device="cuda"), torch.empty(5, dtype=torch.float64, device="cuda")
    lib = binding.load_library()
    for handle in (0, 1, 2):  # the null stream, hipStreamLegacy, hipStreamPerThread
        ws = torch.zeros(lib.cat_pca_workspace_bytes(len(x), 100, 5, 0), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        assert lib.cat_pca_fit(t.data_ptr(), len(x), 100, 5, 0, 0, mean.data_ptr(), comps.data_ptr(), evals.data_ptr(),
                               ws.data_ptr(), ws.numel(), handle) == 0
        torch.cuda.synchronize()
        assert binding.debug_pca_route(ws, len(x), 100, 5) == "grid"
        _check(x, mean, comps, evals)
