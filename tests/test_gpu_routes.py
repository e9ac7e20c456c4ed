"""The launches a call enqueues: which route it took, and that they do not follow max_iter where a tolerance
stops the pairs early.  A call is captured into a graph, whose kernel nodes are counted; nothing of it runs."""
import ctypes

import numpy as np
import pytest

from cfgsynth import Grammar, make_cfg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cfm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_02423_amd import cfsim
    return cfsim


def launches(cfm, call):
    """Kernels that call(stream) enqueues."""
    L = cfm.lib()
    stream = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert L.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 2) == 0
    rc = call(stream.cuda_stream)
    assert L.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert rc == 0, L.cfsim_last_error()
    assert L.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert L.hipGraphDestroy(graph) == 0
    return n.value


@pytest.fixture(scope="module")
def ctx(cfm):
    return cfm.Context(0)


def _score_launches(cfm, ctx, n_a, n_b, dtype, max_iter, tol, ws_bytes=None):
    gs = cfm.pack(ctx, [make_cfg(n, Grammar(counts="trip"), seed=n) for n in (n_a, n_b)])
    opt = cfm.options(dtype, max_iter, tol)
    A, B = gs.graph(0), gs.graph(1)
    L = cfm.lib()
    size = ws_bytes or L.cfsim_score_workspace_size(ctx.handle, n_a, n_b, ctypes.byref(opt))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    match = torch.empty(n_b, dtype=torch.int32, device="cuda")
    res = torch.empty(cfm.RESULT_BYTES, dtype=torch.uint8, device="cuda")
    return launches(cfm, lambda s: L.cfsim_score(ctx.handle, ctypes.byref(A), ctypes.byref(B), ctypes.byref(opt), None,
                                                 match.data_ptr(), res.data_ptr(), ws.data_ptr(), size, s))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_a_single_pairs_launches(cfm, ctx, dtype):
    assert _score_launches(cfm, ctx, 150, 160, dtype, 200, 1e-12) > 200   # strips
    assert _score_launches(cfm, ctx, 150, 160, dtype, 2000, 1e-2) == 1    # one workgroup
    e = 8 if dtype == "f64" else 4
    assert _score_launches(cfm, ctx, 150, 160, dtype, 200, 1e-12, ws_bytes=2 * 150 * 160 * e + 256) == 1


@pytest.mark.parametrize("kw", [dict(dtype="f64"), dict(dtype="f32"), dict(dtype="f64", path="damped", alpha=0.85),
                                dict(dtype="f32", path="damped", alpha=0.85)])
def test_few_pairs_past_lds_score_as_among_many(cfm, ctx, kw):
    # up to one pair per CU each has a CU's LDS to itself; the kernel and its
    # results are the same
    graphs = [make_cfg(n, Grammar(counts="trip"), seed=n) for n in (150, 163, 201, 149)]
    gs = cfm.pack(ctx, graphs)
    a, b = np.triu_indices(4)
    a, b = a.astype(np.int32), b.astype(np.int32)
    out = []
    for times in (1, 30):   # 10 and 300 pairs
        B = cfm.Batch(ctx, gs, np.tile(a, times), np.tile(b, times), max_iter=12, tol=0.0, want_S=True, **kw)
        assert (B.buckets() == 5).all()
        B.run()
        torch.cuda.synchronize()
        out.append((B.results()[:10].tobytes(), [m.tobytes() for m in B.matches()[:10]],
                    [x.tobytes() for x in B.S_list()[:10]]))
    assert out[0] == out[1]


def _backward_launches(cfm, ctx, sizes, pairs, dtype, max_iter, tol, every):
    gs = cfm.pack(ctx, [make_cfg(n, Grammar(counts="trip"), seed=q) for q, n in enumerate(sizes)])
    a = np.arange(pairs, dtype=np.int32) % len(sizes)
    B = cfm.Batch(ctx, gs, a, a[::-1].copy(), dtype=dtype, max_iter=max_iter, tol=tol, checkpoint_every=every)
    B.run()
    L = cfm.lib()
    size = L.cfsim_backward_workspace_size(ctx.handle, ctypes.byref(B.set_c), pairs, ctypes.byref(B.opt), every)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    one = torch.ones(pairs, dtype=torch.float64, device="cuda")
    grad = torch.zeros(gs.total_edges, dtype=torch.float64, device="cuda")
    return launches(cfm, lambda s: L.cfsim_score_backward(
        ctx.handle, ctypes.byref(B.set_c), B.pair_a.data_ptr(), B.pair_b.data_ptr(), pairs, ctypes.byref(B.opt),
        B.res.data_ptr(), B.match.data_ptr(), B.match_off.data_ptr(), one.data_ptr(), grad.data_ptr(), None, every,
        B.ckpt.data_ptr(), B.ckpt_off.data_ptr(), ws.data_ptr(), size, s))


ONE_WORKGROUP = 2   # the queue's counter and the kernel


def test_the_reverses_launches(cfm, ctx):
    def n(*a):
        return _backward_launches(cfm, ctx, *a)
    # strips: (rounds + 1) of a segment's launches, a seam before the first and between rounds
    assert n([128, 100, 60], 3, "f32", 40, 0.0, 8) == 3 + 6 * 8 + 6 + ONE_WORKGROUP
    assert n([128, 100, 60], 3, "f64", 40, 0.0, 8) == 3 + 6 * 8 + 6 + ONE_WORKGROUP
    assert n([128, 100, 60], 3, "f32", 40, 0.0, 1000) == 3 + 2 * 40 + 2 + ONE_WORKGROUP  # a segment as long as the call
    # one workgroup per pair: stopped early, too many in FP64, pairs that are no strips' pairs
    assert n([128, 100, 60], 3, "f32", 2000, 0.5, 8) == ONE_WORKGROUP
    assert n([64, 50, 60], 130, "f64", 16, 0.0, 4) == ONE_WORKGROUP
    assert n([400, 420], 2, "f32", 16, 0.0, 4) == ONE_WORKGROUP


@pytest.mark.parametrize("dtype,pairs", [("f32", 600), ("f64", 300)])
def test_many_small_pairs_on_the_large_path(cfm, ctx, dtype, pairs):
    # past the strips' line: the tiles give what strips give for the first few of them, up to rounding (20 updates of
    # at most one rounding each, and of the norms)
    graphs = [make_cfg(n, Grammar(counts="trip"), seed=n) for n in (60, 63, 64, 57)]
    gs = cfm.pack(ctx, graphs)
    a, b = (np.tile(x.astype(np.int32), pairs // 6) for x in np.triu_indices(4, 1))
    L = cfm.lib()
    out = []
    for m in (6, pairs):
        B = cfm.Batch(ctx, gs, a[:m], b[:m], dtype=dtype, max_iter=20, tol=0.0, want_S=True, path="large")
        assert L.cfsim_route_large_strips(ctypes.byref(B.set_c), ctypes.c_int64(m), ctypes.byref(B.opt)) == (m == 6)
        B.run()
        torch.cuda.synchronize()
        out.append((B.S_list()[:6], B.results()[:6].copy(), B.S_list()[-6:]))
    for q in range(6):
        S = out[0][0][q]
        assert np.abs(S - out[1][0][q]).max() <= (2e-6 if dtype == "f32" else 1e-13) * np.abs(S).max()
        assert out[0][1]["iters"][q] == out[1][1]["iters"][q] == 20
        np.testing.assert_array_equal(out[1][0][q], out[1][2][q])
