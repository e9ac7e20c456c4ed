"""Routes of the strips at their limits, each with the route it took stated or counted: the largest graphs, columns
past a workgroup's first pass, workspaces without room for strips, and a reverse call with a pair for nearly every CU.

Tolerances are those of the suite for the same quantities: S within 1e-5 (FP32) and 1e-10 (FP64) of the oracle's,
gradients on strips within 1e-4 and 1e-10 of the largest one in the one-workgroup kernel.
"""
import ctypes
import re

import numpy as np
import pytest

from cfgsynth import CFG, Grammar, make_cfg
from tests.parity import check_matching, oracle_pair, rel_err
from tests.test_gpu_routes import ONE_WORKGROUP, launches
from tests.test_gpu_strips import _wide

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cfm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1707_02423_amd import cfsim
    return cfsim


@pytest.fixture(scope="module")
def ctx(cfm):
    return cfm.Context(0)


def _graph(n, kind, seed):
    return _wide(n, seed) if kind == "wide" else make_cfg(n, Grammar(counts="trip"), seed=seed)


def _tol(dtype):
    return 1e-10 if dtype == "f64" else 1e-5


def _score(cfm, ctx, gs, dtype, max_iter, two_buffers=False):
    """One pair through the C ABI: (result, S, match, launches)."""
    L = cfm.lib()
    opt = cfm.options(dtype, max_iter, 0.0)
    A, B = gs.graph(0), gs.graph(1)
    dt = torch.float64 if dtype == "f64" else torch.float32
    size = L.cfsim_score_workspace_size(ctx.handle, A.n, B.n, ctypes.byref(opt))
    if two_buffers:
        size = (2 * A.n * B.n * dt.itemsize + 255) // 256 * 256
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    S = torch.empty(A.n * B.n, dtype=dt, device="cuda")
    match = torch.empty(B.n, dtype=torch.int32, device="cuda")
    res = torch.empty(cfm.RESULT_BYTES, dtype=torch.uint8, device="cuda")

    def call(stream):
        return L.cfsim_score(ctx.handle, ctypes.byref(A), ctypes.byref(B), ctypes.byref(opt), S.data_ptr(),
                             match.data_ptr(), res.data_ptr(), ws.data_ptr(), size, stream)
    n = launches(cfm, call)
    torch.cuda.synchronize()
    assert call(None) == 0
    torch.cuda.synchronize()
    return (res.cpu().numpy().view(cfm.RESULT_DTYPE)[0], S.cpu().numpy().reshape(B.n, A.n), match.cpu().numpy(), n)


@pytest.mark.parametrize("dtype,nA,nB,kind,strips", [
    # 640 and 520 columns: a second pass of the eight waves over the columns
    ("f32", 64, 640, "cfg", True), ("f32", 64, 640, "wide", True), ("f64", 64, 520, "cfg", True),
    # the largest graph of a pair on strips, and one node more
    ("f32", 1024, 24, "cfg", True), ("f32", 1025, 24, "cfg", False), ("f64", 24, 1024, "cfg", True),
    ("f64", 24, 1025, "cfg", False),
])
def test_single_pairs_at_the_limits_of_the_strips(cfm, ctx, dtype, nA, nB, kind, strips):
    graphs = [_graph(nA, kind, 11), _graph(nB, kind, 12)]
    res, S, match, n = _score(cfm, ctx, cfm.pack(ctx, graphs), dtype, 12)
    assert n > 12 if strips else n == 1
    ref = oracle_pair(graphs, 0, 1, max_iter=12, tol=0.0)
    assert rel_err(S, ref.S) <= _tol(dtype)
    assert res["iters"] == 12 and (res["status"] & 15) == ref.status
    check_matching(S, match, ref.S, dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nA,nB,kind", [(160, 192, "cfg"), (190, 257, "wide"), (64, 520, "cfg")])
def test_a_workspace_of_two_buffers_runs_one_workgroup(cfm, ctx, nA, nB, kind, dtype):
    graphs = [_graph(nA, kind, 5), _graph(nB, kind, 6)]
    res, S, match, n = _score(cfm, ctx, cfm.pack(ctx, graphs), dtype, 13, two_buffers=True)
    assert n == 1
    ref = oracle_pair(graphs, 0, 1, max_iter=13, tol=0.0)
    assert rel_err(S, ref.S) <= _tol(dtype)
    assert res["iters"] == 13 and (res["status"] & 15) == ref.status
    check_matching(S, match, ref.S, dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind,max_iter", [("cfg", 20), ("wide", 13), ("wide", 1)])
def test_large_pairs_without_room_for_strips_run_on_the_tiles(cfm, ctx, kind, max_iter, dtype):
    graphs = [_graph(n, kind, n) for n in (65, 64, 257, 130, 131, 511)]
    gs = cfm.pack(ctx, graphs)
    a, b = np.array([0, 2, 4], np.int32), np.array([1, 3, 5], np.int32)
    B = cfm.Batch(ctx, gs, a, b, dtype=dtype, max_iter=max_iter, tol=0.0, want_S=True, path="large")
    full, B.ws_bytes = B.ws_bytes, 1
    with pytest.raises(cfm.CfsimError) as e:
        B.run()
    B.ws_bytes = int(re.search(r"(\d+) needed", str(e.value)).group(1))
    assert B.ws_bytes < full
    B.run()
    torch.cuda.synchronize()
    res = B.results()
    for q, (S, match) in enumerate(zip(B.S_list(), B.matches())):
        ref = oracle_pair(graphs, a[q], b[q], max_iter=max_iter, tol=0.0)
        assert rel_err(S, ref.S) <= _tol(dtype)
        assert res["iters"][q] == ref.iters and (res["status"][q] & 15) == ref.status
        check_matching(S, match, ref.S, dtype)


@pytest.mark.parametrize("jumps", [0, 1, 300])
def test_batch_pairs_past_lds_around_three_jumps_per_node(cfm, ctx, jumps):
    # up to three per node on strips, above on gathers
    rng = np.random.default_rng(jumps)
    graphs = []
    for n, extra in ((160, 0), (175, jumps)):
        m = 3 * n + extra
        graphs.append(CFG(n, rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32),
                          rng.integers(1, 100, m).astype(np.float64)))
    gs = cfm.pack(ctx, graphs)
    res, match, S = cfm.score_batch(ctx, gs, [0, 1], [1, 0], dtype="f32", max_iter=20, tol=0.0, want_S=True)
    for q, (a, b) in enumerate([(0, 1), (1, 0)]):
        ref = oracle_pair(graphs, a, b, max_iter=20, tol=0.0)
        assert rel_err(S[q], ref.S) <= _tol("f32")
        assert res["iters"][q] == ref.iters and (res["status"][q] & 15) == ref.status
        check_matching(S[q], match[q], ref.S, "f32")


@pytest.mark.parametrize("dtype,pairs,step", [("f32", 253, 1), ("f64", 127, 2)])
def test_a_reverse_call_of_many_unequal_pairs_on_strips(cfm, ctx, dtype, pairs, step):
    # an odd number of pairs over the XCDs, 8 to 48 (88) nodes
    graphs = [make_cfg(8 + step * (i % 41), Grammar(counts="trip"), seed=i) for i in range(46)]
    gs = cfm.pack(ctx, graphs)
    a, b = (x.astype(np.int32)[:pairs] for x in np.triu_indices(46))
    weight = torch.linspace(0.5, 1.5, pairs, dtype=torch.float64, device="cuda")
    out = []
    for every in (0, 4):
        B = cfm.Batch(ctx, gs, a, b, dtype=dtype, max_iter=60, tol=0.0, checkpoint_every=every)
        B.run()
        grad = torch.zeros(gs.total_edges, dtype=torch.float64, device="cuda")
        status = cfm.backward(B, weight, grad, checkpoint_every=4)
        out.append((grad.cpu().numpy(), status.cpu().numpy()))
    L = cfm.lib()
    size = L.cfsim_backward_workspace_size(ctx.handle, ctypes.byref(B.set_c), pairs, ctypes.byref(B.opt), 4)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    n = launches(cfm, lambda s: L.cfsim_score_backward(
        ctx.handle, ctypes.byref(B.set_c), B.pair_a.data_ptr(), B.pair_b.data_ptr(), pairs, ctypes.byref(B.opt),
        B.res.data_ptr(), B.match.data_ptr(), B.match_off.data_ptr(), weight.data_ptr(), grad.data_ptr(), None, 4,
        B.ckpt.data_ptr(), B.ckpt_off.data_ptr(), ws.data_ptr(), size, s))
    assert n == 3 + 16 * 4 + 16 + ONE_WORKGROUP   # strips
    (g0, s0), (g1, s1) = out
    assert (s0 == 0).all() and (s1 == 0).all()
    assert np.abs(g0).max() > 0.0
    assert np.abs(g0 - g1).max() <= _tol(dtype) * (10 if dtype == "f32" else 1) * np.abs(g0).max()
