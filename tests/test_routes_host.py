"""The host rules that choose between a call's routes (no GPU needed)."""
import ctypes

import pytest

from paper_1707_02423_amd import cfsim as cf


def _set(max_nodes, n_graphs=14, jumps=1.4):
    nodes = n_graphs * max_nodes // 2
    # pointers are never dereferenced: the rules read the counts alone
    return cf.GraphSetC(n_graphs, max_nodes, nodes, int(jumps * nodes), *([0x1000] * 8))


@pytest.mark.parametrize("dtype,resize,max_nodes,jumps,branch", [
    ("f32", 0, 8, 1.4, 0), ("f32", 0, 76, 1.4, 0), ("f32", 0, 128, 1.4, 0), ("f32", 0, 150, 1.4, 1),
    ("f32", 0, 120, 40.0, 1), ("f64", 0, 76, 1.4, 0), ("f64", 0, 128, 1.4, 1),
    ("f32", 1, 76, 1.4, 0), ("f32", 1, 128, 1.4, 1), ("f64", 1, 40, 1.4, 0), ("f64", 1, 128, 1.4, 1),
    ("f32", 0, 512, 1.4, 1), ("f32", 0, 65536, 1e6, 1),
])
def test_a_batch_branches_only_for_pairs_past_lds(dtype, resize, max_nodes, jumps, branch):
    s = _set(max_nodes, jumps=jumps)
    d = {"f64": cf.F64, "f32": cf.F32}[dtype]
    assert cf.lib().cfsim_route_branch(ctypes.byref(s), d, resize) == branch


@pytest.mark.parametrize("mean,most,resize,branch", [
    (145, 150, 0, 0), (120, 150, 0, 1), (145, 150, 1, 1),
    (130, 140, 0, 1),   # the mean pair is in LDS
    (300, 400, 0, 1), (390, 400, 0, 0),
])
def test_a_batch_of_equal_sizes_past_lds_stays_one_chain(mean, most, resize, branch):
    s = cf.GraphSetC(20, most, 20 * mean, 28 * mean, *([0x1000] * 8))
    assert cf.lib().cfsim_route_branch(ctypes.byref(s), cf.F32, resize) == branch


@pytest.mark.parametrize("dtype,n_a,n_b,max_iter,tol,strips", [
    ("f32", 150, 150, 200, 1e-12, 1), ("f64", 150, 150, 200, 1e-12, 1), ("f32", 333, 410, 200, 1e-3, 1),
    ("f32", 150, 150, 200, 1e-3, 1), ("f32", 150, 150, 1000, 1e-12, 1), ("f32", 150, 150, 4096, 0.0, 1),
    # stopped early: the launches of max_iter updates would not be paid for
    ("f32", 150, 150, 2000, 1e-2, 0), ("f64", 150, 150, 2000, 1e-2, 0), ("f32", 333, 410, 4096, 1e-2, 0),
    ("f32", 150, 150, 200, 1.0, 0), ("f32", 150, 150, 1, 1e3, 0),
    # limits of the strips
    ("f32", 1024, 24, 200, 0.0, 1), ("f32", 1025, 24, 200, 0.0, 0), ("f32", 24, 1025, 200, 0.0, 0),
    ("f32", 150, 150, 4097, 0.0, 0),
])
def test_a_pair_takes_strips_where_its_updates_pay_for_the_launches(dtype, n_a, n_b, max_iter, tol, strips):
    opt = cf.options(dtype, max_iter, tol)
    assert cf.lib().cfsim_route_score_strips(n_a, n_b, ctypes.byref(opt)) == strips


@pytest.mark.parametrize("dtype,n_a,n_b,kw,buffers", [
    ("f32", 97, 121, {}, 2), ("f64", 90, 80, {}, 2),                      # in LDS
    ("f32", 150, 150, {}, 4), ("f64", 110, 120, {}, 4), ("f32", 333, 410, {}, 4), ("f32", 1024, 60, {}, 4),
    ("f32", 1025, 60, {}, 2), ("f32", 3000, 3000, {}, 2), ("f32", 333, 410, dict(max_iter=4097), 2),
    ("f32", 333, 410, dict(max_iter=4096, tol=1e-2), 2),                   # one workgroup
    ("f32", 333, 410, dict(fp64_final=True), 4),   # FP32 strips, or two FP64 iterates: the same size but for the lists
    ("f32", 97, 121, dict(fp64_final=True), 4),    # two FP64 iterates
])
def test_the_workspace_of_a_pair_is_that_of_its_route(dtype, n_a, n_b, kw, buffers):
    opt = cf.options(dtype, **kw)
    size = cf.lib().cfsim_score_workspace_size(None, n_a, n_b, ctypes.byref(opt))
    one = n_a * n_b * (8 if dtype == "f64" else 4)
    # strips keep lists of 56 (FP64: 96) bytes per column and tables of 496 (1,152) per four rows beside their iterates
    lists = 200 * (n_a + n_b + 64) * (2 if dtype == "f64" else 1)
    assert buffers * one <= size <= buffers * one + (lists if buffers == 4 else 256)


@pytest.mark.parametrize("dtype,max_nodes,pairs,max_iter,tol,every,strips", [
    ("f32", 256, 160, 200, 1e-12, 8, 1), ("f32", 256, 256, 200, 1e-12, 8, 1), ("f32", 32, 1, 200, 1e-12, 8, 1),
    ("f64", 128, 128, 200, 1e-12, 8, 1), ("f32", 128, 100, 200, 1e-3, 8, 1), ("f32", 256, 4, 1000, 0.0, 8, 1),
    # more pairs than the strips gain from, and sizes below and past them
    ("f32", 256, 257, 200, 1e-12, 8, 0), ("f64", 128, 129, 200, 1e-12, 8, 0), ("f32", 31, 1, 200, 1e-12, 8, 0),
    ("f64", 256, 100, 200, 1e-12, 8, 0), ("f32", 512, 16, 200, 1e-12, 8, 0), ("f32", 513, 1, 200, 1e-12, 8, 0),
    # stopped early, or too few updates
    ("f32", 256, 2, 2000, 1e-2, 8, 0), ("f32", 64, 100, 200, 1e-2, 8, 0), ("f64", 128, 10, 4000, 1e-4, 8, 0),
    ("f32", 40, 1, 2, 0.0, 8, 0), ("f32", 128, 1, 200, 1.0, 8, 0),
    # a segment longer than the call has no launches of its own
    ("f32", 128, 10, 200, 1e-12, 100000, 1),
])
def test_the_reverse_takes_strips_where_they_pay(dtype, max_nodes, pairs, max_iter, tol, every, strips):
    s = _set(max_nodes)
    opt = cf.options(dtype, max_iter, tol)
    L = cf.lib()
    assert L.cfsim_route_backward_strips(ctypes.byref(s), ctypes.c_int64(pairs), ctypes.byref(opt), every, 256) == strips


@pytest.mark.parametrize("dtype,max_nodes,pairs,jumps,strips", [
    ("f64", 40, 26, 1.37, 1), ("f64", 40, 27, 1.37, 0), ("f64", 64, 79, 1.37, 1), ("f64", 64, 80, 1.0, 0),
    ("f64", 32, 9, 1.37, 0), ("f64", 87, 128, 1.37, 1), ("f32", 40, 80, 1.1, 1), ("f32", 40, 81, 1.1, 0),
    ("f32", 40, 256, 1.37, 1), ("f32", 76, 256, 1.0, 1), ("f32", 64, 201, 1.0, 0),
])
def test_the_reverse_of_small_graphs_takes_strips_for_fewer_pairs(dtype, max_nodes, pairs, jumps, strips):
    s = cf.GraphSetC(20, max_nodes, 20 * max_nodes, int(20 * max_nodes * jumps) + 1, *([0x1000] * 8))
    opt = cf.options(dtype, 200, 1e-12)
    L = cf.lib()
    assert L.cfsim_route_backward_strips(ctypes.byref(s), ctypes.c_int64(pairs), ctypes.byref(opt), 8, 256) == strips


@pytest.mark.parametrize("dtype,n,pairs,jumps,strips", [
    ("f32", 64, 276, 1.37, 1), ("f32", 64, 1128, 1.37, 0), ("f32", 191, 300, 1.37, 0), ("f32", 192, 100000, 1.37, 1),
    ("f32", 256, 66, 1.2, 1), ("f32", 256, 276, 1.2, 0), ("f32", 400, 100000, 1.2, 1), ("f32", 400, 120, 1.0, 0),
    ("f32", 2048, 64, 1.37, 1), ("f32", 4992, 2, 1.37, 1), ("f32", 4993, 2, 1.37, 0),
    ("f64", 125, 120, 1.37, 1), ("f64", 125, 276, 1.37, 0), ("f64", 400, 66, 1.37, 1), ("f64", 400, 120, 1.37, 0),
    ("f64", 768, 1000, 1.37, 1), ("f64", 256, 28, 1.0, 0), ("f64", 256, 10, 1.0, 1), ("f64", 2496, 1, 1.37, 1),
    ("f64", 2497, 1, 1.37, 0),
])
def test_large_calls_take_strips_or_tiles_by_size(dtype, n, pairs, jumps, strips):
    s = cf.GraphSetC(20, n, 20 * n, int(20 * n * jumps) + 1, *([0x1000] * 8))
    L = cf.lib()
    for kw in (dict(), dict(resize="bilinear"), dict(mfma=True)):
        if dtype == "f64" and "mfma" in kw:
            continue
        opt = cf.options(dtype, **kw)
        got = L.cfsim_route_large_strips(ctypes.byref(s), ctypes.c_int64(pairs), ctypes.byref(opt))
        assert got == (strips if not kw else 0)
    # the workspace is that of the route: tiles need no strip lists
    size = L.cfsim_large_workspace_size(None, ctypes.byref(s), ctypes.c_int64(pairs), ctypes.byref(cf.options(dtype)))
    assert size >= pairs * 4 * n * n * (8 if dtype == "f64" else 4)
