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
