"""Reverse mode on strips (a forward that left checkpoints) against the
one-workgroup kernel (no checkpoints: it recomputes the forward).

The two start a segment from the forward's iterate and from the recomputed
one, which differ by the rounding of the scale: 1e-10 of the largest gradient
in FP64, 1e-4 in FP32, the bounds of that comparison elsewhere in the suite.
"""
import numpy as np
import pytest

from cfgsynth import CFG, Grammar, make_cfg
from tests.test_gpu_strips import _wide

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02423_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(cf):
    return cf.Context(0)


def _grads(cf, ctx, graphs, pa, pb, dtype, max_iter, every, tol=0.0):
    gs = cf.pack(ctx, graphs)
    out = []
    gsc = torch.linspace(0.5, 1.5, len(pa), dtype=torch.float64)
    gsc[len(pa) // 2] = 0.0
    for ck in (0, every):
        b = cf.Batch(ctx, gs, np.asarray(pa, np.int32), np.asarray(pb, np.int32), dtype=dtype, max_iter=max_iter,
                     tol=tol, want_match=True, checkpoint_every=ck) if ck else \
            cf.Batch(ctx, gs, np.asarray(pa, np.int32), np.asarray(pb, np.int32), dtype=dtype, max_iter=max_iter,
                     tol=tol, want_match=True)
        b.run()
        g = torch.zeros(gs.total_edges, dtype=torch.float64, device="cuda")
        st = cf.backward(b, gsc, g, checkpoint_every=every)
        torch.cuda.synchronize()
        out.append((g.cpu().numpy(), st.cpu().numpy(), b.results().copy()))
    return out


def _check(out, dtype):
    (g0, s0, r0), (g1, s1, r1) = out
    assert r0.tobytes() == r1.tobytes()
    np.testing.assert_array_equal(s0, s1)
    assert np.abs(g0).max() > 0.0
    assert np.abs(g0 - g1).max() <= (1e-10 if dtype == "f64" else 1e-4) * np.abs(g0).max()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("max_iter,every", [(1, 8), (2, 1), (8, 8), (9, 8), (17, 8), (24, 5), (6, 16), (40, 3)])
def test_segments_of_the_reverse(cf, ctx, max_iter, every, dtype):
    g = Grammar(counts="trip")
    sizes = [3, 5, 64, 65, 130, 63, 97, 121]
    graphs = [make_cfg(n, g, seed=n) for n in sizes]
    _check(_grads(cf, ctx, graphs, [0, 2, 3, 4, 6, 1, 7], [1, 3, 2, 5, 7, 4, 7], dtype, max_iter, every), dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_long_lists_unequal_counts_and_empty_graphs(cf, ctx, dtype):
    empty = CFG(20, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0))
    graphs = [_wide(40, 1), _wide(129, 2), _wide(90, 3), make_cfg(170, Grammar(counts="trip"), seed=4), empty]
    # tol stops the pairs after different numbers of updates
    _check(_grads(cf, ctx, graphs, [0, 1, 2, 3, 1, 4, 2], [1, 0, 2, 1, 3, 2, 4], dtype, 40, 8, tol=3e-3), dtype)


def test_a_pair_for_every_cu(cf, ctx):
    # 253 pairs: an odd number over the XCDs, unequal work
    graphs = [make_cfg(3 + i % 37, Grammar(counts="trip"), seed=i) for i in range(46)]
    a, b = np.triu_indices(46)
    _check(_grads(cf, ctx, graphs, a[:253], b[:253], "f64", 12, 4), "f64")


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_a_graph_above_the_sets_largest_size(cf, ctx, dtype):
    # 64 x 10 entries fit a slot of 33 x 33, which is all the one-workgroup
    # kernel asks for; the strips' tables are laid out for 33 nodes
    graphs = [make_cfg(n, Grammar(counts="trip"), seed=n) for n in (64, 10, 33, 30)]
    out = []
    for ck in (0, 8):
        gs = cf.pack(ctx, graphs)
        gs.max_nodes = 33
        b = cf.Batch(ctx, gs, np.array([0, 1, 2], np.int32), np.array([1, 0, 3], np.int32), dtype=dtype, max_iter=24,
                     tol=0.0, want_match=True, checkpoint_every=ck)
        b.run()
        g = torch.zeros(gs.total_edges, dtype=torch.float64, device="cuda")
        st = cf.backward(b, torch.ones(3, dtype=torch.float64), g, checkpoint_every=8)
        out.append((g.cpu().numpy(), st.cpu().numpy(), b.results().copy()))
    assert (out[0][1] == 0).all()
    _check(out, dtype)
