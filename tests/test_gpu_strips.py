"""Plain pairs on strips: past LDS against the one-workgroup kernel, large pairs against the oracle.

Both kernels add an entry's terms in the same order; only the FP64 norm sums
are grouped differently (relative 1e-15), so S agrees to a few roundings of
the scale: 20 updates of at most one FP32 rounding each (20 * 2^-24 < 2e-6),
and 1e-13 in FP64.
"""
import numpy as np
import pytest

from cfgsynth import CFG, Grammar, make_cfg
from tests.parity import check_matching, oracle_pair, rel_err

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


def _wide(n, seed):
    """A CFG with hubs: out-degree 6 and in-degree up to 9, repeated jumps."""
    g = make_cfg(n, Grammar(counts="uniform"), seed=seed)
    rng = np.random.default_rng(seed + 1)
    hubs = rng.choice(n - 1, 3, replace=False)
    src = np.concatenate([g.src] + [np.full(5, h) for h in hubs] + [rng.integers(0, n - 1, 7) for _ in hubs])
    dst = np.concatenate([g.dst] + [rng.integers(0, n, 5) for _ in hubs] + [np.full(7, h) for h in hubs])
    return CFG(n, src.astype(np.int32), dst.astype(np.int32),
               np.concatenate([g.count, rng.integers(1, 1000, src.size - g.nnz).astype(np.float64)]))


def _pair(nA, nB, kind):
    if kind == "wide":
        return [_wide(nA, 5), _wide(nB, 6)]
    if kind == "empty":
        return [make_cfg(nA, seed=1), CFG(nB, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0))]
    return [make_cfg(nA, Grammar(counts="trip"), seed=3), make_cfg(nB, Grammar(counts="trip"), seed=4)]


@pytest.mark.parametrize("dtype,tol", [("f32", 2e-6), ("f64", 1e-13)])
@pytest.mark.parametrize("nA,nB,kind,max_iter", [
    (160, 192, "cfg", 20), (205, 207, "cfg", 20), (333, 131, "cfg", 20), (190, 257, "wide", 20),
    (201, 198, "cfg", 1), (201, 198, "wide", 2), (201, 198, "cfg", 3), (150, 170, "empty", 4),
])
def test_strips_equal_the_one_workgroup_kernel(cf, ctx, nA, nB, kind, max_iter, dtype, tol):
    graphs = _pair(nA, nB, kind)
    gs = cf.pack(ctx, graphs)
    one = cf.score(ctx, gs, 0, 1, dtype=dtype, max_iter=max_iter, tol=0.0)
    res, match, S = cf.score_batch(ctx, gs, [0], [1], dtype=dtype, max_iter=max_iter, tol=0.0, want_S=True)
    assert rel_err(one["S"], S[0]) <= tol
    assert one["iters"] == res["iters"][0] and (one["status"] & 15) == (res["status"][0] & 15)
    assert abs(one["nu"] - res["nu"][0]) <= tol * max(res["nu"][0], 1e-300)
    if np.array_equal(one["S"], S[0]):
        np.testing.assert_array_equal(one["match"], match[0])
    ref = oracle_pair(graphs, 0, 1, max_iter=max_iter, tol=0.0)
    assert rel_err(one["S"], ref.S) <= (1e-10 if dtype == "f64" else 1e-5)


def test_strips_converge_and_stop_like_the_oracle(cf, ctx):
    graphs = _pair(150, 200, "cfg")
    gs = cf.pack(ctx, graphs)
    got = cf.score(ctx, gs, 0, 1, dtype="f64", tol=1e-3)
    ref = oracle_pair(graphs, 0, 1, tol=1e-3)
    assert got["iters"] == ref.iters and (got["status"] & 15) == ref.status
    check_matching(got["S"], got["match"], ref.S, "f64")


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-5), ("f64", 1e-10)])
@pytest.mark.parametrize("kind,max_iter", [("cfg", 20), ("wide", 20), ("wide", 1), ("wide", 2), ("wide", 3),
                                           ("empty", 4)])
def test_large_pairs_of_unequal_sizes_on_strips(cf, ctx, kind, max_iter, dtype, tol):
    sizes = [(6, 9), (64, 65), (257, 130), (131, 511)]
    graphs = [g for nA, nB in sizes for g in _pair(nA, nB, kind)]
    gs = cf.pack(ctx, graphs)
    pa, pb = [0, 2, 4, 6, 6], [1, 3, 5, 7, 2]
    res, match, S = cf.score_batch(ctx, gs, pa, pb, dtype=dtype, max_iter=max_iter, tol=0.0, want_S=True,
                                   path="large")
    for q, (a, b) in enumerate(zip(pa, pb)):
        ref = oracle_pair(graphs, a, b, max_iter=max_iter, tol=0.0)
        assert S[q].shape == ref.S.shape and rel_err(S[q], ref.S) <= tol
        assert res["iters"][q] == ref.iters and (res["status"][q] & 15) == ref.status
        check_matching(S[q], match[q], ref.S, dtype)
