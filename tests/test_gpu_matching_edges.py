"""The cached-best matching at the edges of its chunks of 64 columns and rows
per wave, and on ties.  It must be the greedy matching (value descending, flat
index ascending) of the very S it was taken from: no tolerance."""
import numpy as np
import pytest

import oracle
from cfgsynth import CFG, Grammar, make_cfg

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


def _cycle(n):
    """Every entry of S is the same: the order is the flat index alone."""
    src = np.arange(n, dtype=np.int32)
    return CFG(n, src, ((src + 1) % n).astype(np.int32), np.ones(n))


SIZES = [(1, 1), (2, 63), (64, 64), (65, 63), (128, 129), (16, 200), (129, 3), (257, 70), (260, 258)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind", ["cfg", "cycle"])
def test_matching_is_the_greedy_one_of_its_own_scores(cf, ctx, kind, dtype):
    make = lambda n: _cycle(n) if kind == "cycle" or n < 2 else make_cfg(n, Grammar(counts="trip"), seed=n)
    graphs = [make(n) for p in SIZES for n in p]
    gs = cf.pack(ctx, graphs)
    a = np.arange(0, len(graphs), 2, dtype=np.int32)
    _, match, S = cf.score_batch(ctx, gs, a, a + 1, dtype=dtype, max_iter=9, tol=0.0, want_S=True)
    for q in range(len(SIZES)):
        np.testing.assert_array_equal(match[q], oracle.greedy_match(S[q].astype(np.float64))[0])
        one = cf.score(ctx, gs, 2 * q, 2 * q + 1, dtype=dtype, max_iter=9, tol=0.0)
        np.testing.assert_array_equal(one["match"], oracle.greedy_match(one["S"].astype(np.float64))[0])
