"""The matching of pairs past LDS on both sides of its rule (FP64 rows of up to 192 entries by sorted lists, the
others by cached bests).  It must be the greedy matching (value descending, flat index ascending) of the very S it
was taken from: no tolerance."""
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


def _cycle(n):
    """Every entry of S is the same: the order is the flat index alone."""
    src = np.arange(n, dtype=np.int32)
    return CFG(n, src, ((src + 1) % n).astype(np.int32), np.ones(n))


SIZES = [(150, 150), (192, 192), (193, 193), (192, 210), (210, 192), (193, 320), (320, 193), (256, 256), (257, 256)]


@pytest.mark.parametrize("kw", [dict(dtype="f64"), dict(dtype="f32"), dict(dtype="f64", path="damped", alpha=0.8),
                                dict(dtype="f32", path="damped", alpha=0.8)])
@pytest.mark.parametrize("kind", ["cfg", "cycle"])
def test_matching_is_the_greedy_one_of_its_own_scores(cf, kind, kw):
    ctx = cf.Context(0)
    make = _cycle if kind == "cycle" else lambda n: make_cfg(n, Grammar(counts="trip"), seed=n)
    gs = cf.pack(ctx, [make(n) for p in SIZES for n in p])
    a = np.arange(0, 2 * len(SIZES), 2, dtype=np.int32)
    B = cf.Batch(ctx, gs, a, a + 1, max_iter=5, tol=0.0, want_S=True, **kw)
    assert (B.buckets() == 5).all()
    B.run()
    torch.cuda.synchronize()
    for S, match in zip(B.S_list(), B.matches()):
        np.testing.assert_array_equal(match, oracle.greedy_match(S.astype(np.float64))[0])
