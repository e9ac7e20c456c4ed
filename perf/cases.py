"""Timed workloads of the CFG-pair similarity library, through its public entry points.

Each case is one call a program makes again and again: scoring one pair, an
all-pairs batch, a query against a database, large pairs, a training step, and
the measures and clustering beside them.  Graphs come from the seeded CFG
generator; their sizes are fixed by the case (so that every seed costs the
same), structure and execution counts by the seed.

listed() names the cases, draw() gives more of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, work() what a pass
cannot do without, and exact() the result in 64 bits by dense torch products.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import cfgsynth
import paper_1707_02423_amd as cf

DEGREE = 1.365       # jumps per node of the generated graphs
RESULT_BYTES = 40.0  # one pair's result record


def listed():
    return [
        # one pair of small kernels scored on its own: launch and latency of 200 dependent updates
        dict(name="pair_f64_12x16", kind="pair", dtype="f64", n_a=12, n_b=16),
        # one ordinary pair in the default training precision, odd sizes, S resident in one CU's LDS
        dict(name="pair_f32_97x121", kind="pair", dtype="f32", n_a=97, n_b=121),
        # one pair of whole-application graphs, past what one CU's LDS holds
        dict(name="pair_f32_333x410", kind="pair", dtype="f32", n_a=333, n_b=410),
        # the all-pairs matrix of 256 kernels (8 to 128 basic blocks), scores and matchings
        dict(name="allpairs_f32_256", kind="batch", dtype="f32", graphs=256, lo=8, hi=128, tol=1e-12,
             fp64_final=False),
        # the same comparison in double precision, run to convergence
        dict(name="allpairs_f64_96", kind="batch", dtype="f64", graphs=96, lo=8, hi=128, tol=1e-9,
             fp64_final=False),
        # one 200-block kernel looked up in a database of mostly small kernels, 16 best
        dict(name="query_f32_3000", kind="query", dtype="f32", n_query=200, graphs=3000, lo=4, hi=512, k=16),
        # pairs of whole-application graphs of 512 to 2048 blocks
        dict(name="large_f32_8", kind="large", dtype="f32", pairs=8, lo=512, hi=2048, max_iter=200),
        # a training step on the edge weights: scores forward, gradient backward
        dict(name="train_f32_160", kind="train", dtype="f32", pairs=160, lo=16, hi=256, every=8),
        # the paper's comparison with both graphs scaled to a common size first
        dict(name="resized_f32_128", kind="resized", dtype="f32", graphs=128, lo=8, hi=128),
        # the damped measure of the same kind of batch
        dict(name="damped_f32_128", kind="damped", dtype="f32", graphs=128, lo=8, hi=128, alpha=0.85),
        # the five elementwise distances of all pairs
        dict(name="distances_128", kind="distances", graphs=128, lo=8, hi=128, p=3.0),
        # Ward's clustering of kernels by their feature rows (e.g. rows of a score matrix)
        dict(name="ward_768x256", kind="ward", n=768, f=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["pair", "pair", "pair", "batch", "batch", "query", "large", "train", "resized", "damped",
                       "distances", "ward"])
    if kind == "pair":
        return dict(kind=kind, dtype=rng.choice(["f32", "f64"]), n_a=_log_int(rng, 3, 420), n_b=_log_int(rng, 3, 420))
    if kind == "batch":
        dtype = rng.choice(["f32", "f32", "f64"])
        return dict(kind=kind, dtype=dtype, graphs=_log_int(rng, 8, 160), lo=rng.randint(4, 24),
                    hi=_log_int(rng, 32, 150), tol=1e-9 if dtype == "f64" else 1e-12,
                    fp64_final=dtype == "f32" and rng.random() < 0.25)
    if kind == "query":
        return dict(kind=kind, dtype="f32", n_query=_log_int(rng, 20, 300), graphs=_log_int(rng, 200, 3000), lo=4,
                    hi=_log_int(rng, 64, 512), k=rng.choice([1, 10, 16]))
    if kind == "large":
        lo = _log_int(rng, 200, 700)
        return dict(kind=kind, dtype="f32", pairs=rng.randint(1, 6), lo=lo, hi=_log_int(rng, lo + 64, 1800),
                    max_iter=rng.choice([100, 200]))
    if kind == "train":
        return dict(kind=kind, dtype="f32", pairs=_log_int(rng, 8, 160), lo=16, hi=_log_int(rng, 48, 256),
                    every=rng.choice([4, 8, 16]))
    if kind == "ward":
        return dict(kind=kind, n=_log_int(rng, 64, 1200), f=_log_int(rng, 8, 512))
    c = dict(kind=kind, graphs=_log_int(rng, 8, 128), lo=rng.randint(4, 24), hi=_log_int(rng, 32, 150))
    if kind == "distances":
        c["p"] = rng.choice([1.5, 2.0, 3.0])
    else:
        c["dtype"] = "f32"
    if kind == "damped":
        c["alpha"] = round(rng.uniform(0.5, 0.95), 2)
    return c


# ---------------------------------------------------------------- sizes and graphs
def _even(lo, hi, count):
    return np.linspace(lo, hi, count).round().astype(np.int64)


def _sizes(case):
    """Sizes of the case's graphs (of the database's for a query)."""
    kind = case["kind"]
    if kind == "pair":
        return np.array([case["n_a"], case["n_b"]], np.int64)
    if kind == "query":  # p(n) ~ n^-2 on [lo, hi]: quantiles of the discrete law
        n = np.arange(case["lo"], case["hi"] + 1, dtype=np.float64)
        cdf = np.cumsum(n ** -2.0) / np.sum(n ** -2.0)
        q = (np.arange(case["graphs"]) + 0.5) / case["graphs"]
        return n[np.minimum(np.searchsorted(cdf, q), n.size - 1)].astype(np.int64)
    if kind in ("large", "train"):
        # pair p compares graph 2p with 2p + 1: a size and one from elsewhere in the range
        s = _even(case["lo"], case["hi"], 2 * case["pairs"])
        return np.stack([s[: case["pairs"]], s[case["pairs"]:]], 1).reshape(-1)
    return _even(case["lo"], case["hi"], case["graphs"])


def _graphs(case, seed):
    """The case's graphs and its pair list (host arrays)."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    grammar = cfgsynth.Grammar(counts="trip")
    if kind == "large":  # long straight code with shallow loops
        grammar = cfgsynth.Grammar(w_seq=0.70, w_ifthen=0.08, w_ifelse=0.07, w_loop=0.15, p_selfloop=0.05,
                                   max_loop_depth=4, counts="trip")
    if kind == "pair":
        grammar = cfgsynth.Grammar(counts="uniform")
    sizes = _sizes(case)
    if case["kind"] in ("batch", "resized", "damped", "distances", "query"):
        sizes = np.random.default_rng(1).permutation(sizes)  # sizes in no order, the same for every seed
    graphs = [cfgsynth.make_cfg(int(n), grammar, rng) for n in sizes]
    if kind == "query":
        graphs = [cfgsynth.make_cfg(case["n_query"], grammar, rng)] + graphs
        b = np.arange(1, len(graphs), dtype=np.int32)
        return graphs, np.zeros_like(b), b
    if kind in ("pair", "large", "train"):
        a = np.arange(0, len(graphs), 2, dtype=np.int32)
        return graphs, a, a + 1
    a, b = cfgsynth.all_pairs(len(graphs))
    return graphs, a, b


# ---------------------------------------------------------------- what a program holds, and one pass
_CTX = None


def _context():
    global _CTX
    if _CTX is None:
        _CTX = cf.Context(0)
    return _CTX


def _ward_points(case, seed):
    """Feature rows in loose groups, as kernels of the same application score alike."""
    g = torch.Generator(device="cpu").manual_seed(int(seed))
    n, f = case["n"], case["f"]
    centres = torch.rand(max(2, n // 24), f, generator=g, dtype=torch.float64) * 1.3
    which = torch.randint(0, centres.shape[0], (n,), generator=g)
    return (centres[which] + 0.1 * torch.randn(n, f, generator=g, dtype=torch.float64)).cuda()


def prepare(case, seed):
    ctx = _context() if case["kind"] in ("pair", "distances", "ward") else cf.Context(0)
    kind = case["kind"]
    if kind == "ward":
        return dict(case=case, ctx=ctx, X=_ward_points(case, seed))
    graphs, a, b = _graphs(case, seed)
    gs = cf.pack(ctx, graphs)
    st = dict(case=case, ctx=ctx, gs=gs)
    if kind == "distances":
        st["a"], st["b"] = (torch.as_tensor(x).cuda() for x in (a, b))
    elif kind == "batch":
        st["batch"] = cf.Batch(ctx, gs, a, b, dtype=case["dtype"], tol=case["tol"], fp64_final=case["fp64_final"])
    elif kind == "query":
        st["batch"] = cf.Batch(ctx, gs, a, b, dtype=case["dtype"])
    elif kind == "resized":
        st["batch"] = cf.Batch(ctx, gs, a, b, dtype=case["dtype"], resize="bilinear")
    elif kind == "damped":
        st["batch"] = cf.Batch(ctx, gs, a, b, dtype=case["dtype"], path="damped", alpha=case["alpha"])
    elif kind == "large":
        st["batch"] = cf.Batch(ctx, gs, a, b, dtype=case["dtype"], path="large", max_iter=case["max_iter"],
                               want_S=True)
    elif kind == "train":
        st["a"], st["b"] = a, b
        g = torch.Generator(device="cpu").manual_seed(int(seed))
        st["grad_out"] = torch.rand(a.size, generator=g, dtype=torch.float64).cuda() + 0.5
    return st


def _fields(res, n):
    """Every field of n result records."""
    f = res.view(torch.float64).view(n, 5)
    i = res.view(torch.int32).view(n, 10)
    return dict(score=f[:, 0], nu=f[:, 1], delta=f[:, 2], margin=f[:, 3], iters=i[:, 8], status=i[:, 9])


def _padded(grad, case):
    return torch.nn.functional.pad(grad, (0, 2 * int(_sizes(case).sum()) - grad.numel()))


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "pair":
        out = cf.score(ctx, st["gs"], 0, 1, dtype=case["dtype"], sync=False)
        return dict(_fields(out["res"], 1), match=out["match"], S=out["S"])
    if kind == "distances":
        return cf.distances(ctx, st["gs"], st["a"], st["b"], p=case["p"])
    if kind == "ward":
        return cf.ward(ctx, st["X"])
    if kind == "train":
        w = st["gs"].w.detach().requires_grad_()
        scores = cf.CfsimScore.apply(w, ctx, st["gs"], st["a"], st["b"], case["dtype"], 200, 1e-12, case["every"])
        scores.backward(st["grad_out"])
        # a node has at most two jumps: the gradient in a buffer that holds any set of these sizes
        return dict(scores=scores.detach(), grad=_padded(w.grad, case))
    batch = st["batch"]
    batch.run()
    out = dict(_fields(batch.res, batch.n_pairs), match=batch.match)
    if kind == "large":
        out["S"] = batch.S
    if kind == "query":
        out["top"], out["top_score"] = batch.topk(case["k"])
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "ward":
        n, f = float(case["n"]), float(case["f"])
        # distances of all pairs, then per merge one recurrence over the clusters left
        return dict(bytes=8.0 * (n * f + 4.0 * (n - 1)), flops=1.5 * n * n * f + 8.0 * 0.5 * n * n)
    s = _sizes(case).astype(np.float64)
    graph_bytes = float(np.sum(s)) * (DEGREE * 20.0 + 8.0)  # weights, both index lists, offsets
    if kind in ("pair", "large", "train"):
        na, nb = s[0::2], s[1::2]
    elif kind == "query":
        nb = s
        na = np.full_like(s, case["n_query"])
        graph_bytes += case["n_query"] * (DEGREE * 20.0 + 8.0)
    else:
        i, j = np.triu_indices(s.size, k=1)
        na, nb = s[i], s[j]
    pairs = float(na.size)
    if kind == "distances":
        m = np.maximum(na, nb)
        return dict(bytes=graph_bytes + pairs * 48.0, flops=float(np.sum(m * m)) * 10.0)
    iters = float(case.get("max_iter", 200))
    edges = DEGREE * DEGREE * na * nb
    # one multiply-add per pair of jumps and direction, a scale and a squared norm per entry
    flops = iters * float(np.sum(4.0 * edges + 3.0 * na * nb))
    out = pairs * RESULT_BYTES + 4.0 * float(np.sum(nb))
    if kind in ("pair", "large"):
        out += float(np.sum(na * nb)) * (8.0 if case["dtype"] == "f64" else 4.0)
    if kind == "train":
        flops *= 4.0  # the adjoint operator, and the two edge sums, beside the forward
        out = pairs * 16.0 + float(np.sum(s)) * DEGREE * 8.0
    return dict(bytes=graph_bytes + out, flops=flops)


# ---------------------------------------------------------------- the same results in 64 bits
def _dense(g, w=None):
    """Dense transition matrix (rows sum to one), from the jump counts or given weights."""
    P = np.zeros((g.n, g.n))
    np.add.at(P, (g.src, g.dst), g.count)
    tot = P.sum(1, keepdims=True)
    return np.divide(P, tot, out=np.zeros_like(P), where=tot > 0)


def _interp(m, M):
    """Order-1 interpolation matrix from m to M points."""
    R = np.zeros((M, m))
    for p in range(M):
        x = p * (m - 1)
        r0, f = x // (M - 1), (x % (M - 1)) / (M - 1)
        R[p, r0] += 1.0 - f
        R[p, min(r0 + 1, m - 1)] += f
    return R


def _resized(P, M):
    if P.shape[0] == M:
        return P
    R = _interp(P.shape[0], M)
    return R @ P @ R.T


def _stack(mats, n):
    out = torch.zeros(len(mats), n, n, dtype=torch.float64)
    for k, x in enumerate(mats):
        out[k, : x.shape[0], : x.shape[1]] = torch.as_tensor(x)
    return out.cuda()


def _apply(A, B, S):
    At, Bt = A.transpose(1, 2).contiguous(), B.transpose(1, 2).contiguous()
    return lambda X: torch.bmm(torch.bmm(B, X), At) + torch.bmm(torch.bmm(Bt, X), A)


def _iterate(A, B, na, nb, max_iter, tol):
    """S and nu of every pair of a padded group (normalised iteration)."""
    P, N, K = A.shape[0], B.shape[1], A.shape[1]
    rows = torch.arange(N, device="cuda")[None, :, None] < nb[:, None, None]
    cols = torch.arange(K, device="cuda")[None, None, :] < na[:, None, None]
    S = torch.where(rows & cols, (1.0 / torch.sqrt((na * nb).double()))[:, None, None], 0.0)
    M = _apply(A, B, S)
    nu = torch.zeros(P, dtype=torch.float64, device="cuda")
    live = torch.ones(P, dtype=torch.bool, device="cuda")
    old = S
    for k in range(1, max_iter + 1):
        Y = M(S)
        norm = Y.flatten(1).norm(dim=1)
        T = Y / torch.where(norm > 0, norm, 1.0)[:, None, None]
        S_new = torch.where(live[:, None, None], T, S)
        nu = torch.where(live, norm, nu)
        S = S_new
        if k % 2 == 0:
            live = live & ((S - old).flatten(1).norm(dim=1) >= tol)
            old = S
            if k % 20 == 0 and not bool(live.any()):
                break
    return S, nu


def _damped(A, B, na, nb, alpha, max_iter, tol):
    P, N, K = A.shape[0], B.shape[1], A.shape[1]
    rows = torch.arange(N, device="cuda")[None, :, None] < nb[:, None, None]
    cols = torch.arange(K, device="cuda")[None, None, :] < na[:, None, None]
    E = torch.where(rows & cols, (1.0 / (na * nb).double())[:, None, None], 0.0)
    d = B.sum(1)[:, :, None] * A.sum(1)[:, None, :] + B.sum(2)[:, :, None] * A.sum(2)[:, None, :]
    inv = torch.where(d > 0, 1.0 / torch.where(d > 0, d, 1.0), 0.0)
    M = _apply(A, B, E)
    x = E
    live = torch.ones(P, dtype=torch.bool, device="cuda")
    for _ in range(max_iter):
        y = alpha * M(x * inv) + (1.0 - alpha) * E
        change = (y - x).flatten(1).abs().sum(1)
        x = torch.where(live[:, None, None], y, x)
        live = live & (change >= tol)
        if not bool(live.any()):
            break
    nu = x.flatten(1).norm(dim=1)
    return x / nu[:, None, None], nu


def _greedy(S, na, nb):
    """Score of the greedy matching of every pair (largest entry first)."""
    P, N, K = S.shape
    rows = torch.arange(N, device="cuda")[None, :, None] < nb[:, None, None]
    cols = torch.arange(K, device="cuda")[None, None, :] < na[:, None, None]
    X = torch.where(rows & cols, S, -1.0)
    score = torch.zeros(P, dtype=torch.float64, device="cuda")
    at = torch.arange(P, device="cuda")
    picks = torch.full((P, N), -1, dtype=torch.int64, device="cuda")
    for _ in range(int(torch.minimum(na, nb).max())):
        v, i = X.view(P, -1).max(1)
        r, c = i // K, i % K
        ok = v >= 0
        score += torch.where(ok, v, 0.0)
        picks[at, r] = torch.where(ok, c, picks[at, r])
        X[at, r, :] = -1.0
        X[at, :, c] = -1.0
    return score, picks


def _groups(na, nb, most_bytes=1.5e9):
    """Pair indices of similar padded sizes, few enough to iterate at once."""
    pad = lambda n: int(min(p for p in (16, 32, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 4096)
                            if p >= n))
    by = {}
    for q, (x, y) in enumerate(zip(na, nb)):
        by.setdefault((pad(x), pad(y)), []).append(q)
    for (x, y), idx in by.items():
        step = max(1, int(most_bytes / (8.0 * max(x, y) ** 2)))
        for o in range(0, len(idx), step):
            yield x, y, idx[o:o + step]


def _exact_ward(case, seed):
    if case["n"] > 1200:
        return None
    X = _ward_points(case, seed).cpu().numpy()
    n = X.shape[0]
    D = np.stack([((X[i] - X) ** 2).sum(-1) for i in range(n)])
    D[np.tril_indices(n)] = np.inf  # slot i < j
    size, ident = np.ones(n), np.arange(n)
    near = D.argmin(1)
    best = D[np.arange(n), near]
    Z = np.zeros((n - 1, 4))
    alive = np.ones(n, bool)
    for s in range(n - 1):
        i = int(best.argmin())
        j = int(near[i])
        h = D[i, j]
        Z[s] = [min(ident[i], ident[j]), max(ident[i], ident[j]), h, size[i] + size[j]]
        di = np.where(np.arange(n) < i, D[:, i], D[i])
        dj = np.where(np.arange(n) < j, D[:, j], D[j])
        new = ((size[i] + size) * di + (size[j] + size) * dj - size * h) / (size[i] + size[j] + size)
        alive[j] = False
        new[~alive] = np.inf
        new[i] = np.inf
        size[i] += size[j]
        ident[i] = n + s
        D[j, :] = np.inf
        D[:, j] = np.inf
        D[:i, i] = new[:i]
        D[i, i + 1:] = new[i + 1:]
        stale = np.nonzero(alive & ((near == i) | (near == j)))[0]
        for r in np.union1d(stale, [i]):
            near[r] = D[r].argmin()
            best[r] = D[r, near[r]]
        lower = np.nonzero(alive[:i] & (D[:i, i] < best[:i]))[0]
        near[lower] = i
        best[lower] = D[lower, i]
        best[j] = np.inf
    return Z


def _exact_distances(case, graphs, a, b):
    P = [_dense(g) for g in graphs]
    cache = {}

    def at(g, M):
        if (g, M) not in cache:
            cache[(g, M)] = torch.as_tensor(_resized(P[g], M)).cuda()
        return cache[(g, M)]

    out = torch.zeros(a.size, 5, dtype=torch.float64, device="cuda")
    for q, (i, j) in enumerate(zip(a, b)):
        M = max(graphs[i].n, graphs[j].n)
        x, y = at(int(i), M), at(int(j), M)
        d = (x - y).abs()
        d2, xx, yy, xy = (d * d).sum(), (x * x).sum(), (y * y).sum(), (x * y).sum()
        out[q] = torch.stack([d2.sqrt(), d.sum(), (d ** case["p"]).sum() ** (1.0 / case["p"]),
                              d2 / (xx + yy - xy), 1.0 - xy / (xx * yy).sqrt()])
    return out.cpu()


def _exact_train(case, seed, graphs, a, b):
    """Scores and d(sum grad_out score)/dw by autograd, matching held fixed."""
    g = torch.Generator(device="cpu").manual_seed(int(seed))
    gout = (torch.rand(a.size, generator=g, dtype=torch.float64) + 0.5).cuda()
    src, dst, wts, off = [], [], [], [0]
    for x in graphs:  # packed edge order: rows, then columns
        o = np.lexsort((x.dst, x.src))
        src.append(x.src[o])
        dst.append(x.dst[o])
        tot = np.bincount(x.src, weights=x.count, minlength=x.n)
        wts.append(np.divide(x.count[o], tot[x.src[o]], out=np.zeros(o.size), where=tot[x.src[o]] > 0))
        off.append(off[-1] + o.size)
    w = torch.as_tensor(np.concatenate(wts)).cuda().requires_grad_()
    scores = torch.zeros(a.size, dtype=torch.float64, device="cuda")
    na = np.array([graphs[i].n for i in a])
    nb = np.array([graphs[j].n for j in b])
    for x, y, idx in _groups(na, nb, 2.5e7):
        def dense(which, n):
            e = np.concatenate([np.arange(off[t], off[t + 1]) for t in which])
            k = np.concatenate([np.full(off[t + 1] - off[t], q) for q, t in enumerate(which)])
            flat = k * n * n + np.concatenate([src[t] for t in which]) * n + np.concatenate([dst[t] for t in which])
            z = torch.zeros(len(which) * n * n, dtype=torch.float64, device="cuda")
            return z.index_add(0, torch.as_tensor(flat).cuda(), w[torch.as_tensor(e).cuda()]).view(-1, n, n)
        A, B = dense([int(a[q]) for q in idx], x), dense([int(b[q]) for q in idx], y)
        ta, tb = torch.as_tensor(na[idx]).cuda(), torch.as_tensor(nb[idx]).cuda()
        with torch.no_grad():
            S, _ = _iterate(A, B, ta, tb, 200, 1e-12)
            score, picks = _greedy(S, ta, tb)
        rows = torch.arange(y, device="cuda")[None, :, None] < tb[:, None, None]
        cols = torch.arange(x, device="cuda")[None, None, :] < ta[:, None, None]
        S = torch.where(rows & cols, (1.0 / torch.sqrt((ta * tb).double()))[:, None, None], 0.0)
        M = _apply(A, B, S)
        for _ in range(200):
            Y = M(S)
            S = Y / Y.flatten(1).norm(dim=1)[:, None, None]
        got = torch.where(picks >= 0, S.gather(2, picks.clamp(min=0)[:, :, None])[:, :, 0], 0.0).sum(1)
        t = torch.as_tensor(np.asarray(idx)).cuda()
        scores[t] = got.detach()
        (got * gout[t]).sum().backward()
    return dict(scores=scores.cpu(), grad=_padded(w.grad, case).cpu())


def exact(case, seed):
    kind = case["kind"]
    if kind == "ward":
        return _exact_ward(case, seed)
    graphs, a, b = _graphs(case, seed)
    if kind == "distances":
        return _exact_distances(case, graphs, a, b)
    if kind == "train":
        return _exact_train(case, seed, graphs, a, b)
    P = [_dense(g) for g in graphs]
    na = np.array([graphs[i].n for i in a])
    nb = np.array([graphs[j].n for j in b])
    if kind == "resized":
        na = nb = np.maximum(na, nb)
    scores = torch.zeros(a.size, dtype=torch.float64, device="cuda")
    nus = torch.zeros_like(scores)
    Ss = [None] * a.size
    cache = {}

    def at(g, M):
        if kind != "resized":
            return P[g]
        if (g, M) not in cache:
            cache[(g, M)] = _resized(P[g], M)
        return cache[(g, M)]

    for x, y, idx in _groups(na, nb):
        A = _stack([at(int(a[q]), int(na[q])) for q in idx], x)
        B = _stack([at(int(b[q]), int(nb[q])) for q in idx], y)
        ta, tb = torch.as_tensor(na[idx]).cuda(), torch.as_tensor(nb[idx]).cuda()
        if kind == "damped":
            S, nu = _damped(A, B, ta, tb, case["alpha"], 200, 1e-12)
        else:
            S, nu = _iterate(A, B, ta, tb, case.get("max_iter", 200), case.get("tol", 1e-12))
        t = torch.as_tensor(np.asarray(idx)).cuda()
        scores[t], _ = _greedy(S, ta, tb)
        nus[t] = nu
        if kind in ("pair", "large"):
            for k, q in enumerate(idx):
                Ss[q] = S[k, : nb[q], : na[q]].reshape(-1)
    out = dict(score=scores.cpu(), nu=nus.cpu(), delta=None, margin=None, iters=None, status=None, match=None)
    if kind in ("pair", "large"):
        out["S"] = torch.cat(Ss).cpu()
    if kind == "query":
        out["top"], out["top_score"] = None, torch.topk(scores, case["k"]).values.cpu()
    return out
