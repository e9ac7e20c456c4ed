// Reverse mode (adjoint.hip states the recurrences) with every update of all
// pairs in one launch, on strips of four rows of the transposed iterates
// (strips.h), so that a call's largest pairs run on as many CUs as they have
// strips instead of on one each.
//
// Segments of `ckpt` updates are walked backwards.  Round t recomputes segment
// s_last - t forward (Y_{k+1} = M S_k, kept unnormalised: readers multiply by
// 1 / nu, which rounds as the stored product would) while it reverses the
// segment of the round before; launch j of a round holds, for every pair,
//   - the forward strips of update j,
//   - the strips of G_k = M Ybar_k with Ybar_k = (G_{k+1} - a S_{k+1}) / nu_k
//     formed as the sources are read, and <G_k, S_k> for the next launch's a,
//   - the edge sums from Ybar_k and S_k: eight waves, as many partial sums per
//     A edge as the one-workgroup kernel has, in its order.
// A seam launch between rounds takes a = <G, S> against the recomputed last
// iterate of the next segment and transposes the checkpoint of the one after.
// Iterates are kept twice: X = S^T for the strips (consecutive B nodes) and S
// with rows of A nodes for the edge sums.  The entries' terms are added in the
// order of the one-workgroup kernel: the same bits; the FP64 norms, dots and
// gradient sums are grouped differently.
//
// A launch is bound by instruction issue and the latency of its reads: 160 FP32
// pairs of 16-256 nodes 61 us per launch (edge sums alone 28, strips alone 41,
// an empty launch 5), 12.9 ms for 200 updates against 43.4 ms with one
// workgroup per pair, which waits for the largest.  One workgroup per strip
// with a barrier between its stages took 80 us (the scales' sums repeated in
// every wave), the strips of both directions in one item 107 us (spills), one
// wave per partial sum of the edges 10 us more.
#include "adjoint_job.h"
#include "strips.h"

namespace cfsim {

namespace {

using namespace dev;
using namespace strips;

constexpr int kDP = 4;            // predecessor slots of the column lists
constexpr int kNT = 256;
constexpr int kNW = kNT / kWave;
constexpr int kMaxPairs = 1024;   // pairs of a call (adj_items: one thread each)
constexpr int kXcds = 8;
constexpr int kListEdges = kBwdLds / 12;  // edges of a pair that fits the other kernel's LDS
constexpr int kEdgeGroups = kEdgeWaves;   // workgroups of a pair's edge sums

struct AdjPair {
    int p, nR, nC, K, s_last, kept_a, kept_b, strips, active;
};
// A partial sum of a pair's edges (a workgroup's work) or a strip (a wave's),
// with its pair (one read instead of two dependent ones).
struct alignas(16) AdjItem {
    AdjPair st;
    int slot, index;
};

// Byte offsets in a pair's slot.
struct AdjLayout {
    size_t buf, cols, tabs, src, g_a, g_b, nu, dot, inv, total;
    int max_strips;
};

struct AdjJob {
    BwdJob J;
    AdjLayout L;
    int np;                  // pairs
    AdjPair* pairs;
    AdjItem* items;          // by XCD: its pairs' edge sums, then their strips
    int* item_off;           // [kXcds][2] and the end
    unsigned char* slots;
};

size_t up(size_t x) { return (x + 255) & ~(size_t)255; }

template <typename T>
AdjLayout layout_of(int max_nodes, long long slot_elems, int ckpt) {
    AdjLayout l;
    l.max_strips = (max_nodes + kRows - 1) / kRows;
    l.buf = up((size_t)(slot_elems + (kRows - 1) * (long long)max_nodes) * sizeof(T));
    size_t o = (size_t)(4 * ckpt + 8) * l.buf;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += up(bytes);
        return at;
    };
    l.cols = take(cols_bytes<T>(max_nodes, kDP));
    l.tabs = take((size_t)l.max_strips * sizeof(StripTab<T>));
    l.src = take((size_t)kListEdges * 4);
    l.g_a = take((size_t)kEdgeWaves * kAChunks * kWave * 8);
    l.g_b = take((size_t)kListEdges * 8);
    l.nu = take((size_t)2 * ckpt * l.max_strips * 8);
    l.dot = take((size_t)2 * l.max_strips * 8);
    l.inv = take((size_t)2 * ckpt * sizeof(T));
    l.total = o;
    return l;
}

size_t group_items(int np, int max_strips) { return (size_t)np * (kEdgeGroups + (size_t)max_strips); }
size_t header_bytes(int np, int max_strips) {
    return up((2 * kXcds + 1) * 4) + up((size_t)np * sizeof(AdjPair)) + up(group_items(np, max_strips) * sizeof(AdjItem));
}

// ---------------------------------------------------------------- a pair's slot
template <typename T>
struct Slot {
    unsigned char* base;
    const AdjLayout* l;
    int ckpt;

    __device__ T* buf(int b) const { return reinterpret_cast<T*>(base + (size_t)b * l->buf); }
    // slot s (1 .. ckpt) of the segment of parity par: X and its natural layout
    __device__ T* seg_x(int par, int s) const { return buf(par * ckpt + s - 1); }
    __device__ T* seg_n(int par, int s) const { return buf((2 + par) * ckpt + s - 1); }
    __device__ T* first_x(int ring) const { return buf(4 * ckpt + ring); }   // a segment's first iterate
    __device__ T* start_n() const { return buf(4 * ckpt + 3); }              // S_0
    __device__ T* g_x(int par) const { return buf(4 * ckpt + 4 + par); }
    __device__ T* g_n(int par) const { return buf(4 * ckpt + 6 + par); }
    __device__ double* nu(int par, int s) const {
        return reinterpret_cast<double*>(base + l->nu) + (size_t)(par * ckpt + s - 1) * l->max_strips;
    }
    __device__ double* dot(int par) const {
        return reinterpret_cast<double*>(base + l->dot) + (size_t)par * l->max_strips;
    }
    // 1 / nu of a segment's iterates, left by the first that sums the partials
    __device__ T* inv(int par, int s) const { return reinterpret_cast<T*>(base + l->inv) + par * ckpt + s - 1; }
    __device__ Cols<T> cols(int nR) const { return carve_cols<T>(base + l->cols, nR, kDP); }
    __device__ StripTab<T>* tabs() const { return reinterpret_cast<StripTab<T>*>(base + l->tabs); }
    __device__ int* src() const { return reinterpret_cast<int*>(base + l->src); }  // of A's edges, then B's
    __device__ double* grad_a() const { return reinterpret_cast<double*>(base + l->g_a); }
    __device__ double* grad_b() const { return reinterpret_cast<double*>(base + l->g_b); }
};
template <typename T>
__device__ inline Slot<T> slot_of(const AdjJob& A, int slot) {
    return Slot<T>{A.slots + (size_t)slot * A.L.total, &A.L, A.J.ckpt};
}

__device__ inline int row_stride(int nC) { return (nC + kRows - 1) & ~(kRows - 1); }

// Sum of a pair's partials, the same in every wave, in two parts: the reads,
// and the sum of what they brought.
__device__ inline double part_read(const double* part, int n) {
    double x = 0.0;
    for (int q = (int)(threadIdx.x & (kWave - 1)); q < n; q += kWave) x += part[q];
    return x;
}
template <typename T>
__device__ inline T inv_of(double part) {
    return uni(T(1.0 / sqrt(wave_sum(part))));
}

// ---------------------------------------------------------------- set-up
template <typename T>
__global__ __launch_bounds__(kNT) void adj_init(AdjJob A) {
    const int slot = blockIdx.y, p = slot;
    const int tid = blockIdx.x * kNT + threadIdx.x, nt = gridDim.x * kNT;
    GraphRef a{}, b{};
    AdjPair st{};
    bool on = bwd_pair(A.J, p, &a, &b);
    if (on) on = bwd_on_strips(A.J, a, b, bwd_shape(a, b, (int)sizeof(T)));
    const double gs = A.J.grad_score[p];
    const cfsim_pair_result* fr = A.J.fwd + p;
    if (on) {
        if (tid == 0 && A.J.pair_status) A.J.pair_status[p] = 0;
        st.active = !((fr->status & CFSIM_DEGENERATE) || fr->iters == 0 || gs == 0.0);
    }
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            st.p = p;
            if (st.active) {
                st.nR = b.n;
                st.nC = a.n;
                st.K = fr->iters;
                st.s_last = (st.K - 1) / A.J.ckpt;
                st.kept_a = a.rp[a.n];
                st.kept_b = b.rp[b.n];
                st.strips = (a.n + kRows - 1) / kRows;
            }
            A.pairs[slot] = st;
        }
    }
    if (!st.active) return;
    const Slot<T> S = slot_of<T>(A, slot);
    const int nR = b.n, nC = a.n, ld = row_stride(nC);
    const Cols<T> cols = S.cols(nR);
    for (int i = tid; i < cols.stride; i += nt) build_col<T, kDP>(b, i, cols);
    for (int s = tid; s * kRows < nC; s += nt) build_strip<T, kDP>(a, s * kRows, nR, S.tabs() + s);
    int* src_a = S.src();
    int* src_b = src_a + a.nnz;
    for (int r = tid; r < nC; r += nt)
        for (int e = a.rp[r]; e < a.rp[r + 1]; ++e) src_a[e] = r;
    for (int r = tid; r < nR; r += nt)
        for (int e = b.rp[r]; e < b.rp[r + 1]; ++e) src_b[e] = r;
    for (int e = tid; e < kEdgeWaves * kAChunks * kWave; e += nt) S.grad_a()[e] = 0.0;
    for (int e = tid; e < b.nnz; e += nt) S.grad_b()[e] = 0.0;
    // S_0, and G = g * indicator(matching)
    const T s0 = T(1.0 / sqrt((double)nR * (double)nC));
    const int32_t* match = A.J.match + A.J.match_off[p];
    T* gx = S.g_x(0);
    T* gn = S.g_n(0);
    T* sn = S.start_n();
    for (int o = tid; o < nR * nC; o += nt) {
        const int i = o / nC, c = o - i * nC;
        sn[o] = s0;
        gn[i * ld + c] = match[i] == c ? T(gs) : T(0);
    }
    for (int o = tid; o < nR * nC; o += nt) {
        const int c = o / nR, i = o - c * nR;
        gx[o] = match[i] == c ? T(gs) : T(0);
    }
}

// Work items: a pair's on one XCD (its iterates stay in that L2), the
// pairs cut into eight ranges of about equal work; the edge sums, which take
// longest, first.
__global__ __launch_bounds__(kMaxPairs) void adj_items(AdjJob A) {
    __shared__ int strips[kMaxPairs], xcd[kMaxPairs], at_e[kMaxPairs], at_s[kMaxPairs];
    __shared__ int off[kXcds + 1], ne[kXcds], ns[kXcds];
    const int tid = threadIdx.x;
    const bool act = tid < A.np && A.pairs[tid].active;
    strips[tid] = act ? A.pairs[tid].strips : 0;
    __syncthreads();
    if (tid == 0) {
        long long total = 0, run = 0;
        for (int q = 0; q < A.np; ++q) total += strips[q] ? strips[q] + kEdgeGroups : 0;
        for (int x = 0; x < kXcds; ++x) ne[x] = ns[x] = 0;
        for (int q = 0; q < A.np; ++q) {
            if (!strips[q]) continue;
            const int work = strips[q] + kEdgeGroups;
            const int x = (int)((2 * run + work) * kXcds / (2 * total));
            run += work;
            xcd[q] = x;
            at_e[q] = ne[x];
            at_s[q] = ns[x];
            ne[x] += kEdgeGroups;
            ns[x] += strips[q];
        }
        int o = 0;
        for (int x = 0; x < kXcds; ++x) {
            off[x] = o;
            o += ne[x] + ns[x];
        }
        off[kXcds] = o;
    }
    __syncthreads();
    if (tid <= kXcds) A.item_off[2 * tid] = off[tid];
    if (tid < kXcds) A.item_off[2 * tid + 1] = off[tid] + ne[tid];
    if (!act) return;
    const int x = xcd[tid];
    AdjItem* it = A.items + off[x];
    const AdjPair st = A.pairs[tid];
    for (int g = 0; g < kEdgeGroups; ++g) it[at_e[tid] + g] = AdjItem{st, tid, g};
    for (int s = 0; s < strips[tid]; ++s) it[ne[x] + at_s[tid] + s] = AdjItem{st, tid, s};
}

// ---------------------------------------------------------------- strips
// Values the operator is applied to: S_k from an unnormalised iterate, or
// Ybar_k from G_{k+1} and S_{k+1}.  A read takes raw values (so that it can be
// issued before the scales are known); finish() makes the entry.
template <typename T>
struct Scaled {
    typedef T Raw;
    const T* x;
    T inv;
    __device__ Raw read(uint32_t off) const { return at_byte(x, off); }
    __device__ T finish(Raw r) const { return r * inv; }
};
template <typename T>
struct Ybar {
    struct Raw {
        T g, s;
    };
    const T *g, *s1;
    T a, inv;
    __device__ Raw read(uint32_t off) const { return Raw{at_byte(g, off), at_byte(s1, off)}; }
    __device__ T finish(Raw r) const { return fma_t(-a, r.s * inv, r.g) * inv; }
};

// Stage A by one wave with the values of `ld` (wave_sources); scales() is
// called behind the first reads.  Weights of 16 sources stand in one register,
// of which the matrix instruction broadcasts the block it needs.
template <typename Load, typename Scales>
__device__ __forceinline__ void stage(Load& ld, const Scales& scales, int nR, const StripTab<float>* t,
                                      Quad<float>* P1, Quad<float>* P2) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const float* wt = &t->ws[0][0];  // ws and wp lie one behind the other
    const float w = wt[lane], w2 = wt[64 + (lane & 31)];
    const int src = t->src_s[lane < 24 ? lane : 0];  // src_s and src_p too
    const int ns = uni(t->ns), np = uni(t->np);
    const int nch = (nR + kWave - 1) / kWave;
    for (int ch = 0; ch < nch; ++ch) {
        const int col = ch * kWave + lane;
        const uint32_t at = (uint32_t)min(col, nR - 1) * 4u;
        typename Load::Raw x[6][4];
        auto read = [&](int g, int q0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) x[g][q] = ld.read((uint32_t)lane_value(src, q0 + q) + at);
        };
        read(0, 0);
        read(2, 8);
        if (ns > 4) read(1, 4);
        if (np > 4) read(3, 12);
        if (ch == 0) scales();
        floatx4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = {0.0f, 0.0f, 0.0f, 0.0f};
        auto four = [&](int g, float (&v)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = ld.finish(x[g][q]);
        };
        float v[4];
        four(0, v);
        add_blocks<0>(a, w, v);
        four(2, v);
        add_blocks<8>(b, w, v);
        if (ns > 4) {
            four(1, v);
            add_blocks<4>(a, w, v);
        }
        if (np > 4) {
            four(3, v);
            add_blocks<12>(b, w, v);
        }
        if (np > 8) {
            read(4, 16);
            four(4, v);
            add_blocks<0>(b, w2, v);
        }
        if (np > 12) {
            read(5, 20);
            four(5, v);
            add_blocks<4>(b, w2, v);
        }
        *reinterpret_cast<floatx4*>(&P1[col]) = a;
        *reinterpret_cast<floatx4*>(&P2[col]) = b;
    }
}
template <typename Load, typename Scales>
__device__ __forceinline__ void stage(Load& ld, const Scales& scales, int nR, const StripTab<double>* t,
                                      Quad<double>* P1, Quad<double>* P2) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int src = t->src_s[lane < 24 ? lane : 0];  // src_s and src_p lie one behind the other
    const int ns = uni(t->ns), np = uni(t->np);
    const int nch = (nR + kWave - 1) / kWave;
    for (int ch = 0; ch < nch; ++ch) {
        const int col = ch * kWave + lane;
        const uint32_t at = (uint32_t)min(col, nR - 1) * 8u;
        Quad<double> a{}, b{};
        auto add = [&](Quad<double>& acc, int q0, const double (*w)[kRows]) {
            typename Load::Raw x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = ld.read((uint32_t)lane_value(src, q0 + q) + at);
            if (ch == 0 && q0 == 0) scales();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double v = ld.finish(x[q]);
#pragma unroll
                for (int r = 0; r < kRows; ++r) acc.v[r] = fma_t(w[q][r], v, acc.v[r]);
            }
        };
        add(a, 0, t->ws);
        if (ns > 4) add(a, 4, t->ws + 4);
        add(b, 8, t->wp);
        for (int q = 4; q < np; q += 4) add(b, 8 + q, t->wp + q);
        P1[col] = a;
        P2[col] = b;
    }
}

// long_row_terms for column i from its slots: two orders, by the length of the
// column's lists; entries of longer lists come from its graph.
template <typename T, typename Load>
__device__ __forceinline__ T row_rest(const Load& ld, const ColSlots<T, kDP>& k, int nR, int pad, int i,
                                      const GraphRef& R, const GraphRef& C, int c) {
    const auto X = [&](int row, int off) {  // neighbour at byte offset `off` of P1 / P2
        const uint32_t u = (uint32_t)min(off / (int)(kRows * sizeof(T)), nR - 1);
        return ld.finish(ld.read(((uint32_t)row * (uint32_t)nR + u) * (uint32_t)sizeof(T)));
    };
    const int cs0 = C.rp[c] + 2, cs1 = C.rp[c + 1], cp0 = C.cp[c] + kDP, cp1 = C.cp[c + 1];
    const bool longer = k.lng;
    const bool inner = !longer && k.po[3] == pad;   // at most 2 successors and 3 predecessors
    T y = T(0);
    if (inner) {
        for (int q = cs0; q < cs1; ++q) {
            T s = T(0);
#pragma unroll
            for (int a = 0; a < 2; ++a) s = fma_t(k.sw[a], X(C.ci[q], k.so[a]), s);
            y = fma_t(T(C.w[q]), s, y);
        }
        for (int q = cp0; q < cp1; ++q) {
            T s = T(0);
#pragma unroll
            for (int b = 0; b < 3; ++b) s = fma_t(k.pw[b], X(C.ri[q], k.po[b]), s);
            y = fma_t(T(C.w[C.eid[q]]), s, y);
        }
        return y;
    }
    const auto outer_s = [&](T w, int off) {
        T s = T(0);
        for (int q = cs0; q < cs1; ++q) s = fma_t(T(C.w[q]), X(C.ci[q], off), s);
        y = fma_t(w, s, y);
    };
    const auto outer_p = [&](T w, int off) {
        T s = T(0);
        for (int q = cp0; q < cp1; ++q) s = fma_t(T(C.w[C.eid[q]]), X(C.ri[q], off), s);
        y = fma_t(w, s, y);
    };
    constexpr int kEntry = kRows * (int)sizeof(T);
    if (cs0 < cs1) {
#pragma unroll
        for (int a = 0; a < 2; ++a) outer_s(k.sw[a], k.so[a]);
        if (longer)
            for (int e = R.rp[i] + 2; e < R.rp[i + 1]; ++e) outer_s(T(R.w[e]), R.ci[e] * kEntry);
    }
    if (cp0 < cp1) {
#pragma unroll
        for (int b = 0; b < kDP; ++b) outer_p(k.pw[b], k.po[b]);
        if (longer)
            for (int e = R.cp[i] + kDP; e < R.cp[i + 1]; ++e) outer_p(T(R.w[R.eid[e]]), R.ri[e] * kEntry);
    }
    return y;
}

template <typename T>
__device__ inline void put_quad(T* at, const Quad<T>& q) {
    if constexpr (sizeof(T) == 4) {
        const floatx4 v = {q.v[0], q.v[1], q.v[2], q.v[3]};
        *reinterpret_cast<floatx4*>(at) = v;
    } else {
        *reinterpret_cast<Quad<T>*>(at) = q;
    }
}

// One strip of out = M x by one wave, in both layouts; the sum of y^2 or, with
// a second factor (mul, times mul_inv), of y * that is left in *sum.
template <typename T, typename Load, typename Scales>
__device__ __forceinline__ void strip_apply(const AdjItem& item, const Slot<T>& S, const BwdJob& J, Load ld,
                                            const Scales& scales, T* out_x, T* out_n, const T* mul, T mul_inv,
                                            Quad<T>* P1, Quad<T>* P2, double* sum_at) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int nR = item.st.nR, nC = item.st.nC, nch = (nR + kWave - 1) / kWave, ldn = row_stride(nC);
    const int c0 = item.index * kRows, left = nC - c0;
    const StripTab<T>* tab = S.tabs() + item.index;
    const Cols<T> cols = S.cols(nR);
    const int flags = uni(tab->long_rows);
    const auto graph_b = [&] { return graph_of(J.set, J.pair_b[item.st.p]); };
    if (lane < 2) (lane ? P2 : P1)[col_stride(nR)] = Quad<T>{};
    stage(ld, [&] { scales(ld); }, nR, tab, P1, P2);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double sum = 0.0;
    const uint32_t rowb = (uint32_t)nR * (uint32_t)sizeof(T);
    for (int ch = 0; ch < nch; ++ch) {
        const int i = ch * kWave + lane;
        const uint32_t o = (uint32_t)c0 * rowb + (uint32_t)min(i, nR - 1) * (uint32_t)sizeof(T);
        T m[kRows] = {};
        if (mul) {
#pragma unroll
            for (int r = 0; r < kRows; ++r) m[r] = at_byte(mul, o + (r < left ? r : 0) * rowb);
        }
        const ColSlots<T, kDP> k = load_col<T, kDP>(cols, i);
        const Quad<T> y = gather_slots<T, kDP>(k, i, P1, P2, __ballot(k.lng) != 0, graph_b);
        if (i >= nR) continue;
        put_quad(out_n + (i * ldn + c0), y);  // past n_C: the row's padding
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            if (r >= left) break;
            *reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(out_x) + (o + r * rowb)) = y.v[r];
            if (!((flags >> r) & 1)) sum += (double)y.v[r] * (double)(mul ? T(m[r] * mul_inv) : y.v[r]);
        }
    }
    if (flags) {  // rows with longer lists: their other terms
        const GraphRef R = graph_b(), C = graph_of(J.set, J.pair_a[item.st.p]);
        const int pad = col_stride(nR) * kRows * (int)sizeof(T);
        for (int ch = 0; ch < nch; ++ch) {
            const int i = ch * kWave + lane;
            const ColSlots<T, kDP> k = load_col<T, kDP>(cols, i);
            for (int r = 0; r < kRows; ++r) {
                if (!((flags >> r) & 1) || i >= nR) continue;
                const int o = (c0 + r) * nR + i;
                const T v = out_x[o] + row_rest<T, Load>(ld, k, nR, pad, i, R, C, c0 + r);
                out_x[o] = v;
                out_n[i * ldn + c0 + r] = v;
                sum += (double)v * (double)(mul ? T(mul[o] * mul_inv) : v);
            }
        }
    }
    sum = wave_sum(sum);
    if (lane == 0) *sum_at = sum;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// ---------------------------------------------------------------- edge sums
// Partial sum w of eight takes the B edges f = w, w + 8, ... in order (one
// workgroup); an A edge's terms are w_f c(f, e), a B edge's w_e c(f, e) over
// the A edges, with c = Ybar[i][p] S[u][q] + S[i][p] Ybar[u][q] for f = (i, u),
// e = (p, q).  The waves form c for the next B edges, two at a time (lane l: A
// edges l + 64 ch, whose sum is that of the B edge), and leave it in LDS; then
// each thread adds its A edges' terms in the order of f.
//
// Bound by the latency of the reads: a pair's eight workgroups have eight B
// edges each in flight, where one wave per partial sum had two.
template <typename T>
struct EdgeRows {
    const T *g, *s1, *s0;   // G_{k+1}, S_{k+1}, S_k by rows of A nodes
    int ld, ld0;
    T a, inv1, inv0;
};
constexpr int kEdgeU = 2;                       // B edges a wave reads together
constexpr int kEdgeStep = kEdgeU * kNW;
template <typename T>
__host__ __device__ constexpr size_t edge_lds() {
    return (size_t)kEdgeStep * kAChunks * kWave * sizeof(T);
}
template <typename T, int NCH>
__device__ __forceinline__ void edge_sums(const EdgeRows<T>& E, const AdjPair& st, const Slot<T>& S,
                                          const GraphRef& A, const GraphRef& B, int w, T* cbuf) {
    constexpr int kBlock = kAChunks / NCH * kEdgeStep;   // B edges per barrier
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = uni(tid / kWave);
    const int* src_a = S.src();
    const int* src_b = src_a + A.nnz;
    uint32_t ep[NCH], eq[NCH];  // byte offsets in a row
    T ew[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int e = ch * kWave + lane;
        const bool has = e < st.kept_a;  // absent edges read entry 0 with weight 0
        ep[ch] = (has ? src_a[e] : 0) * (uint32_t)sizeof(T);
        eq[ch] = (has ? A.ci[e] : 0) * (uint32_t)sizeof(T);
        ew[ch] = has ? T(A.w[e]) : T(0);
    }
    const T *g = E.g, *s1 = E.s1, *s0 = E.s0;
    const int ld = E.ld * (int)sizeof(T), ld0 = E.ld0 * (int)sizeof(T);
    const T a = E.a, inv1 = E.inv1, inv0 = E.inv0;
    const int nf = (st.kept_b - w + kEdgeWaves - 1) / kEdgeWaves;
    constexpr int kOwn = (NCH * kWave + kNT - 1) / kNT;  // A edges of a thread
    T acc[kOwn];
#pragma unroll
    for (int z = 0; z < kOwn; ++z) acc[z] = T(0);
    for (int b0 = 0; b0 < nf; b0 += kWave) {             // 64 B edges' lists in the lanes
        const int m = min(kWave, nf - b0);
        const int f = w + kEdgeWaves * (b0 + lane);
        const bool has = lane < m;
        const int fi = has ? src_b[f] : 0, fu = has ? B.ci[f] : 0;
        const T fw = has ? T(B.w[f]) : T(0);
        double mine = 0.0;
        for (int c0 = 0; c0 < m; c0 += kBlock) {
            const int mb = min(kBlock, m - c0);
            __syncthreads();  // the block before has been added
            for (int q0 = wave * kEdgeU; q0 < mb; q0 += kEdgeStep) {
                T gi[kEdgeU][NCH], hi[kEdgeU][NCH], si[kEdgeU][NCH], gu[kEdgeU][NCH], hu[kEdgeU][NCH], su[kEdgeU][NCH];
#pragma unroll
                for (int z = 0; z < kEdgeU; ++z) {
                    const int l = c0 + min(q0 + z, mb - 1);
                    const int i = lane_value(fi, l), u = lane_value(fu, l);
#pragma unroll
                    for (int ch = 0; ch < NCH; ++ch) {
                        gi[z][ch] = at_byte(g, (uint32_t)(i * ld) + ep[ch]);
                        hi[z][ch] = at_byte(s1, (uint32_t)(i * ld) + ep[ch]);
                        si[z][ch] = at_byte(s0, (uint32_t)(i * ld0) + ep[ch]);
                        gu[z][ch] = at_byte(g, (uint32_t)(u * ld) + eq[ch]);
                        hu[z][ch] = at_byte(s1, (uint32_t)(u * ld) + eq[ch]);
                        su[z][ch] = at_byte(s0, (uint32_t)(u * ld0) + eq[ch]);
                    }
                }
#pragma unroll
                for (int z = 0; z < kEdgeU; ++z) {
                    if (q0 + z >= mb) break;
                    T pb = T(0);
#pragma unroll
                    for (int ch = 0; ch < NCH; ++ch) {
                        const T yi = fma_t(-a, hi[z][ch] * inv1, gi[z][ch]) * inv1;
                        const T yu = fma_t(-a, hu[z][ch] * inv1, gu[z][ch]) * inv1;
                        const T c = fma_t(yi, su[z][ch] * inv0, (si[z][ch] * inv0) * yu);
                        cbuf[((q0 + z) * NCH + ch) * kWave + lane] = c;
                        pb = fma_t(ew[ch], c, pb);
                    }
                    const double sb = wave_sum((double)pb);
                    if (lane == c0 + q0 + z) mine = sb;
                }
            }
            __syncthreads();
            for (int q = 0; q < mb; ++q) {
                const T wf = lane_value(fw, c0 + q);
#pragma unroll
                for (int z = 0; z < kOwn; ++z) {
                    const int e = z * kNT + tid;
                    if (e < NCH * kWave) acc[z] = fma_t(wf, cbuf[q * (NCH * kWave) + e], acc[z]);
                }
            }
        }
        // the wave's own B edges: c0 + q0 + z with q0 / kEdgeU = wave mod kNW
        if (has && ((lane % kBlock) / kEdgeU) % kNW == wave) S.grad_b()[f] += mine;
    }
    double* ga = S.grad_a() + w * (kAChunks * kWave);
#pragma unroll
    for (int z = 0; z < kOwn; ++z) {
        const int e = z * kNT + tid;
        if (e < NCH * kWave) ga[e] += (double)acc[z];
    }
}

// ---------------------------------------------------------------- the launches
// A segment of a pair, counted from its last: [k0, k0 + len).
struct Segment {
    int k0, len, index;
};
__device__ inline Segment segment(const AdjPair& st, int ckpt, int back) {
    Segment s;
    s.index = st.s_last - back;
    s.k0 = s.index * ckpt;
    s.len = back < 0 || s.index < 0 ? 0 : min(ckpt, st.K - s.k0);
    return s;
}

// Launch j of round t (the n-th launch of the call): the edge sums of the
// step back, one workgroup each, then the strips, one wave each.
template <typename T>
__global__ __launch_bounds__(kNT, 4) void adj_step(AdjJob A, int t, int j, int n, int wave_lds) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = uni((int)threadIdx.x / kWave);
    const int x = blockIdx.x & (kXcds - 1), wg = blockIdx.x / kXcds, wgs = gridDim.x / kXcds;
    const int mid = A.item_off[2 * x + 1], end = A.item_off[2 * x + 2];
    const int fpar = t & 1, rpar = fpar ^ 1;
    for (int q = A.item_off[2 * x] + wg; q < mid; q += wgs) {
        const AdjItem item = A.items[q];
        const AdjPair st = item.st;
        const Segment rseg = segment(st, A.J.ckpt, t - 1);
        const int s1 = rseg.len - j, s0 = s1 - 1, k = rseg.k0 + s0;
        if (s0 < 0) continue;
        const Slot<T> S = slot_of<T>(A, item.slot);
        const int gp = (st.K - 1 - k) & 1;  // G_{k+1}
        const double dots = part_read(S.dot((n - 1) & 1), st.strips);
        const GraphRef ga = graph_of(A.J.set, A.J.pair_a[st.p]), gb = graph_of(A.J.set, A.J.pair_b[st.p]);
        EdgeRows<T> E;
        E.g = S.g_n(gp);
        E.s1 = S.seg_n(rpar, s1);
        E.ld = row_stride(st.nC);
        if (s0 != 0) {
            E.s0 = S.seg_n(rpar, s0);
            E.ld0 = E.ld;
        } else {
            E.ld0 = st.nC;
            E.s0 = rseg.index == 0 ? S.start_n()
                                  : reinterpret_cast<const T*>(A.J.fck) + A.J.fck_off[st.p] +
                                        (long long)(rseg.index - 1) * st.nR * st.nC;
        }
        E.a = T(uni(wave_sum(dots)));
        E.inv1 = *S.inv(rpar, s1);
        E.inv0 = s0 == 0 ? T(1) : *S.inv(rpar, s0);
        T* cbuf = reinterpret_cast<T*>(smem);
        switch ((st.kept_a + kWave - 1) / kWave) {
            case 1: edge_sums<T, 1>(E, st, S, ga, gb, item.index, cbuf); break;
            case 2: edge_sums<T, 2>(E, st, S, ga, gb, item.index, cbuf); break;
            case 3: edge_sums<T, 3>(E, st, S, ga, gb, item.index, cbuf); break;
            case 4: edge_sums<T, 4>(E, st, S, ga, gb, item.index, cbuf); break;
            case 5: edge_sums<T, 5>(E, st, S, ga, gb, item.index, cbuf); break;
            case 6: edge_sums<T, 6>(E, st, S, ga, gb, item.index, cbuf); break;
            case 7: edge_sums<T, 7>(E, st, S, ga, gb, item.index, cbuf); break;
            case 8: edge_sums<T, 8>(E, st, S, ga, gb, item.index, cbuf); break;
            default: break;  // no A edge: no dependence on the weights
        }
    }
    __syncthreads();
    // the strips back, then the strips forward
    const int strips = end - mid, waves = wgs * kNW;
    Quad<T>* P1 = reinterpret_cast<Quad<T>*>(smem + (size_t)wave * wave_lds);
    for (int q = wg * kNW + wave; q < 2 * strips; q += waves) {
        const AdjItem item = A.items[mid + (q < strips ? q : q - strips)];
        const AdjPair st = item.st;
        const Slot<T> S = slot_of<T>(A, item.slot);
        Quad<T>* P2 = P1 + col_stride(st.nR) + 1;
        if (q < strips) {
            const Segment rseg = segment(st, A.J.ckpt, t - 1);
            const int s1 = rseg.len - j, s0 = s1 - 1, k = rseg.k0 + s0;
            if (s0 < 0 || k == 0) continue;  // no update before the first
            const int gp = (st.K - 1 - k) & 1;
            const double dots = part_read(S.dot((n - 1) & 1), st.strips);
            const Ybar<T> ld{S.g_x(gp), S.seg_x(rpar, s1), T(0), *S.inv(rpar, s1)};
            strip_apply<T>(item, S, A.J, ld, [&](Ybar<T>& l) { l.a = T(uni(wave_sum(dots))); }, S.g_x(gp ^ 1),
                           S.g_n(gp ^ 1), s0 == 0 ? S.first_x((t - 1) % 3) : S.seg_x(rpar, s0),
                           s0 == 0 ? T(1) : *S.inv(rpar, s0), P1, P2, S.dot(n & 1) + item.index);
        } else {
            const Segment fseg = segment(st, A.J.ckpt, t);
            if (j >= fseg.len) continue;
            const double nu = j ? part_read(S.nu(fpar, j), st.strips) : 0.0;
            const Scaled<T> ld{j == 0 ? S.first_x(t % 3) : S.seg_x(fpar, j), T(1)};
            const auto scales = [&](Scaled<T>& l) {
                if (j == 0) return;
                l.inv = inv_of<T>(nu);
                if (item.index == 0 && (threadIdx.x & (kWave - 1)) == 0) *S.inv(fpar, j) = l.inv;
            };
            strip_apply<T>(item, S, A.J, ld, scales, S.seg_x(fpar, j + 1), S.seg_n(fpar, j + 1), (const T*)nullptr,
                           T(1), P1, P2, S.nu(fpar, j + 1) + item.index);
        }
    }
}


// After round t (t = -1: before the first).
template <typename T>
__global__ __launch_bounds__(kNT) void adj_seam(AdjJob A, int t, int n) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = uni((int)threadIdx.x / kWave);
    const int x = blockIdx.x & (kXcds - 1), wg = blockIdx.x / kXcds, waves = gridDim.x / kXcds * kNW;
    const int end = A.item_off[2 * x + 2];
    for (int q = A.item_off[2 * x + 1] + wg * kNW + wave; q < end; q += waves) {
        const AdjItem item = A.items[q];
        const AdjPair st = item.st;
        const Slot<T> S = slot_of<T>(A, item.slot);
        const int c0 = item.index * kRows, rows = min(kRows, st.nC - c0);
        const Segment done = segment(st, A.J.ckpt, t), next = segment(st, A.J.ckpt, t + 1);
        if (done.len > 0) {
            const T inv = inv_of<T>(part_read(S.nu(t & 1, done.len), st.strips));
            if (item.index == 0 && lane == 0) *S.inv(t & 1, done.len) = inv;
            const T* y = S.seg_x(t & 1, done.len) + c0 * st.nR;
            const T* g = S.g_x((st.K - done.k0 - done.len) & 1) + c0 * st.nR;
            double dot = 0.0;
            for (int o = lane; o < rows * st.nR; o += kWave) dot += (double)(T)(y[o] * inv) * (double)g[o];
            dot = wave_sum(dot);
            if (lane == 0) S.dot(n & 1)[item.index] = dot;
        }
        if (next.len > 0) {
            T* out = S.first_x((t + 1) % 3) + c0 * st.nR;
            const T* in = next.index == 0 ? S.start_n()
                                          : reinterpret_cast<const T*>(A.J.fck) + A.J.fck_off[st.p] +
                                                (long long)(next.index - 1) * st.nR * st.nC;
            for (int i = lane; i < st.nR; i += kWave)
                for (int r = 0; r < rows; ++r) out[r * st.nR + i] = in[i * st.nC + c0 + r];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kNT) void adj_finish(AdjJob A) {
    const AdjPair st = A.pairs[blockIdx.x];
    if (!st.active) return;
    const Slot<T> S = slot_of<T>(A, blockIdx.x);
    double* out_a = A.J.grad_w + A.J.set.edge_off[A.J.pair_a[st.p]];
    double* out_b = A.J.grad_w + A.J.set.edge_off[A.J.pair_b[st.p]];
    for (int e = threadIdx.x; e < st.kept_a; e += kNT) {
        double g = 0.0;
        for (int w = 0; w < kEdgeWaves; ++w) g += S.grad_a()[w * (kAChunks * kWave) + e];
        atomicAdd(out_a + e, g);
    }
    for (int f = threadIdx.x; f < st.kept_b; f += kNT) atomicAdd(out_b + f, S.grad_b()[f]);
}

template <typename T>
int run(const BwdJob& J, int max_nodes, int num_cus, hipStream_t stream) {
    AdjJob A;
    A.J = J;
    A.L = layout_of<T>(max_nodes, J.slot_elems, J.ckpt);
    A.np = J.n_pairs;
    unsigned char* at = static_cast<unsigned char*>(J.ws);
    A.slots = at + header_bytes(A.np, A.L.max_strips);
    A.item_off = reinterpret_cast<int*>(at);
    at += up((2 * kXcds + 1) * 4);
    A.pairs = reinterpret_cast<AdjPair*>(at);
    at += up((size_t)A.np * sizeof(AdjPair));
    A.items = reinterpret_cast<AdjItem*>(at);
    const size_t strip = strip_lds<T>(max_nodes), lds = strip * kNW > edge_lds<T>() ? strip * kNW : edge_lds<T>();
    int e = (int)hipFuncSetAttribute(reinterpret_cast<const void*>(&adj_step<T>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != 0) return e;
    hipLaunchKernelGGL(adj_init<T>, dim3(8, A.np), dim3(kNT), 0, stream, A);
    if ((e = (int)hipGetLastError()) != 0) return e;
    hipLaunchKernelGGL(adj_items, dim3(1), dim3(kMaxPairs), 0, stream, A);
    if ((e = (int)hipGetLastError()) != 0) return e;
    // workgroups for a call whose items all lie on one XCD, as many as stay resident
    const size_t items = kXcds * group_items(A.np, A.L.max_strips), most = (size_t)num_cus * 12 / kXcds * kXcds;
    const dim3 grid((unsigned)(items < most ? items : most));
    const int rounds = (J.max_iter + J.ckpt - 1) / J.ckpt;
    int n = 0;
    for (int t = -1; t <= rounds; ++t) {
        for (int j = 0; t >= 0 && j < J.ckpt; ++j) {
            hipLaunchKernelGGL(adj_step<T>, grid, dim3(kNT), lds, stream, A, t, j, n++, (int)strip);
            if ((e = (int)hipGetLastError()) != 0) return e;
        }
        if (t == rounds) break;
        hipLaunchKernelGGL(adj_seam<T>, grid, dim3(kNT), 0, stream, A, t, n++);
        if ((e = (int)hipGetLastError()) != 0) return e;
    }
    hipLaunchKernelGGL(adj_finish<T>, dim3(A.np), dim3(kNT), 0, stream, A);
    return (int)hipGetLastError();
}

}  // namespace

size_t bwd_strips_bytes(int max_nodes, long long n_pairs, int ckpt, int esize) {
    const long long elems = (long long)max_nodes * max_nodes;
    const AdjLayout l = esize == 8 ? layout_of<double>(max_nodes, elems, ckpt) : layout_of<float>(max_nodes, elems, ckpt);
    return header_bytes((int)n_pairs, l.max_strips) + (size_t)n_pairs * l.total;
}

int launch_bwd_strips(int dtype, const BwdJob& J, int max_nodes, int num_cus, hipStream_t stream) {
    return dtype == CFSIM_F64 ? run<double>(J, max_nodes, num_cus, stream) : run<float>(J, max_nodes, num_cus, stream);
}

}  // namespace cfsim

// Calls that have the forward's checkpoints run on strips
//   - up to one pair per CU (the one-workgroup kernel then leaves CUs idle or
//     waits for its largest pair), in FP64 up to one per two CUs, of 32 nodes or
//     more.  Backward of 200 updates, one workgroup per pair against strips (ms):
//     FP32, 2 pairs of 250-256 nodes 54.5 / 6.2; 160 of 16-256 paired by size 82.2 / 19.4; 100 of
//     90-128 17.3 / 6.5, 250 of them 22.7 / 13.2; 100 of 60-64 7.7 / 3.5, 250
//     8.6 / 6.2; 64 of 8-48 3.3 / 2.0; but 512 of 120-128 31.8 / 35.2, 512 of
//     8-64 5.9 / 6.4 and one of 12 x 16 1.2 / 1.6.  FP64, 100 of 90-128 22.5 /
//     12.5, 100 of 60-64 8.7 / 5.9, 64 of 8-48 3.6 / 3.3, but 250 of 90-128 29.9 /
//     32.3 and of 60-64 10.2 / 12.8.
//   - of small graphs fewer pairs, 2.2 (n - 28) in FP64 and 5 (n - 24) in FP32
//     sets of nearly straight code: a strip's cost does not shrink with its columns,
//     and one workgroup holds such a pair's update in few instructions.  Time of one
//     workgroup over that of strips, backward of 100 updates: FP64, 20 pairs of 27-33
//     nodes 0.89-1.01, 48 of 34-40 0.89-1.00 and 128 of them 0.63-0.71, 48 of 42-48
//     0.94-1.03, 90 of 58-64 1.01-1.08, 128 of 74-80 0.85-0.96, of 90-96 1.01-1.15;
//     FP32 chains, 128 of 34-40 0.90 and 190 of them 0.82, 128 of 42-48 1.00, 190 of
//     58-64 0.96; with 1.35 jumps per node 190 of 34-48 0.99-1.00.
//   - where the set's largest pairs are strips' pairs: else the one-workgroup
//     kernel, which takes those after the strips, sets the time alone (FP64, 160
//     pairs of 16-256: 163 / 203).
//   - where the updates to expect pay for the launches, 4.2 us each and as many
//     as max_iter asks for whenever the pairs stopped, against a saving that
//     grows with the pair, about n^2 / 400 us per update (FP64 n^2 / 1000; FP32
//     3 to 7 us for 40-48 nodes, 10-22 for 64, 47-55 for 128, 240 for 256; FP64 2
//     for 40-48, 10-15 for 64, 48 for 128): two FP32 pairs of 250-256 nodes that
//     stopped after two updates of max_iter 2000 take 0.7 ms in one workgroup each
//     and 8.9 on strips.
extern "C" int cfsim_route_backward_strips(const cfsim_graph_set* set, int64_t n_pairs, const cfsim_options* opt,
                                           int32_t checkpoint_every, int32_t num_cus) {
    using namespace cfsim;
    const bool f64 = opt->dtype == CFSIM_F64;
    const int n = set->max_nodes;
    if (n < 32 || n > kBwdStripNodes) return 0;
    if (n_pairs < 1 || n_pairs > (f64 ? num_cus / 2 : num_cus) || n_pairs > kMaxPairs) return 0;
    const int nnz = mean_jumps(set, n);
    if (f64 ? 5 * n_pairs > 11 * (n - 28) : 4 * nnz < 5 * n && n_pairs > 5 * (n - 24)) return 0;
    const BwdShape s = bwd_shape(n, n, nnz, nnz, nnz, f64 ? 8 : 4);
    if (!s.fits || !s.lane_edges) return 0;
    const double every = checkpoint_every < opt->max_iter ? checkpoint_every : opt->max_iter;
    const double launches = (ceil(opt->max_iter / every) + 1.0) * (every + 1.0) + 5.0;
    return 4.2 * launches <= updates_expected(opt) * (n * (double)n / (f64 ? 1000.0 : 400.0) + 4.2 * (1.0 + 1.0 / every));
}
