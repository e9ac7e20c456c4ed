// The update Y = B S A^T + B^T S A on strips of four rows of X = S^T, for
// iterates in global memory (one workgroup per strip and launch).
//
// X has a row per node c of the C graph and a column per node i of the R
// graph.  An entry of the update is
//   Y[i][c] = sum_{u in succ(i)} w_iu P1[u] + sum_{u in pred(i)} w_ui P2[u],
//   P1[u] = sum_{v in succ(c)} w_cv X[v][u],  P2[u] = sum_{v in pred(c)} w_vc X[v][u].
// Stage A forms P1 and P2 of the strip's four rows: their source rows are
// merged into one list (a strip's rows are consecutive nodes, which share
// most neighbours), each read once, coalesced, and added to all four rows by
// a matrix instruction (FP32: v_mfma_f32_4x4x1, an outer product of the four
// weights with 64 columns; its terms round like fma, and a weight of zero
// leaves a row unchanged).  Stage B gathers every column's neighbours from P1
// and P2 in LDS, four rows per 16-byte read, at addresses from lists that are
// laid out per column.  Nothing is gathered from global memory.  The terms of
// an entry are added in the order of the gathers from S (inner over C's list,
// outer over R's list), so the bits are the same.
#pragma once

#include "pair_device.h"

namespace cfsim {
namespace strips {

constexpr int kRows = 4;           // rows of X per strip
constexpr int kThreads = 512;      // workgroup of a strip
constexpr int kWaves = kThreads / kWave;
constexpr int kSrcS = 8;           // merged successor sources of a strip (4 rows, at most 2 each)
constexpr int kSrcP = 16;          // merged predecessor sources (4 rows, at most 4 each)

// Sources of one strip: byte offsets of rows of X and the four rows' weights
// of each.
template <typename T>
struct alignas(16) StripTab {
    T ws[kSrcS][kRows];
    T wp[kSrcP][kRows];
    int src_s[kSrcS], src_p[kSrcP];
    int ns, np;                    // sources
    int long_rows;                 // bit r: row r has list entries past the slots
    int pad;
};

// Lists of the columns (R nodes), one array per slot of `stride` entries:
// byte offsets of the neighbours in P1 / P2 and weights; absent slots point at
// the zero entry behind the last column, with weight 0.  Bit 0 of the first
// successor's offset: the column's lists are longer than the slots.
template <typename T>
struct Cols {
    const int* so;   // [2][stride]
    const int* po;   // [4][stride]
    const T* sw;
    const T* pw;
    int stride;
};

__host__ __device__ inline int col_stride(int nR) { return (nR + kWave - 1) / kWave * kWave; }
template <typename T>
__host__ __device__ inline size_t cols_bytes(int nR, int dp) {
    return (size_t)col_stride(nR) * (2 + dp) * (sizeof(int) + sizeof(T));
}
template <typename T>
__device__ inline Cols<T> carve_cols(unsigned char* base, int nR, int dp) {
    Cols<T> c;
    c.stride = col_stride(nR);
    c.sw = reinterpret_cast<const T*>(base);
    c.pw = c.sw + 2 * (size_t)c.stride;
    c.so = reinterpret_cast<const int*>(c.pw + (size_t)dp * c.stride);
    c.po = c.so + 2 * (size_t)c.stride;
    return c;
}
// LDS of a strip: P1 and P2, four values per column and the zero entry.
template <typename T>
__host__ __device__ inline size_t strip_lds(int nR) {
    return 2 * (size_t)(col_stride(nR) + 1) * kRows * sizeof(T);
}

// Column i's slots (DP predecessor slots).
template <typename T, int DP>
__device__ inline void build_col(const GraphRef& R, int i, Cols<T> c) {
    const bool has = i < R.n;
    const int sb = has ? R.rp[i] : 0, ns = has ? R.rp[i + 1] - sb : 0;
    const int pb = has ? R.cp[i] : 0, np = has ? R.cp[i + 1] - pb : 0;
    constexpr int vb = kRows * (int)sizeof(T);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const_cast<int*>(c.so)[q * c.stride + i] =
            (q < ns ? R.ci[sb + q] : c.stride) * vb + (q == 0 && (ns > 2 || np > DP) ? 1 : 0);
        const_cast<T*>(c.sw)[q * c.stride + i] = q < ns ? T(R.w[sb + q]) : T(0);
    }
#pragma unroll
    for (int q = 0; q < DP; ++q) {
        const_cast<int*>(c.po)[q * c.stride + i] = (q < np ? R.ri[pb + q] : c.stride) * vb;
        const_cast<T*>(c.pw)[q * c.stride + i] = q < np ? T(R.w[R.eid[pb + q]]) : T(0);
    }
}

// Merges the first `slots` list entries of rows c0 .. c0 + 3 (val(r, q) gives
// entry q of row r: node and weight; len(r) its length) into sources: at each
// step the smallest node at the head of any row, taken by every row that has
// it there, so that every row's entries keep their order.
template <typename T, int MAX, typename Len, typename Val>
__device__ inline int merge_sources(int slots, Len len, Val val, int* src, T (*w)[kRows]) {
    int head[kRows] = {0, 0, 0, 0};
    int n = 0;
    for (; n < MAX; ++n) {
        int v = INT_MAX;
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            if (head[r] < min(len(r), slots)) {
                T x;
                v = min(v, val(r, head[r], x));
            }
        if (v == INT_MAX) break;
        src[n] = v;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            T x = T(0);
            bool take = false;
            if (head[r] < min(len(r), slots)) take = val(r, head[r], x) == v;
            w[n][r] = take ? x : T(0);
            head[r] += take ? 1 : 0;
        }
    }
    for (int q = n; q < MAX; ++q) {  // padding: a source that is read anyway, weight 0
        src[q] = n > 0 ? src[0] : 0;
#pragma unroll
        for (int r = 0; r < kRows; ++r) w[q][r] = T(0);
    }
    return n;
}

// The table of the strip that starts at row c0 (one thread; X's row stride
// is nR, its bytes fit 31 bits).
template <typename T, int DP>
__device__ inline void build_strip(const GraphRef& C, int c0, int nR, StripTab<T>* t) {
    auto row = [&](int r) { return c0 + r < C.n ? c0 + r : -1; };
    t->ns = merge_sources<T, kSrcS>(
        2, [&](int r) { return row(r) < 0 ? 0 : C.rp[row(r) + 1] - C.rp[row(r)]; },
        [&](int r, int q, T& w) {
            const int e = C.rp[row(r)] + q;
            w = T(C.w[e]);
            return C.ci[e];
        },
        t->src_s, t->ws);
    t->np = merge_sources<T, kSrcP>(
        DP, [&](int r) { return row(r) < 0 ? 0 : C.cp[row(r) + 1] - C.cp[row(r)]; },
        [&](int r, int q, T& w) {
            const int e = C.cp[row(r)] + q;
            w = T(C.w[C.eid[e]]);
            return C.ri[e];
        },
        t->src_p, t->wp);
    int lng = 0;
    for (int r = 0; r < kRows; ++r)
        if (row(r) >= 0 &&
            (C.rp[row(r) + 1] - C.rp[row(r)] > 2 || C.cp[row(r) + 1] - C.cp[row(r)] > DP))
            lng |= 1 << r;
    t->long_rows = lng;
    for (int q = 0; q < kSrcS; ++q) t->src_s[q] *= nR * (int)sizeof(T);
    for (int q = 0; q < kSrcP; ++q) t->src_p[q] *= nR * (int)sizeof(T);
}

// Entry at a byte offset of an iterate.
template <typename T>
__device__ __forceinline__ T at_byte(const T* X, uint32_t off) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(X) + off);
}

template <typename T>
struct Quad {
    T v[kRows];
};
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Stage A by one wave: P1 and P2 of the strip (X: row stride nR) for the chunks
// of 64 columns ch0, ch0 + step, ....  The whole wave takes part in every source
// (the matrix instruction reads all lanes): lanes past the last column read the
// last one.  FP32: one register holds the weights of 16 sources (lane 4 q + r), of which the matrix instruction broadcasts the
// block it needs (cbsz = 4, abid = the source).
template <int Q>
__device__ __forceinline__ void add_block(floatx4& acc, float w, float x) {
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(w, x, acc, 4, Q, 0);
}
template <int W>
__device__ __forceinline__ void add_blocks(floatx4& acc, float w, const float (&x)[4]) {
    add_block<W>(acc, w, x[0]);
    add_block<W + 1>(acc, w, x[1]);
    add_block<W + 2>(acc, w, x[2]);
    add_block<W + 3>(acc, w, x[3]);
}
__device__ __forceinline__ void wave_sources(const float* X, int nR, const StripTab<float>* t, Quad<float>* P1,
                                             Quad<float>* P2, int ch0 = 0, int step = 1) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const float* wt = &t->ws[0][0];  // ws and wp lie one behind the other
    const float w = wt[lane], w2 = wt[64 + (lane & 31)];
    const int src = t->src_s[lane < 24 ? lane : 0];  // src_s and src_p too
    const int ns = dev::uni(t->ns), np = dev::uni(t->np);
    const int nch = (nR + kWave - 1) / kWave;
    for (int ch = ch0; ch < nch; ch += step) {
        const int col = ch * kWave + lane;
        const uint32_t at = (uint32_t)min(col, nR - 1) * 4u;
        float x[6][4];
        auto read = [&](int g, int q0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) x[g][q] = at_byte(X, (uint32_t)dev::lane_value(src, q0 + q) + at);
        };
        read(0, 0);
        read(2, 8);
        if (ns > 4) read(1, 4);
        if (np > 4) read(3, 12);
        floatx4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = {0.0f, 0.0f, 0.0f, 0.0f};
        add_blocks<0>(a, w, x[0]);
        add_blocks<8>(b, w, x[2]);
        if (ns > 4) add_blocks<4>(a, w, x[1]);
        if (np > 4) add_blocks<12>(b, w, x[3]);
        if (np > 8) {
            read(4, 16);
            add_blocks<0>(b, w2, x[4]);
        }
        if (np > 12) {
            read(5, 20);
            add_blocks<4>(b, w2, x[5]);
        }
        *reinterpret_cast<floatx4*>(&P1[col]) = a;
        *reinterpret_cast<floatx4*>(&P2[col]) = b;
    }
}
__device__ __forceinline__ void wave_sources(const double* X, int nR, const StripTab<double>* t, Quad<double>* P1,
                                             Quad<double>* P2, int ch0 = 0, int step = 1) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int src = t->src_s[lane < 24 ? lane : 0];  // src_s and src_p lie one behind the other
    const int ns = dev::uni(t->ns), np = dev::uni(t->np);
    const int nch = (nR + kWave - 1) / kWave;
    for (int ch = ch0; ch < nch; ch += step) {
        const int col = ch * kWave + lane;
        const uint32_t at = (uint32_t)min(col, nR - 1) * 8u;
        double x[4][4];
        auto read = [&](int g, int q0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) x[g][q] = at_byte(X, (uint32_t)dev::lane_value(src, q0 + q) + at);
        };
        Quad<double> a{}, b{};
        auto add = [&](Quad<double>& acc, int g, const double (*w)[kRows]) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < kRows; ++r) acc.v[r] = dev::fma_t(w[q][r], x[g][q], acc.v[r]);
        };
        read(0, 0);
        read(2, 8);
        if (ns > 4) read(1, 4);
        if (np > 4) read(3, 12);
        add(a, 0, t->ws);
        add(b, 2, t->wp);
        if (ns > 4) add(a, 1, t->ws + 4);
        if (np > 4) add(b, 3, t->wp + 4);
        for (int q = 8; q < np; q += 4) {
#pragma unroll
            for (int z = 0; z < 4; ++z) x[0][z] = at_byte(X, (uint32_t)dev::uni(t->src_p[q + z]) + at);
            add(b, 0, t->wp + q);
        }
        P1[col] = a;
        P2[col] = b;
    }
}

template <typename T>
__device__ __forceinline__ const Quad<T>& quad_at(const Quad<T>* P, int off) {
    return *reinterpret_cast<const Quad<T>*>(reinterpret_cast<const unsigned char*>(P) + off);
}

// Terms of a row c of C whose lists are longer than the slots (2 successors,
// 4 predecessors), for column i, as the pair kernels add them: for a node i
// within 2 successors and 3 predecessors the sum over i's slots inside the
// sum over the rest of c's lists, else the other way round.
// X(row, column) reads the iterate.
template <typename T, typename At>
__device__ inline T long_row_terms(At X, const GraphRef& R, const GraphRef& C, int i, int c) {
    const int sb = R.rp[i], ns = R.rp[i + 1] - sb, pb = R.cp[i], np = R.cp[i + 1] - pb;
    const int cs0 = C.rp[c] + 2, cs1 = C.rp[c + 1], cp0 = C.cp[c] + 4, cp1 = C.cp[c + 1];
    T y = T(0);
    if (ns <= 2 && np <= 3) {
        for (int q = cs0; q < cs1; ++q) {
            const int row = C.ci[q];
            T s = T(0);
            for (int a = 0; a < ns; ++a) s = dev::fma_t(T(R.w[sb + a]), X(row, R.ci[sb + a]), s);
            y = dev::fma_t(T(C.w[q]), s, y);
        }
        for (int q = cp0; q < cp1; ++q) {
            const int row = C.ri[q];
            T s = T(0);
            for (int b = 0; b < np; ++b) s = dev::fma_t(T(R.w[R.eid[pb + b]]), X(row, R.ri[pb + b]), s);
            y = dev::fma_t(T(C.w[C.eid[q]]), s, y);
        }
    } else {
        for (int a = 0; a < ns; ++a) {
            T s = T(0);
            for (int q = cs0; q < cs1; ++q) s = dev::fma_t(T(C.w[q]), X(C.ci[q], R.ci[sb + a]), s);
            y = dev::fma_t(T(R.w[sb + a]), s, y);
        }
        for (int b = 0; b < np; ++b) {
            T s = T(0);
            for (int q = cp0; q < cp1; ++q) s = dev::fma_t(T(C.w[C.eid[q]]), X(C.ri[q], R.ri[pb + b]), s);
            y = dev::fma_t(T(R.w[R.eid[pb + b]]), s, y);
        }
    }
    return y;
}

// Out of line, for the pair kernel that is at its register budget (there the
// pass below, whose body needs more registers, is slower: 21.8 against 18.0 ms
// for the query of 3,000 graphs).
template <typename T>
__device__ __noinline__ T long_row_call(const T* X, int nR, const GraphRef& R, const GraphRef& C, int i, int c) {
    return long_row_terms<T>([=](int v, int u) { return X[(long long)v * nR + u]; }, R, C, i, c);
}

// One column's slots.
template <typename T, int DP>
struct ColSlots {
    int so[2], po[DP];
    T sw[2], pw[DP];
    bool lng;   // longer lists
};
template <typename T, int DP>
__device__ __forceinline__ ColSlots<T, DP> load_col(const Cols<T>& c, int i) {
    ColSlots<T, DP> k;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        k.so[q] = c.so[q * c.stride + i];
        k.sw[q] = c.sw[q * c.stride + i];
    }
    k.lng = (k.so[0] & 1) != 0;
    k.so[0] &= ~1;
#pragma unroll
    for (int q = 0; q < DP; ++q) {
        k.po[q] = c.po[q * c.stride + i];
        k.pw[q] = c.pw[q * c.stride + i];
    }
    return k;
}

// Stage B for one column (DP predecessor slots): the terms of its slots and,
// when `rest` (some lane's lists are longer), those of longer lists, in list
// order, successors before predecessors; graph() is the R graph.
template <typename T, int DP, typename Graph>
__device__ __forceinline__ Quad<T> gather_slots(const ColSlots<T, DP>& k, int i, const Quad<T>* P1,
                                                const Quad<T>* P2, bool rest, const Graph& graph) {
    Quad<T> y;
    {
        const Quad<T> g = quad_at(P1, k.so[0]);
#pragma unroll
        for (int r = 0; r < kRows; ++r) y.v[r] = k.sw[0] * g.v[r];
    }
    {
        const Quad<T> g = quad_at(P1, k.so[1]);
#pragma unroll
        for (int r = 0; r < kRows; ++r) y.v[r] = dev::fma_t(k.sw[1], g.v[r], y.v[r]);
    }
    if (rest) {
        const GraphRef R = graph();
        if (i < R.n)
            for (int e = R.rp[i] + 2; e < R.rp[i + 1]; ++e) {
                const Quad<T> g = P1[R.ci[e]];
                const T w = T(R.w[e]);
#pragma unroll
                for (int r = 0; r < kRows; ++r) y.v[r] = dev::fma_t(w, g.v[r], y.v[r]);
            }
    }
#pragma unroll
    for (int q = 0; q < DP; ++q) {
        const Quad<T> g = quad_at(P2, k.po[q]);
#pragma unroll
        for (int r = 0; r < kRows; ++r) y.v[r] = dev::fma_t(k.pw[q], g.v[r], y.v[r]);
    }
    if (rest) {
        const GraphRef R = graph();
        if (i < R.n)
            for (int e = R.cp[i] + DP; e < R.cp[i + 1]; ++e) {
                const Quad<T> g = P2[R.ri[e]];
                const T w = T(R.w[R.eid[e]]);
#pragma unroll
                for (int r = 0; r < kRows; ++r) y.v[r] = dev::fma_t(w, g.v[r], y.v[r]);
            }
    }
    return y;
}
template <typename T, int DP>
__device__ __forceinline__ Quad<T> gather_col(const Cols<T>& c, int i, const Quad<T>* P1, const Quad<T>* P2,
                                              bool rest, const GraphRef& R) {
    return gather_slots<T, DP>(load_col<T, DP>(c, i), i, P1, P2, rest, [&] { return R; });
}

// The rows of a strip whose lists are longer than the slots, by the pair
// kernels' rules: all of the row, from P1 and P2, X_{k-1} (Xc) and X_{k-2}
// (Xo).  Out of line and after the other rows, so that the loop
// over the columns holds no call.  Columns of chunks ch0, ch0 + step, ...;
// returns nu^2 and the even-step sums.
struct RowSums {
    double nu2, dy2, dyy;
};
template <typename T, int DP>
__device__ __noinline__ RowSums long_rows_pass(const T* Xc, T* Xn, const T* Xo, int nR, int nC, int c0, int long_rows,
                                               unsigned char* cols_at, const Quad<T>* P1, const Quad<T>* P2,
                                               GraphRef R, GraphRef C, T sigma, int even, int ch0, int step) {
    RowSums s{0.0, 0.0, 0.0};
    const Cols<T> cols = carve_cols<T>(cols_at, nR, DP);
    const int lane = (int)(threadIdx.x & (kWave - 1));
    for (int ch = ch0; ch * kWave < nR; ch += step) {
        const int i = ch * kWave + lane;
        if (i >= nR) continue;
        const Quad<T> y = gather_col<T, DP>(cols, i, P1, P2, true, R);
        for (int r = 0; r < kRows; ++r) {
            if (!((long_rows >> r) & 1) || c0 + r >= nC) continue;
            T z = T(0);
#pragma unroll
            for (int q = 0; q < kRows; ++q)
                if (q == r) z = y.v[q];
            const auto at_X = [=](int v, int u) { return Xc[(long long)v * nR + u]; };
            const T f = (z + long_row_terms<T>(at_X, R, C, i, c0 + r)) * sigma;
            T* at = Xn + (long long)(c0 + r) * nR + i;
            if (even) {
                const double dy = (double)f - (double)Xo[(long long)(c0 + r) * nR + i];
                s.dy2 += dy * dy;
                s.dyy += dy * (double)f;
            }
            *at = f;
            s.nu2 += (double)f * (double)f;
        }
    }
    return s;
}

}  // namespace strips
}  // namespace cfsim
