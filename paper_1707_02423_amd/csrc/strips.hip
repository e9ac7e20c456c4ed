// One plain pair past a workgroup's LDS on the undamped measure: every update
// is one launch over strips of four rows of X = S^T (strips.h), so that the
// pair runs on as many CUs as it has strips instead of on one.  A launch reads
// the norm partials the previous one left and takes the stopping decision
// itself, the same in every workgroup, so an update is one launch without a
// reduction between.  The terms of an entry are added in the order of the
// one-workgroup kernel; the norms' partial sums are grouped by strips and 1 / nu
// is rounded twice here, so that S agrees up to the rounding of the scale.
//
// Bound by the latency of one launch: its start, three dependent reads from
// memory and the barrier between the two stages, 6.3 us per update for a
// 333 x 410 FP32 pair (103 workgroups) against 145 us on one CU; 13.9 us where one
// node of the pair has more than four predecessors (the pass over such rows is
// a serial chain of its own).  The launches follow max_iter, not the updates
// done: cfsim_route_score_strips (api.hip) says where that pays.  Such a pair is
// matched in 0.6 ms by the large path's kernels (lines sorted over the chip), in
// 1.9 ms by one workgroup that keeps the columns' bests (which most columns
// agree on, so that most of them are looked up again at every pick).
#include "strip_job.h"
#include "strips.h"

namespace cfsim {

namespace {

using namespace dev;
using namespace strips;

constexpr int kDP = 4;   // predecessor slots of the pair kernels

// Lists, strip tables, X_0 and the first state.
template <typename T>
__global__ __launch_bounds__(256) void strip_build(StripJob S) {
    __shared__ int pos[2];
    const GraphRef R = pick_graph(S.swap != 0, S.J.ga, S.J.gb), C = pick_graph(S.swap != 0, S.J.gb, S.J.ga);
    const int tid = blockIdx.x * 256 + threadIdx.x, nt = gridDim.x * 256;
    const Cols<T> cols = carve_cols<T>(S.cols, S.nR, kDP);
    for (int i = tid; i < cols.stride; i += nt) build_col<T, kDP>(R, i, cols);
    StripTab<T>* tabs = reinterpret_cast<StripTab<T>*>(S.tabs);
    for (int s = tid; s < S.strips; s += nt) build_strip<T, kDP>(C, s * kRows, S.nR, tabs + s);
    const T s0 = T(1.0 / sqrt((double)S.nR * (double)S.nC));
    T* X = reinterpret_cast<T*>(S.x[0]);
    for (long long t = tid; t < (long long)S.nR * S.nC; t += nt) X[t] = s0;
    if (blockIdx.x != 0) return;
    if (threadIdx.x < 2) pos[threadIdx.x] = 0;
    __syncthreads();
    for (int e = threadIdx.x; e < R.nnz; e += 256)
        if (R.w[e] > 0.0) pos[0] = 1;
    for (int e = threadIdx.x; e < C.nnz; e += 256)
        if (C.w[e] > 0.0) pos[1] = 1;
    __syncthreads();
    if (threadIdx.x == 0) {
        StripState st{};
        st.status = pos[0] && pos[1] ? 0u : (unsigned)CFSIM_DEGENERATE;
        st.d2 = -1.0;
        st.a_even = 1.0;
        st.inv = 1.0;
        S.st[0] = st;  // the state after step 0
    }
}

// The state after step k from the one before and the strips' partials of
// step k (nu^2 and, for even k, the even-step sums), by one wave: the loop
// body of the one-workgroup kernels after their block reduction.
__device__ inline StripState step_state(StripState s, const double* part, int ntask, int k, int max_iter,
                                        double tol) {
    if (s.status != 0) return s;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    double v[3] = {0.0, 0.0, 0.0};
    for (int t = lane; t < ntask; t += kWave)
#pragma unroll
        for (int a = 0; a < 3; ++a) v[a] += part[3 * t + a];
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = wave_sum(v[a]);
    const double tot = v[0];
    if (!(tot > 0.0) || !isfinite(tot)) {  // cannot normalise: keep S_{k-1}
        s.status = CFSIM_DEGENERATE;
        return s;
    }
    s.iters = k;
    s.tot = tot;
    s.inv = 1.0 / sqrt(tot);
    if ((k & 1) == 0) {
        const double b = s.inv - s.a_even;
        s.d2 = fmax(s.a_even * s.a_even * v[1] + 2.0 * s.a_even * b * v[2] + b * b * tot, 0.0);
        s.a_even = s.inv;
        if (sqrt(s.d2) < tol) s.status = CFSIM_CONVERGED;
    }
    if (s.status == 0 && k == max_iter) s.status = CFSIM_HIT_MAX_ITER;
    return s;
}

// State after step k >= 0 (k = 0: as strip_build left it); st holds the state
// after step k - 1 in slot (k - 1) & 1.
__device__ inline StripState state_after(const StripJob& S, int k) {
    if (k == 0) return S.st[0];
    return step_state(S.st[(k - 1) & 1], S.part + (size_t)(k & 1) * 3 * S.strips, S.strips, k, S.J.max_iter, S.J.tol);
}

// Update k: X_k from X_{k-1}, one strip per workgroup.  Workgroups are dealt
// to the 8 XCDs round-robin; each XCD takes one contiguous range of strips, so
// that neighbouring strips find the rows they share in its L2.
template <typename T>
__global__ __launch_bounds__(kThreads) void strip_update(StripJob S, int k) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[3 * kWaves];
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = uni((int)threadIdx.x / kWave);
    const bool even = (k & 1) == 0;
    const int xcd = blockIdx.x & 7;
    const int strip = S.strips * xcd / 8 + (int)(blockIdx.x >> 3);
    if (strip >= S.strips * (xcd + 1) / 8) return;
    const int c0 = strip * kRows;
    const int nR = S.nR, nC = S.nC;
    const T* Xc = reinterpret_cast<const T*>(S.x[(k - 1) & 3]);
    T* Xn = reinterpret_cast<T*>(S.x[k & 3]);
    const T* Xo = reinterpret_cast<const T*>(S.x[(k - 2) & 3]);  // X_{k-2}
    const StripTab<T>* tab = reinterpret_cast<const StripTab<T>*>(S.tabs) + strip;
    Quad<T>* P1 = reinterpret_cast<Quad<T>*>(smem);
    Quad<T>* P2 = P1 + col_stride(nR) + 1;
    // what does not depend on the staged rows is read before them
    const Cols<T> cols = carve_cols<T>(S.cols, nR, kDP);
    const int nch = (nR + kWave - 1) / kWave;
    ColSlots<T, kDP> slots{};
    if (wave < nch) slots = load_col<T, kDP>(cols, wave * kWave + lane);
    if (threadIdx.x < 2) (threadIdx.x ? P2 : P1)[col_stride(nR)] = Quad<T>{};
    wave_sources(Xc, nR, tab, P1, P2, wave, kWaves);
    const StripState st = state_after(S, k - 1);
    if (strip == 0 && threadIdx.x == 0) S.st[(k - 1) & 1] = st;
    if (st.status != 0) return;  // the same in every thread
    const T sigma = k == 1 ? T(1) : T(st.inv);
    const GraphRef R = pick_graph(S.swap != 0, S.J.ga, S.J.gb), C = pick_graph(S.swap != 0, S.J.gb, S.J.ga);
    const int long_rows = uni(tab->long_rows);
    __syncthreads();
    double v[3] = {0.0, 0.0, 0.0};
    for (int ch = wave; ch < nch; ch += kWaves) {
        const int i = ch * kWave + lane;
        const bool valid = i < nR;
        T old[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            old[r] = even && valid && c0 + r < nC ? Xo[(long long)(c0 + r) * nR + i] : T(0);
        if (ch != wave) slots = load_col<T, kDP>(cols, i);
        const Quad<T> y = gather_slots<T, kDP>(slots, i, P1, P2, __ballot(slots.lng) != 0, [&] { return R; });
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            if (!valid || c0 + r >= nC || ((long_rows >> r) & 1)) continue;
            const T f = y.v[r] * sigma;
            Xn[(long long)(c0 + r) * nR + i] = f;
            v[0] += (double)f * (double)f;
            if (even) {
                const double dy = (double)f - (double)old[r];
                v[1] += dy * dy;
                v[2] += dy * (double)f;
            }
        }
    }
    if (long_rows) {
        const RowSums ls = long_rows_pass<T, kDP>(Xc, Xn, Xo, nR, nC, c0, long_rows, S.cols, P1, P2, R, C, sigma, even, wave,
                                                  kWaves);
        v[0] += ls.nu2;
        v[1] += ls.dy2;
        v[2] += ls.dyy;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = wave_sum(v[a]);
    if (lane == 0)
#pragma unroll
        for (int a = 0; a < 3; ++a) red[a * kWaves + wave] = v[a];
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        for (int w = 0; w < kWaves; ++w) s += red[threadIdx.x * kWaves + w];
        S.part[(size_t)(k & 1) * 3 * S.strips + 3 * strip + threadIdx.x] = s;
    }
}

// The final state as the large path keeps it.
__global__ void strip_large_state(StripJob S) {
    const StripState st = state_after(S, S.J.max_iter);
    if (threadIdx.x != 0) return;
    LargeState l{};
    l.nA = S.J.ga.n;
    l.nB = S.J.gb.n;
    l.nR = l.nB;
    l.nC = l.nA;
    l.status = st.status;
    l.final_step = st.iters;
    l.nu = st.iters > 0 ? sqrt(st.tot) : 0.0;
    l.delta = st.d2 >= 0.0 ? sqrt(st.d2) : __builtin_inf();
    for (int b = 0; b < 4; ++b) {
        l.nu_k[b] = st.iters > 0 ? l.nu : 1.0;
        l.inv_k[b] = 1.0 / l.nu_k[b];
    }
    *S.large = l;
}

template <typename T>
int launch_t(const StripJob& S, hipStream_t stream) {
    hipLaunchKernelGGL(strip_build<T>, dim3(64), dim3(256), 0, stream, S);
    int e = (int)hipGetLastError();
    if (e != 0) return e;
    const int grid = 8 * ((S.strips + 7) / 8);
    for (int k = 1; k <= S.J.max_iter; ++k) {
        hipLaunchKernelGGL(strip_update<T>, dim3(grid), dim3(kThreads), strip_lds<T>(S.nR), stream, S, k);
        if ((e = (int)hipGetLastError()) != 0) return e;
    }
    hipLaunchKernelGGL(strip_large_state, dim3(1), dim3(kWave), 0, stream, S);
    if ((e = (int)hipGetLastError()) != 0) return e;
    LargeJob L{};
    L.single = 1;
    L.ga = S.J.ga;
    L.gb = S.J.gb;
    L.n_pairs = 1;
    L.max_nodes = S.nR > S.nC ? S.nR : S.nC;
    L.max_iter = S.J.max_iter;
    L.tie_tol = S.J.tie_tol;
    L.res = S.J.res;
    L.match = S.J.match;
    L.S_out = S.J.S_out;
    L.st = S.large;
    L.bufs = S.x[0];
    L.nslots = 4;
    L.slot_elems = S.slot_elems;
    L.strips = !S.swap;  // X is S^T, or with swap S itself
    return launch_large_finish(sizeof(T) == 8 ? CFSIM_F64 : CFSIM_F32, L, stream);
}

template <typename T>
size_t carve_t(StripJob* S, unsigned char* ws, int nR, int nC) {
    const int strips = (nC + kRows - 1) / kRows;
    size_t o = 0;
    auto take = [&](size_t b) {
        unsigned char* p = ws + o;
        o += align16(b);
        return p;
    };
    const size_t buf = align16((size_t)nR * nC * sizeof(T));
    unsigned char* x = take(4 * buf);
    unsigned char* cols = take(cols_bytes<T>(nR, kDP));
    unsigned char* tabs = take((size_t)strips * sizeof(StripTab<T>));
    unsigned char* part = take((size_t)strips * 6 * sizeof(double));
    unsigned char* st = take(2 * sizeof(StripState));
    unsigned char* large = take(sizeof(LargeState));
    if (S) {
        S->strips = strips;
        for (int b = 0; b < 4; ++b) S->x[b] = x + (size_t)b * buf;
        S->slot_elems = (long long)(buf / sizeof(T));
        S->large = reinterpret_cast<LargeState*>(large);
        S->cols = cols;
        S->tabs = tabs;
        S->part = reinterpret_cast<double*>(part);
        S->st = reinterpret_cast<StripState*>(st);
    }
    return o;
}

}  // namespace

size_t strip_bytes(int nA, int nB, int esize) {
    const int swap = preferred_swap(nA, nB);
    const int nR = swap ? nA : nB, nC = swap ? nB : nA;
    return esize == 8 ? carve_t<double>(nullptr, nullptr, nR, nC) : carve_t<float>(nullptr, nullptr, nR, nC);
}

void carve_strips(StripJob* S, void* ws, int esize) {
    const int nA = S->J.ga.n, nB = S->J.gb.n;
    S->swap = preferred_swap(nA, nB);
    S->nR = S->swap ? nA : nB;
    S->nC = S->swap ? nB : nA;
    if (esize == 8)
        carve_t<double>(S, static_cast<unsigned char*>(ws), S->nR, S->nC);
    else
        carve_t<float>(S, static_cast<unsigned char*>(ws), S->nR, S->nC);
}

int set_strip_attributes() {
    int e = (int)hipFuncSetAttribute(reinterpret_cast<const void*>(&strip_update<float>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)strip_lds<float>(kStripMaxNodes));
    e |= (int)hipFuncSetAttribute(reinterpret_cast<const void*>(&strip_update<double>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)strip_lds<double>(kStripMaxNodes));
    return e;
}

int launch_strips(int dtype, const StripJob& job, hipStream_t stream) {
    return dtype == CFSIM_F64 ? launch_t<double>(job, stream) : launch_t<float>(job, stream);
}

}  // namespace cfsim
