// Ward's minimum-variance clustering (Section 6.2, "Clustering of Kernels")
// of n observations with f features each: squared Euclidean distances
// d_ij = ||X_i - X_j||^2, then n - 1 merges, each of the pair of current
// clusters with the smallest distance (ties: smaller slot pair), the merged
// cluster's distances following the Lance-Williams recurrence of Ward's method
// on squared distances,
//   d(k, i u j) = ((n_i + n_k) d_ki + (n_j + n_k) d_kj - n_k d_ij) / (n_i + n_j + n_k).
//
// Two kernels.  ward_distances fills the n x n matrix in the workspace (16 x 16
// pairs per workgroup, features staged through LDS 32 at a time, each sum
// taken in feature order).  ward_merge is one 1024-thread workgroup that keeps
// every slot's nearest neighbour (distance, index) in LDS: a merge step is a
// block argmin over the slots' cached neighbours, the recurrence for the
// merged slot's row and column with the slots' caches compared to it (one
// thread per slot), and the rescan of the rows whose neighbour was one of the
// merged pair (and of the merged slot's), one wave per row: three barriers.
// Under the tie rule the cached minimum over slots is the same pair the
// definition picks by scanning all pairs.  Arithmetic is FP64 without fused
// multiply-adds, in the order the definition states it, so heights are
// reproducible to the last bit.
//
// Bound by the chain of n - 1 dependent steps on one CU, 4.4 us each at
// n = 768 (3.4 ms with 256 features; 7.9 us, 6.1 ms, with six barriers, reads
// of columns, a rescan that waited for every read, and comparisons of values
// and indices in each of the argmin's steps, which now compare ranks).
#include <limits.h>
#include <math.h>

#include "cfsim_internal.h"
#include "pair_device.h"

namespace cfsim {

namespace {

using namespace dev;

constexpr int kDistTile = 16;
constexpr int kFeatTile = 32;
constexpr int kMergeThreads = 1024;
constexpr int kMergeWaves = kMergeThreads / kWave;

#pragma clang fp contract(off)

__global__ __launch_bounds__(kDistTile * kDistTile) void ward_distances(const double* __restrict__ X, int n, int f,
                                                                        double* __restrict__ D) {
    __shared__ double xi[kDistTile][kFeatTile + 1];
    __shared__ double xj[kDistTile][kFeatTile + 1];
    const int tx = threadIdx.x % kDistTile, ty = threadIdx.x / kDistTile;
    const int i0 = blockIdx.y * kDistTile, j0 = blockIdx.x * kDistTile;
    const int i = i0 + ty, j = j0 + tx;
    double d = 0.0;
    for (int k0 = 0; k0 < f; k0 += kFeatTile) {
        for (int t = threadIdx.x; t < kDistTile * kFeatTile; t += kDistTile * kDistTile) {
            const int r = t / kFeatTile, k = k0 + t % kFeatTile;
            const double a = (i0 + r < n && k < f) ? X[(long long)(i0 + r) * f + k] : 0.0;
            const double b = (j0 + r < n && k < f) ? X[(long long)(j0 + r) * f + k] : 0.0;
            xi[r][t % kFeatTile] = a;
            xj[r][t % kFeatTile] = b;
        }
        __syncthreads();
        const int kn = f - k0 < kFeatTile ? f - k0 : kFeatTile;
        for (int k = 0; k < kn; ++k) {
            const double t = xi[ty][k] - xj[tx][k];
            d = d + t * t;
        }
        __syncthreads();
    }
    if (i < n && j < n) D[(long long)i * n + j] = d;
}

// Distance from slot k to the union of slots i and j.
__device__ inline double ward_update(double dki, double dkj, double dij, double ni, double nj, double nk) {
    return ((ni + nk) * dki + (nj + nk) * dkj - nk * dij) / (ni + nj + nk);
}

// Rank of a distance: larger is nearer, 0 for NaN (never chosen).
__device__ inline uint64_t nearness(double d) {
    const uint64_t b = (uint64_t)__double_as_longlong(d + 0.0);  // -0 ranks as +0
    return d != d ? 0 : ~(b ^ ((b >> 63) ? ~0ull : 1ull << 63));
}
__device__ inline double distance_of(uint64_t rank) {
    const uint64_t b = ~rank;
    return __longlong_as_double((long long)(b >> 63 ? b ^ (1ull << 63) : ~b));
}
template <int CTRL>
__device__ inline uint64_t max_step(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), CTRL, 0xF, 0xF, true);
    const uint64_t y = ((uint64_t)hi << 32) | lo;
    return y > x ? y : x;
}
__device__ inline uint64_t lane_bits(uint64_t x, int l) {
    return ((uint64_t)(uint32_t)lane_value((int)(uint32_t)(x >> 32), l) << 32) | (uint32_t)lane_value((int)(uint32_t)x, l);
}
// Largest rank of the wave and its smallest index, the same in every lane;
// indices are compared only where several lanes hold that rank.
__device__ inline void wave_nearest(uint64_t& rank, int& index) {
    uint64_t m = max_step<kDppXor1>(rank);
    m = max_step<kDppXor2>(m);
    m = max_step<kDppHalfMirror>(m);
    m = max_step<kDppMirror>(m);
    uint64_t t = lane_bits(m, 0);
#pragma unroll
    for (int r = 16; r < kWave; r += 16) {
        const uint64_t o = lane_bits(m, r);
        t = o > t ? o : t;
    }
    const uint64_t at = __ballot(rank == t);
    if ((at & (at - 1)) != 0)
        index = (int)wave_min_u32(rank == t ? (uint32_t)index : 0xFFFFFFFFu);
    else
        index = lane_value(index, (int)__builtin_ctzll(at));
    rank = t;
}

// Nearest active slot of row k other than `gone` (smallest distance, then
// smallest index) by one wave; (NaN, INT_MAX) if there is none.  The
// reads do not depend on the slots' states, so that 16 are in flight.
__device__ inline void row_nearest(const double* D, int n, int k, int gone, const int* active, double& bd, int& bj) {
    uint64_t rank = 0;
    int key = INT_MAX;
    const double* row = D + (long long)k * n;
    constexpr int kBatch = 16;
    for (int j0 = threadIdx.x % kWave; j0 < n; j0 += kBatch * kWave) {
        double x[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) x[u] = row[min(j0 + u * kWave, n - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {  // ascending: the first of equal ranks stays
            const int j = j0 + u * kWave;
            if (j >= n) break;
            const uint64_t r = nearness(x[u]);
            if (j != k && j != gone && active[j] && r > rank) {
                rank = r;
                key = j;
            }
        }
    }
    wave_nearest(rank, key);
    bj = rank ? key : INT_MAX;
    bd = rank ? distance_of(rank) : __builtin_nan("");  // ranks as no candidate
}

__global__ __launch_bounds__(kMergeThreads) void ward_merge(const double* X, int f, double* D, int n, double* Z) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* nnd = reinterpret_cast<double*>(smem);  // [n] distance to the nearest active slot
    double* size = nnd + n;                         // [n] observations in the slot's cluster
    double* ident = size + n;                       // [n] cluster number of the slot
    int* nn = reinterpret_cast<int*>(ident + n);    // [n] nearest active slot
    int* active = nn + n;                           // [n]
    int* todo = active + n;                         // [n] slots to rescan
    __shared__ uint64_t wv[kMergeWaves];
    __shared__ int wk[kMergeWaves];
    __shared__ int ntodo[2];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    int nonfinite = 0;
    for (long long t = tid; t < (long long)n * f; t += kMergeThreads) nonfinite |= !isfinite(X[t]);
    if (__syncthreads_or(nonfinite)) {  // a non-finite feature: every row of the linkage is NaN
        for (long long t = tid; t < 4ll * (n - 1); t += kMergeThreads) Z[t] = __builtin_nan("");
        return;
    }
    for (int k = tid; k < n; k += kMergeThreads) {
        size[k] = 1.0;
        ident[k] = (double)k;
        active[k] = 1;
    }
    __syncthreads();
    for (int k = wave; k < n; k += kMergeWaves) {
        double bd;
        int bj;
        row_nearest(D, n, k, k, active, bd, bj);
        if (lane == 0) {
            nnd[k] = bd;
            nn[k] = bj;
        }
    }
    if (tid < 2) ntodo[tid] = 0;
    __syncthreads();
    for (int s = 0; s < n - 1; ++s) {
        // the active slot with the nearest neighbour (distance, then slot)
        uint64_t rank = 0;
        int key = INT_MAX;
        for (int k = tid; k < n; k += kMergeThreads) {
            const uint64_t r = active[k] ? nearness(nnd[k]) : 0;
            if (r > rank) {
                rank = r;
                key = k;
            }
        }
        wave_nearest(rank, key);
        if (lane == 0) {
            wv[wave] = rank;
            wk[wave] = key;
        }
        __syncthreads();
        rank = lane < kMergeWaves ? wv[lane] : 0;
        key = lane < kMergeWaves ? wk[lane] : INT_MAX;
        wave_nearest(rank, key);
        const int r = key, q = rank ? nn[r] : INT_MAX;
        if (q >= n) {  // no distance is a number any more (features of 1e150 and up)
            for (int t = 4 * s + tid; t < 4 * (n - 1); t += kMergeThreads) Z[t] = __builtin_nan("");
            return;
        }
        const int i = r < q ? r : q, j = r < q ? q : r;
        const double dij = nnd[r];
        const double ni = size[i], nj = size[j];
        // a slot's own thread updates its distance to the union and its cached
        // neighbour; rows i and j are read along, columns only written
        int* count = ntodo + (s & 1);
        for (int k = tid; k < n; k += kMergeThreads) {
            if (!active[k] || k == j) continue;
            if (k == i) {
                todo[atomicAdd(count, 1)] = k;
                continue;
            }
            const double d = ward_update(D[(long long)i * n + k], D[(long long)j * n + k], dij, ni, nj, size[k]);
            D[(long long)k * n + i] = d;
            D[(long long)i * n + k] = d;
            if (nn[k] == i || nn[k] == j) {
                todo[atomicAdd(count, 1)] = k;
            } else if (d < nnd[k] || (d == nnd[k] && i < nn[k])) {
                nnd[k] = d;
                nn[k] = i;
            }
        }
        __syncthreads();
        const int nt = *count;
        for (int t = wave; t < nt; t += kMergeWaves) {
            const int k = todo[t];
            double bd;
            int bj;
            row_nearest(D, n, k, j, active, bd, bj);
            if (lane == 0) {
                nnd[k] = bd;
                nn[k] = bj;
            }
        }
        if (tid == 0) {
            const double a = ident[i], b = ident[j];
            Z[4ll * s + 0] = a < b ? a : b;
            Z[4ll * s + 1] = a < b ? b : a;
            Z[4ll * s + 2] = dij;
            Z[4ll * s + 3] = ni + nj;
            ident[i] = (double)(n + s);
            size[i] = ni + nj;   // read again behind the next barrier only
            active[j] = 0;       // the rescans leave j out by themselves
            ntodo[(s + 1) & 1] = 0;
        }
        __syncthreads();
    }
}

}  // namespace

size_t ward_merge_lds(int n) { return (size_t)n * (3 * sizeof(double) + 3 * sizeof(int)); }

int launch_ward(const double* X, int n, int f, double* Z, double* D, hipStream_t stream) {
    const int tiles = (n + kDistTile - 1) / kDistTile;
    hipLaunchKernelGGL(ward_distances, dim3(tiles, tiles), dim3(kDistTile * kDistTile), 0, stream, X, n, f, D);
    int e = (int)hipGetLastError();
    if (e != 0) return e;
    const size_t lds = ward_merge_lds(n);
    if ((e = (int)hipFuncSetAttribute(reinterpret_cast<const void*>(&ward_merge),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) != 0)
        return e;
    hipLaunchKernelGGL(ward_merge, dim3(1), dim3(kMergeThreads), lds, stream, X, f, D, n, Z);
    return (int)hipGetLastError();
}

}  // namespace cfsim
