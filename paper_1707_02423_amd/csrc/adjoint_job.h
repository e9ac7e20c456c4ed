// What the two reverse-mode paths share (adjoint.hip: one workgroup per pair;
// adjoint_strips.hip: every update of all pairs in one launch).
#pragma once

#include "cfsim_internal.h"
#include "pair_device.h"

namespace cfsim {

constexpr int kBwdThreads = 512;
constexpr int kBwdLds = 78 * 1024;
constexpr int kAChunks = 8;   // A edges held by the lanes (64 per chunk) in the lane-parallel edge sums
constexpr int kEdgeWaves = kBwdThreads / 64;   // partial sums of an A edge, one per wave

struct BwdJob {
    SetRef set;
    const int32_t* pair_a;
    const int32_t* pair_b;
    int n_pairs;
    const cfsim_pair_result* fwd;
    const int32_t* match;
    const int64_t* match_off;
    const double* grad_score;
    double* grad_w;
    int32_t* pair_status;  // optional: 0 done, CFSIM_INVALID_INPUT skipped
    int ckpt, max_iter;
    const void* fck;       // forward checkpoints (NULL: the forward is recomputed here)
    const int64_t* fck_off;
    void* ws;              // gridDim.x slots of slot_bytes
    long long slot_elems, slot_bytes;
    int32_t* queue;
    int strip_nodes;       // the pairs bwd_on_strips() takes are done elsewhere (0: none)
};

// LDS of the one-workgroup kernel: lists | gA, gB | edge sources | per-wave
// partials of the A edges, if they fit.
struct BwdShape {
    size_t lists, scratch_off;
    bool fits, lane_edges;
};
// kept: A's edges after invalid ones were dropped (at most nnzA).
__host__ __device__ inline BwdShape bwd_shape(int nA, int nB, int nnzA, int nnzB, int kept, int esize) {
    BwdShape s;
    s.lists = lds_lists_bytes(nB, nA, nnzB, nnzA, esize);
    s.scratch_off = s.lists + align16((size_t)(nnzA + nnzB) * 8) + align16((size_t)(nnzA + nnzB) * 4);
    s.fits = s.scratch_off <= (size_t)kBwdLds;
    s.lane_edges = kept <= kAChunks * kWave &&
                   s.scratch_off + (size_t)kEdgeWaves * kAChunks * kWave * esize <= (size_t)kBwdLds;
    return s;
}
__device__ inline BwdShape bwd_shape(const GraphRef& A, const GraphRef& B, int esize) {
    return bwd_shape(A.n, B.n, A.nnz, B.nnz, A.rp[A.n], esize);
}

// A pair of the call that can run (graphs and forward result).
__device__ inline bool bwd_pair(const BwdJob& J, int p, GraphRef* A, GraphRef* B) {
    const int ga = J.pair_a[p], gb = J.pair_b[p];
    const int K = J.fwd[p].iters;
    if (!(ga >= 0 && ga < J.set.n_graphs && gb >= 0 && gb < J.set.n_graphs && K >= 0 && K <= J.max_iter &&
          !(J.fwd[p].status & CFSIM_INVALID_INPUT)))
        return false;
    *A = graph_of(J.set, ga);
    *B = graph_of(J.set, gb);
    return A->n >= 1 && B->n >= 1 && (long long)A->n * B->n <= J.slot_elems;
}

// Pairs of the strips path: A edges within the lanes (the order of the partial
// sums is then the other kernel's) and both graphs within the node count that
// the call's tables and its strips' LDS are laid out for (its max_nodes; a
// graph above it may still fit the other kernel's slot).
constexpr int kBwdStripNodes = 512;
__device__ inline bool bwd_on_strips(const BwdJob& J, const GraphRef& A, const GraphRef& B, const BwdShape& s) {
    return s.fits && s.lane_edges && B.n <= J.strip_nodes && A.n <= J.strip_nodes;
}

// Host side of adjoint_strips.hip.
int launch_bwd_strips(int dtype, const BwdJob& J, int max_nodes, int num_cus, hipStream_t stream);

}  // namespace cfsim
