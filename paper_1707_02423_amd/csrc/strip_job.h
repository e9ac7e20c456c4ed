// Launch descriptor of the strip path (strips.hip): one plain pair whose
// iterates live in global memory.
#pragma once

#include "cfsim_internal.h"

namespace cfsim {

constexpr int kStripMaxNodes = 1024;    // its LDS: eight values per R node
constexpr int kStripMaxIter = 4096;     // one launch per update

struct StripState {
    unsigned status;       // CFSIM_* bits once the pair has stopped
    int iters;             // the last update that could be normalised
    double tot, inv;       // its squared norm and 1 / norm
    double a_even, d2;     // 1 / norm of the last even iterate; delta^2 (-1: none)
};

struct StripJob {
    PairJob J;             // the pair (ga, gb), options and outputs
    int swap, nR, nC;      // orientation (as PairShape)
    int strips;
    unsigned char* x[4];   // X_k in x[k % 4], nC x nR
    long long slot_elems;  // elements from one buffer to the next
    unsigned char* cols;   // column lists (strips.h)
    unsigned char* tabs;   // strip tables
    double* part;          // norm partials: two areas of 3 * strips
    StripState* st;        // [2] states after alternate steps
    LargeState* large;     // the final state for the kernels that match large pairs
};

size_t strip_bytes(int nA, int nB, int esize);
// Fills the descriptor's shape and carves its arrays from ws (strip_bytes()).
void carve_strips(StripJob* S, void* ws, int esize);
int set_strip_attributes();
int launch_strips(int dtype, const StripJob& job, hipStream_t stream);

}  // namespace cfsim
