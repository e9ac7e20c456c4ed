// Launch side of the pair kernels: the batch plan (step a8), the kernel of
// every bucket, and the launchers.  The kernels are in pair_kernels.h, one
// translation unit per measure and arithmetic type (pair_<measure>_<type>.hip).
#include "cfsim_internal.h"
#include "pair_device.h"

namespace cfsim {

const void* pair_kernel_plain_f32(int v);
const void* pair_kernel_plain_f64(int v);
const void* pair_kernel_damped_f32(int v);
const void* pair_kernel_damped_f64(int v);
const void* pair_kernel_resized_f32(int v);
const void* pair_kernel_resized_f64(int v);

namespace {

using namespace dev;

constexpr int kModePlain = 0;
constexpr int kModeDamped = 1;
constexpr int kModeResized = 2;

// Pairs no kernel can take get an INVALID_INPUT result.
__global__ void invalid_kernel(PairJob J) {
    const int begin = J.bounds[0], end = J.bounds[1];
    for (int it = begin + blockIdx.x * blockDim.x + threadIdx.x; it < end; it += gridDim.x * blockDim.x)
        write_invalid(J.res + J.order[it]);
}

// ---------------------------------------------------------------- plan (step a8)
constexpr int kPlanThreads = 1024;
constexpr int kClasses = 128;

__device__ void classify(const PlanJob& P, int64_t p, int* bucket, int* cls) {
    const int ga = P.pair_a[p], gb = P.pair_b[p];
    *cls = 0;
    *bucket = kBucketInvalid;
    if (P.filter) {  // FP64 pass of an FP32 call: near-tie pairs only
        const unsigned st = P.filter[p].status;
        if (!(st & CFSIM_NEAR_TIE) || (st & CFSIM_INVALID_INPUT)) {
            *bucket = -1;
            return;
        }
    }
    if (ga < 0 || ga >= P.set.n_graphs || gb < 0 || gb >= P.set.n_graphs) return;
    const int nA = (int)(P.set.node_off[ga + 1] - P.set.node_off[ga]);
    const int nB = (int)(P.set.node_off[gb + 1] - P.set.node_off[gb]);
    const int mA = (int)(P.set.edge_off[ga + 1] - P.set.edge_off[ga]);
    const int mB = (int)(P.set.edge_off[gb + 1] - P.set.edge_off[gb]);
    if (nA < 1 || nB < 1) return;
    PairShape sh;
    int b = kBucketInvalid;
    if (P.resize && nA != nB) {
        // resized mode: the first LDS variant that holds the resized pair, else
        // the global-memory kernel; the rest stay in the invalid bucket and
        // take the tiled path
        const int M = nA > nB ? nA : nB, m = nA > nB ? nB : nA;
        const int nnzL = nA > nB ? mA : mB, nnzX = nA > nB ? mB : mA;
        for (int v = 0; v < kNumVariants && b == kBucketInvalid; ++v)
            if (resized_fits(M, m, nnzL, nnzX, v, P.esize)) b = v;
        if (b == kBucketInvalid && resized_global_fits(M, m, nnzL, nnzX, P.esize, P.slot_elems)) b = kBucketGlobal;
    } else {
        for (int v = 0; v < kNumVariants && b == kBucketInvalid; ++v)
            if (choose_shape(nA, nB, mA, mB, v, P.esize, &sh)) b = v;
        if (b < kNumVariants) {  // a tuned larger variant for the pair's class, if it holds the pair
            const int t = P.tune[tune_class(nA, nB)];
            if (t > b && t < kNumVariants && choose_shape(nA, nB, mA, mB, t, P.esize, &sh)) b = t;
        }
        if (b == kBucketInvalid && !P.resize && global_fits(nA, nB, mA, mB, P.esize, P.slot_elems, &sh))
            b = kBucketGlobal;
    }
    if (P.filter && b == kBucketInvalid) {  // no FP64 kernel holds it: the FP32 result stays
        *bucket = -1;
        return;
    }
    // longest first: cost class from log2 of the work estimate (the resized
    // state is M x m, the iteration's shape either way)
    const double work = (double)nA * (double)nB * (1.0 + (double)(mA + mB) / (double)(nA + nB + 1));
    int c = (int)(4.0 * log2(work > 1.0 ? work : 1.0));
    c = c < 0 ? 0 : (c >= kClasses ? kClasses - 1 : c);
    *bucket = b;
    *cls = kClasses - 1 - c;
}

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(PlanJob P) {
    __shared__ int hist[kBuckets * kClasses];
    const int tid = threadIdx.x;
    for (int i = tid; i < kBuckets * kClasses; i += kPlanThreads) hist[i] = 0;
    __syncthreads();
    for (int64_t p = tid; p < P.n_pairs; p += kPlanThreads) {
        int b, c;
        classify(P, p, &b, &c);
        if (b >= 0) atomicAdd(&hist[b * kClasses + c], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int b = 0; b < kBuckets; ++b) {
            P.bounds[2 * b] = run;
            for (int c = 0; c < kClasses; ++c) {
                const int t = hist[b * kClasses + c];
                hist[b * kClasses + c] = run;
                run += t;
            }
            P.bounds[2 * b + 1] = run;
            P.queues[b] = 0;
        }
    }
    __syncthreads();
    for (int64_t p = tid; p < P.n_pairs; p += kPlanThreads) {
        int b, c;
        classify(P, p, &b, &c);
        if (b < 0) continue;
        const int slot = atomicAdd(&hist[b * kClasses + c], 1);
        P.order[slot] = (int32_t)p;
    }
}

__global__ __launch_bounds__(256) void buckets_kernel(PlanJob P, int32_t* bucket) {
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < P.n_pairs; p += (int64_t)gridDim.x * 256) {
        int b, c;
        classify(P, p, &b, &c);
        bucket[p] = b;
    }
}

const void* variant_kernel(int v, int dtype, int mode = kModePlain) {
    const bool f64 = dtype == CFSIM_F64;
    switch (mode) {
        case kModeDamped: return f64 ? pair_kernel_damped_f64(v) : pair_kernel_damped_f32(v);
        case kModeResized: return f64 ? pair_kernel_resized_f64(v) : pair_kernel_resized_f32(v);
        default: return f64 ? pair_kernel_plain_f64(v) : pair_kernel_plain_f32(v);
    }
}

int threads_of(int v, int esize, int mode) {
    if (v == kBucketGlobal) return mode == kModePlain ? plain_global_threads(esize) : kGlobalThreads;
    return variant_info(v, esize).nt;
}
int lds_of(int v, int esize, int mode) {
    if (v == kBucketGlobal) return mode == kModePlain ? plain_global_lds(esize) : kGlobalLds;
    return variant_info(v, esize).lds_bytes;
}

}  // namespace

int launch_pair_lds(int variant, int dtype, const PairJob& job, int grid, hipStream_t stream, bool whole_cu) {
    if (variant == kBucketInvalid) {
        hipLaunchKernelGGL(invalid_kernel, dim3(64), dim3(256), 0, stream, job);
        return (int)hipGetLastError();
    }
    const int esize = dtype == CFSIM_F64 ? 8 : 4;
    void* args[] = {const_cast<PairJob*>(&job)};
    const int mode = job.damped ? kModeDamped : (job.resize ? kModeResized : kModePlain);
    return (int)hipLaunchKernel(variant_kernel(variant, dtype, mode), dim3(grid),
                                dim3(threads_of(variant, esize, mode)), args,
                                (size_t)(whole_cu ? kCuLds : lds_of(variant, esize, mode)), stream);
}

int launch_plan(const PlanJob& job, hipStream_t stream) {
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, stream, job);
    return (int)hipGetLastError();
}

int launch_buckets(const PlanJob& job, int32_t* bucket, hipStream_t stream) {
    const int64_t blocks = (job.n_pairs + 255) / 256;
    hipLaunchKernelGGL(buckets_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, stream, job,
                       bucket);
    return (int)hipGetLastError();
}

// Kernel names as profilers list them (template arguments as in variant_kernel).
const char* bucket_kernel_name(int bucket, int dtype) {
    static const char* const f64[kBucketGlobal + 1] = {
        "pair_lds_kernel<double, 64, 1>", "pair_lds_kernel<double, 256, 2>", "pair_lds_kernel<double, 512, 2>",
        "pair_lds_kernel<double, 1024, 2>", "pair_lds_kernel<double, 1024, 4>", "pair_global_kernel<double>"};
    static const char* const f32[kBucketGlobal + 1] = {
        "pair_lds_kernel<float, 64, 2>", "pair_lds_kernel<float, 256, 4>", "pair_lds_kernel<float, 512, 2>",
        "pair_lds_kernel<float, 1024, 2>", "pair_lds_kernel<float, 1024, 4>", "pair_global_kernel<float>"};
    if (bucket < 0 || bucket > kBucketGlobal || (dtype != CFSIM_F64 && dtype != CFSIM_F32)) return "";
    return dtype == CFSIM_F64 ? f64[bucket] : f32[bucket];
}

int set_kernel_attributes() {
    int e = 0;
    for (int v = 0; v <= kBucketGlobal; ++v)
        for (int mode = kModePlain; mode <= kModeResized; ++mode) {
            e |= (int)hipFuncSetAttribute(variant_kernel(v, CFSIM_F32, mode),
                                          hipFuncAttributeMaxDynamicSharedMemorySize,
                                          v == kBucketGlobal ? kCuLds : lds_of(v, 4, mode));
            e |= (int)hipFuncSetAttribute(variant_kernel(v, CFSIM_F64, mode),
                                          hipFuncAttributeMaxDynamicSharedMemorySize,
                                          v == kBucketGlobal ? kCuLds : lds_of(v, 8, mode));
        }
    return e;
}

int occupancy_of(int variant, int dtype, int* blocks) {
    const int esize = dtype == CFSIM_F64 ? 8 : 4;
    return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, variant_kernel(variant, dtype),
                                                            threads_of(variant, esize, kModePlain),
                                                            (size_t)lds_of(variant, esize, kModePlain));
}

}  // namespace cfsim
