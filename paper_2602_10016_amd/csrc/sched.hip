// Offsets-driven work ordering (the software tile scheduler of App. "GDPA and Fused PFFN
// Kernel": sequence-length metadata decides the order in which work items are issued, so
// that the long histories start first and the short ones fill the tail).
//
// One workgroup sorts the examples by history length, longest first, with a counting sort
// over NBINS length buckets.  The attention kernels launch one workgroup per
// (example, head, query tile) in that order; the hardware dispatcher hands them to compute
// units as slots free up, which is longest-processing-time-first list scheduling.
// Results never depend on the order: each work item is computed by exactly one wavefront.
#include "common.h"

namespace kunlun {

constexpr int NBINS = 2048;
constexpr int SCHED_THREADS = 1024;

__global__ __launch_bounds__(SCHED_THREADS) void schedule_kernel(const int32_t* __restrict__ kv_off, int B,
                                                                  int max_kv, int32_t* __restrict__ order,
                                                                  int32_t* __restrict__ counters) {
    __shared__ int hist[NBINS];
    __shared__ int totals[16];
    static_assert(NBINS == 2 * SCHED_THREADS && SCHED_THREADS == 1024, "two bins per thread of the scan");
    const int tid = threadIdx.x;
    if (tid < (int)(WS_HEADER_BYTES / sizeof(int32_t))) counters[tid] = 0;
    for (int i = tid; i < NBINS; i += SCHED_THREADS) hist[i] = 0;
    __syncthreads();
    const int64_t span = (int64_t)max_kv + 1;
    auto bin_of = [&](int b) {
        int64_t len = (int64_t)kv_off[b + 1] - kv_off[b];
        int64_t x = len * NBINS / span;
        if (x > NBINS - 1) x = NBINS - 1;
        if (x < 0) x = 0;
        return NBINS - 1 - (int)x;  // bin 0 = longest
    };
    for (int b = tid; b < B; b += SCHED_THREADS) atomicAdd(&hist[bin_of(b)], 1);
    __syncthreads();
    // exclusive scan of hist, two neighbouring bins per thread; hist becomes the running cursor
    const int h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
    const int upto = scan1024(h0 + h1, totals);
    hist[2 * tid] = upto - h0 - h1;
    hist[2 * tid + 1] = upto - h1;
    __syncthreads();
    for (int b = tid; b < B; b += SCHED_THREADS) {
        const int pos = atomicAdd(&hist[bin_of(b)], 1);
        order[pos] = b;
    }
}

// Debug aid: counts the ways in which an offsets array breaks the contract (offsets[0] = 0, lengths in
// [0, max_len], offsets[B] = total); one workgroup, deterministic.
__global__ __launch_bounds__(SCHED_THREADS) void check_offsets_kernel(const int32_t* __restrict__ off, int B, int64_t total,
                                                                       int max_len, int32_t* __restrict__ violations) {
    __shared__ int bad[SCHED_THREADS];
    const int tid = threadIdx.x;
    int n = 0;
    for (int b = tid; b < B; b += SCHED_THREADS) {
        const int64_t len = (int64_t)off[b + 1] - off[b];
        n += (len < 0 || len > max_len) ? 1 : 0;
    }
    if (tid == 0) n += (off[0] != 0 ? 1 : 0) + ((int64_t)off[B] != total ? 1 : 0);
    bad[tid] = n;
    __syncthreads();
    for (int s = SCHED_THREADS / 2; s > 0; s >>= 1) {
        if (tid < s) bad[tid] += bad[tid + s];
        __syncthreads();
    }
    if (tid == 0) *violations = bad[0];
}

hipError_t launch_check_offsets(const int32_t* off, int B, int64_t total, int max_len, int32_t* violations, hipStream_t stream) {
    hipLaunchKernelGGL(check_offsets_kernel, dim3(1), dim3(SCHED_THREADS), 0, stream, off, B, total, max_len, violations);
    return hipGetLastError();
}

// MI355X has 256 compute units.
bool schedule_is_moot(int64_t workgroups, int wgs_per_cu) { return workgroups <= (int64_t)wgs_per_cu * 256; }

hipError_t launch_schedule(const int32_t* kv_off, int B, int max_kv, int32_t* order, int32_t* counters, hipStream_t stream) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(schedule_kernel, dim3(1), dim3(SCHED_THREADS), 0, stream, kv_off, B, max_kv, order, counters);
    return hipGetLastError();
}

int compute_units() {
    static const int n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;  // MI355X
        return cus;
    }();
    return n;
}

}  // namespace kunlun

namespace kunlun {

// ---- gradient of batch-shared seed queries (Sec. "Hierarchical Seed Pooling", stage 1: the learnable seeds are
// shared by all examples, so their gradient is the sum of the per-example query gradients).  No atomics: the
// order of every addition is fixed by (group, example), so the result does not depend on the launch.
// V consecutive elements per thread (16-byte loads when the row length allows it); the additions of one element
// happen in example order whatever V is.  What bounds it: the rows are read once, 134 MB for 256 examples of 256 seeds (8 heads,
// d = 128); with streaming loads 26 us = 5.2 TB/s, with plain ones 34 (eight or sixteen examples in flight instead of four 28, 29).
// Rows of up to 4 MB, which one XCD's L2 holds, are read with plain loads: whole backward calls, streaming over plain, 70 of 0.2 to 4 MB 0.994
// (0.945 to 1.006), from 6 to 16 MB 1.01 (0.99 to 1.05), to 80 MB 1.015 (0.98 to 1.085), beyond 1.02.
// LAST: the only group, its sums are the result.
template <typename T, int V, bool LAST, bool STREAM>
__global__ __launch_bounds__(256) void seed_grad_group_kernel(const T* __restrict__ rows, float* __restrict__ partial, T* __restrict__ d_e, int B,
                                                              int64_t n_elems) {
    typedef T vec_t __attribute__((ext_vector_type(V)));
    const int64_t n = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    const int group = blockIdx.y;
    if (n >= n_elems) return;
    const int b0 = group * SEED_GROUP, b1 = b0 + SEED_GROUP < B ? b0 + SEED_GROUP : B;
    float acc[V];
#pragma unroll
    for (int q = 0; q < V; ++q) acc[q] = 0.f;
#pragma unroll 4
    for (int b = b0; b < b1; ++b) {
        const vec_t* at = (const vec_t*)(rows + (int64_t)b * n_elems + n);
        const vec_t x = STREAM ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] += to_float((T)x[q]);
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
        if (LAST) d_e[n + q] = from_float<T>(acc[q]);
        else partial[(int64_t)group * n_elems + n + q] = acc[q];
    }
}
template <typename T>
__global__ __launch_bounds__(256) void seed_grad_final_kernel(const float* __restrict__ partial, T* __restrict__ d_e, int groups,
                                                              int64_t n_elems) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= n_elems) return;
    float acc = 0.f;
    for (int g = 0; g < groups; ++g) acc += partial[(int64_t)g * n_elems + n];
    d_e[n] = from_float<T>(acc);
}

template <typename T, int V>
static hipError_t launch_seed_grad(const T* rows, T* d_e, float* partial, int B, int64_t n_elems, hipStream_t stream) {
    const int groups = (B + SEED_GROUP - 1) / SEED_GROUP;
    const dim3 grid((unsigned)((n_elems / V + 255) / 256), (unsigned)groups);
    if (groups == 1) {  // up to SEED_GROUP examples: one launch (5 examples of 108 seeds, backward 22.6 / 20.4 us)
        hipLaunchKernelGGL((seed_grad_group_kernel<T, V, true, false>), grid, dim3(256), 0, stream, rows, partial, d_e, B, n_elems);
        return hipGetLastError();
    }
    if ((int64_t)B * n_elems * (int64_t)sizeof(T) > (int64_t)4 << 20)
        hipLaunchKernelGGL((seed_grad_group_kernel<T, V, false, true>), grid, dim3(256), 0, stream, rows, partial, d_e, B, n_elems);
    else
        hipLaunchKernelGGL((seed_grad_group_kernel<T, V, false, false>), grid, dim3(256), 0, stream, rows, partial, d_e, B, n_elems);
    hipLaunchKernelGGL(seed_grad_final_kernel<T>, dim3((unsigned)((n_elems + 255) / 256)), dim3(256), 0, stream, partial, d_e, groups, n_elems);
    return hipGetLastError();
}

hipError_t launch_seed_grad_sum(const void* rows, void* d_e, float* partial, int B, int64_t n_elems, int dtype, hipStream_t stream) {
    if (n_elems <= 0) return hipSuccess;
    const bool aligned = reinterpret_cast<uintptr_t>(rows) % 16 == 0;
    if (dtype == KUNLUN_FP32)
        return aligned && n_elems % 4 == 0 ? launch_seed_grad<float, 4>((const float*)rows, (float*)d_e, partial, B, n_elems, stream)
                                           : launch_seed_grad<float, 1>((const float*)rows, (float*)d_e, partial, B, n_elems, stream);
    return aligned && n_elems % 8 == 0 ? launch_seed_grad<bf16_t, 8>((const bf16_t*)rows, (bf16_t*)d_e, partial, B, n_elems, stream)
                                       : launch_seed_grad<bf16_t, 1>((const bf16_t*)rows, (bf16_t*)d_e, partial, B, n_elems, stream);
}

}  // namespace kunlun
