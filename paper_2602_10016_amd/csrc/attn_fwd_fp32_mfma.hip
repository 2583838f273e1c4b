// fp32 forward of GDPA / softmax attention (Eq. (GDPA), Eq. (PMA)) on the matrix cores, head dimensions 32, 64 and 128:
// v_mfma_f32_16x16x4_f32, full fp32 products and sums, exact score functions.
//
// A workgroup owns one (example, head, block of 16 or 32 queries); its waves take the 32-key steps of the history in
// turn and keep partial results of their own (accumulators, softmax reference and sum), which are merged in LDS in wave
// order.  Nothing else goes through LDS: a wave fetches its operands from memory in the order the instruction wants them.
// Layouts (lane l, r = l % 16, c4 = l / 16): A row r, contraction c4; B column r, contraction c4; C column r, rows
// 4 c4 + v.  S^T = K Q^T contracts over channels in the order in which lane group c4 owns channels c4 d/4 ..: every lane
// reads a quarter of a row of K and Q, contiguous.  The weights of a lane then belong to query r and keys 4 c4 + v, so
// register v is the B operand of contraction step v of O^T += V^T P^T, whose A operand is V[4 c4 + v][channel r].
//
// What bounds it: a call of a few examples is a chain of latencies (row loads, d/4 matrix instructions, score function,
// merge); two examples of 8 queries and 64 keys, 2 heads, d = 32 take 4.3 us against 13.7 us with one wave per query row
// (scalar_kernels.hip, which keeps the other head dimensions, the sliding window and the backward).
#include "common.h"

namespace kunlun {

typedef __attribute__((ext_vector_type(4))) float f4;

template <int D>
struct F32Fwd {
    static constexpr int QC = D / 4;    // channels of a lane group
    static constexpr int CB = D / 16;   // 16-channel blocks of O
    static constexpr int MAX_KS = D == 128 ? 4 : D == 64 ? 8 : 16;  // waves (registers: 512, 256, 128 per lane)
    static constexpr int part_bytes(int qb) { return qb * (CB + 1) * 1024; }  // a wave's accumulators, then reference and sum
};

template <int D, int QB, int ACT>
__device__ __forceinline__ void attn_fwd_fp32_item(const AttnParams& p, char* lds, int h, int64_t q_row0, int nq, int64_t k0, int n_kv) {
    using F = F32Fwd<D>;
    constexpr bool SOFTMAX = ACT == KUNLUN_ACT_SOFTMAX;
    constexpr int QC = F::QC, CB = F::CB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ks = blockDim.x >> 6;
    const int r = lane & 15, c4 = lane >> 4;
    const int64_t hd = (int64_t)p.H * D;
    const float* Q = (const float*)p.q + q_src_row(p, q_row0) * hd + (int64_t)h * D;
    const float* K = (const float*)p.k + (k0 * p.H + h) * D;
    const float* V = (const float*)p.v + (k0 * p.H + h) * D;

    f4 qf[QB][QC / 4];  // rows past the block repeat its last one (never stored)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = 16 * qb + r < nq ? 16 * qb + r : nq - 1;
#pragma unroll
        for (int c = 0; c < QC / 4; ++c) qf[qb][c] = *(const f4*)(Q + row * hd + c4 * QC + 4 * c);
    }
    f4 o[CB][QB];
    float m[QB], l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m[qb] = -INFINITY;
        l[qb] = 0.f;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) o[cb][qb] = (f4){0.f, 0.f, 0.f, 0.f};
    }
    for (int key0 = 32 * wave; key0 < n_kv; key0 += 32 * ks) {
        const int left = n_kv - key0;
        f4 kf[2][QC / 4];
        float vf[2][CB][4];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const int row = 16 * kb + r < left ? 16 * kb + r : left - 1;
#pragma unroll
            for (int c = 0; c < QC / 4; ++c) kf[kb][c] = *(const f4*)(K + (key0 + row) * hd + c4 * QC + 4 * c);
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int key = 16 * kb + 4 * c4 + v;
                const int row = key < left ? key : left - 1;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) vf[kb][cb][v] = V[(key0 + row) * hd + 16 * cb + r];
            }
        // ---- S^T, one query per lane
        f4 s[2][QB];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[kb][qb] = (f4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < QC; ++c)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][c / 4][c % 4], qf[qb][c / 4][c % 4], s[kb][qb], 0, 0, 0);
        // ---- weights; keys past the history get none, and their (repeated) V rows count as zero
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mx = -INFINITY, shift = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[kb][qb][v] *= p.scale;
                    if (SOFTMAX) mx = fmaxf(mx, 16 * kb + 4 * c4 + v < left ? s[kb][qb][v] : -INFINITY);
                }
            if (SOFTMAX) {
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                const float m_new = fmaxf(m[qb], mx);
                shift = m_new == -INFINITY ? 0.f : m_new;  // only scores of -inf so far: their weights are exp(-inf) = 0
                const float corr = expf(m[qb] - shift);    // exp(-inf) = 0 in the first step
                m[qb] = m_new;
                l[qb] *= corr;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) o[cb][qb] *= corr;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool ok = 16 * kb + 4 * c4 + v < left;
                    float w;
                    if (SOFTMAX) {
                        w = ok ? expf(s[kb][qb][v] - shift) : 0.f;
                        l[qb] += w;
                    } else {
                        w = ok ? act_exact<ACT>(s[kb][qb][v]) : 0.f;
                    }
                    s[kb][qb][v] = w;
                }
        }
        if (left < 32) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) vf[kb][cb][v] = 16 * kb + 4 * c4 + v < left ? vf[kb][cb][v] : 0.f;
        }
        // ---- O^T += V^T P^T
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
                        o[cb][qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[kb][cb][v], s[kb][qb][v], o[cb][qb], 0, 0, 0);
    }
    if (SOFTMAX) {  // a query's sum is spread over the four lane groups
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            l[qb] += __shfl_xor(l[qb], 16, 64);
            l[qb] += __shfl_xor(l[qb], 32, 64);
        }
    }
    // ---- merge: every wave but the first leaves its part in LDS, the first adds them in wave order
    if (ks > 1) {
        char* mine = lds + (wave - 1) * F::part_bytes(QB) + lane * 16;
        if (wave > 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) *(f4*)(mine + (qb * (CB + 1) + cb) * 1024) = o[cb][qb];
                if (SOFTMAX) *(f4*)(mine + (qb * (CB + 1) + CB) * 1024) = (f4){m[qb], l[qb], 0.f, 0.f};
            }
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < ks - 1 && 32 * (w + 1) < n_kv; ++w) {  // (a wave past the end of the history saw no key)
            const char* part = lds + w * F::part_bytes(QB) + lane * 16;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float c0 = 1.f, c1 = 1.f;
                if (SOFTMAX) {
                    const f4 ml = *(const f4*)(part + (qb * (CB + 1) + CB) * 1024);
                    const float m_new = fmaxf(m[qb], ml[0]);
                    const float shift = m_new == -INFINITY ? 0.f : m_new;  // as above: a part without a weight counts as zero
                    c0 = expf(m[qb] - shift);
                    c1 = expf(ml[0] - shift);
                    l[qb] = l[qb] * c0 + ml[1] * c1;
                    m[qb] = m_new;
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const f4 x = *(const f4*)(part + (qb * (CB + 1) + cb) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[cb][qb][e] = SOFTMAX ? fmaf(x[e], c1, o[cb][qb][e] * c0) : o[cb][qb][e] + x[e];
                }
            }
        }
    }
    // ---- lane: query 16 qb + r, channels 16 cb + 4 c4 ..
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qi = 16 * qb + r;
        if (qi >= nq) continue;
        float inv = 1.f;
        if (SOFTMAX) {
            inv = l[qb] > 0.f ? 1.f / l[qb] : 1.f;
            if (p.lse && c4 == 0) p.lse[(int64_t)h * p.total_q + q_row0 + qi] = n_kv > 0 ? m[qb] + logf(l[qb]) : -INFINITY;
        }
        float* out = (float*)p.o + (q_row0 + qi) * hd + (int64_t)h * D + 4 * c4;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) *(f4*)(out + 16 * cb) = SOFTMAX ? o[cb][qb] * inv : o[cb][qb];
    }
}

template <int D, int QB>
__global__ __launch_bounds__(64 * F32Fwd<D>::MAX_KS) void gdpa_fwd_fp32_kernel(AttnParams p, int n_qtiles) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int h = (int)(blockIdx.x % p.H);
    const int64_t e = blockIdx.x / p.H;
    const int qt = (int)(e % n_qtiles), b = (int)(e / n_qtiles);
    const int64_t q0 = q_begin(p, b) + (int64_t)qt * 16 * QB;
    const int64_t left = q_end(p, b) - q0;
    if (left <= 0) return;
    const int nq = (int)(left < 16 * QB ? left : 16 * QB);
    const int64_t k0 = p.kv_off[b];
    const int n_kv = p.kv_off[b + 1] - (int)k0;
    switch (p.head_act[h]) {
    case KUNLUN_ACT_SOFTMAX: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_SOFTMAX>(p, lds, h, q0, nq, k0, n_kv); break;
    case KUNLUN_ACT_IDENTITY: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_IDENTITY>(p, lds, h, q0, nq, k0, n_kv); break;
    case KUNLUN_ACT_RELU: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_RELU>(p, lds, h, q0, nq, k0, n_kv); break;
    case KUNLUN_ACT_GELU: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_GELU>(p, lds, h, q0, nq, k0, n_kv); break;
    case KUNLUN_ACT_GELU_TANH: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_GELU_TANH>(p, lds, h, q0, nq, k0, n_kv); break;
    case KUNLUN_ACT_SILU: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_SILU>(p, lds, h, q0, nq, k0, n_kv); break;
    default: attn_fwd_fp32_item<D, QB, KUNLUN_ACT_GELU_POLY>(p, lds, h, q0, nq, k0, n_kv); break;
    }
}

// Queries of a workgroup, and the workgroups of the longest query list the call allows, for every (example, head).
static int fp32_block_rows(int max_q) { return max_q <= 16 ? 16 : 32; }
static int64_t fp32_blocks(const AttnParams& p) {
    const int rows = fp32_block_rows(p.max_q);
    return (int64_t)p.B * p.H * ((p.max_q + rows - 1) / rows);
}

// The grid must stay below 2^32 threads (a larger one is cut off without an error).  And with q_offsets many of its
// workgroups may hold few queries or none, all of those that do perhaps on a quarter of the device: a workgroup has to
// have two query rows on average (one, in the small blocks), else the scalar kernel takes the call.  Scalar / this, us:
//   B = 70000, one query each, 2 keys: bound 16 551 / 523, 32 551 / 913, 128 551 / 3570;  B = 20000, 64 keys, bound 512 1105 / 2228;
//   B = 512, 1..16 queries, 64..512 keys, d = 64: bound 32 1108 / 184, 128 (2.1 rows) 1108 / 478
bool fp32_fwd_supported(const AttnParams& p, int dtype) {
    return dtype == KUNLUN_FP32 && !p.windowed && p.max_q >= 1 && (p.d == 32 || p.d == 64 || p.d == 128) &&
           fp32_blocks(p) < ((int64_t)1 << 26) && fp32_blocks(p) * (fp32_block_rows(p.max_q) / 16) <= p.total_q * p.H;
}

template <int D, int QB>
static hipError_t launch(const AttnParams& p, hipStream_t stream) {
    using F = F32Fwd<D>;
    constexpr int max_bytes = (F::MAX_KS - 1) * F::part_bytes(QB);
    auto kern = gdpa_fwd_fp32_kernel<D, QB>;
    if (max_bytes > 64 * 1024) {
        // once per process (thread-safe initialisation of a function-local static); not a stream operation
        static const hipError_t raised = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, max_bytes);
        if (raised != hipSuccess) return raised;
    }
    const int n_qtiles = (p.max_q + 16 * QB - 1) / (16 * QB);
    const int64_t items = fp32_blocks(p);
    const int steps = (p.max_kv + 31) / 32;
    // as many waves as the longest history has steps, while the waves of all items are fewer than four per SIMD (64 examples
    // of up to 16 queries, 8 heads, d = 64, 64..512 keys: 24 us; one wave per query row 192)
    int ks = 1;
    while (ks < F::MAX_KS && ks < steps && items * ks < 4096) ks *= 2;
    hipLaunchKernelGGL(kern, dim3((unsigned)items), dim3(64 * ks), (ks - 1) * F::part_bytes(QB), stream, p, n_qtiles);
    return hipGetLastError();
}

hipError_t launch_fp32_fwd(const AttnParams& p, hipStream_t stream) {
    if (fp32_block_rows(p.max_q) == 16)
        return p.d == 32 ? launch<32, 1>(p, stream) : p.d == 64 ? launch<64, 1>(p, stream) : launch<128, 1>(p, stream);
    return p.d == 32 ? launch<32, 2>(p, stream) : p.d == 64 ? launch<64, 2>(p, stream) : launch<128, 2>(p, stream);
}

}  // namespace kunlun
