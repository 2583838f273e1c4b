// SumKronLinear forward as ONE kernel, Eq. (SumKronLinear) of Sec. "Hierarchical Seed Pooling" (stage 3):
//     Y_b = sum_i Z_i^T X_b W_i ,   X_b [S, D], Z_i [S, T], W_i [D, D], Y_b [T, D],  T = 32.
// The intermediate U_{b,i} = Z_i^T X_b never leaves the compute unit.  The operator has the shape of the
// attention kernels: per 32-channel block of X,
//     stage 1   U^T_{b,i}[c, t] = sum_s X_b[s, c] Z_i[s, t]      ("scores": rows = channels c of the block, columns = t)
//     stage 2   Y^T_b[n, t]    += sum_c W_i[c, n] U^T_{b,i}[c, t]  ("values": W_i^T, summed over (i, c))
// and as there the transposed first product leaves every lane with one column t and 16 rows c of a 32 x 32 tile,
// which - rounded to bf16 - is directly the B operand of the second product, provided that its A operand (W_i^T)
// is read in the same order of c; X^T comes from the row-major X rows through transposing LDS reads.
//
// A workgroup of 8 waves works on FOUR examples at a time (persistent: groups blockIdx.x, + gridDim.x, ...):
//   stage 1: wave i owns factor Z_i and forms U^T_{e,i} of the block for the four examples, S/16 steps each, A
//            fragments from the X blocks in LDS, B fragments (Z_i) in registers;
//   the packed results go, register image by register image, into an LDS exchange buffer (64 KB);
//   stage 2: wave (g, h) owns the output channels [D/4 * g, D/4 * (g + 1)) of the examples 2h and 2h + 1 (2 * D/128
//            accumulator tiles that live for the whole group): the U^T fragments come from the exchange buffer, the
//            W fragments straight from global memory, three fragment steps ahead of their use, each used for both
//            examples.
// What sets the shape: W (2.4 MB) is read by every workgroup for every group of examples, so the L2 traffic per example
// is W / (examples that share a fragment load).  With two examples per workgroup and one per wave the kernel was bound
// by exactly that (2.4 GB at the 12 TB/s the L2s sustained: 192 us).  Two examples per wave need twice the accumulators; the Z
// fragments stay in registers beside them, read once per workgroup (at D = 384 and S = 256 that is all 256 registers, and two
// addresses go to scratch memory).
// W is prepared once per call in fragment order: the 64 x 16 bytes that the lanes of a wave need for one MFMA are
// 1 KB contiguous (read the other way - 16 bytes per lane from 32 different rows - every load touched 32 cache
// lines and the kernel ran at a third of its speed).  Z likewise transposed, in the c order of the register layout.
// X blocks of the next step set out for LDS at the start of stage 2, as soon as stage 1 has read the old ones, without
// passing through registers.
// Per example: 3840 MFMAs of 32x32x16 (the 126 MFLOP of the operator), X read once.
#include "lds_ring.h"

namespace kunlun {

constexpr int SKF_T = 32;       // output tokens per example (columns of Z_i)
constexpr int SKF_CB = 32;      // channels of X per step
constexpr int SKF_WAVES = 8;
constexpr int SKF_EX = 4;       // examples per workgroup step

// position p of a 16-group holds channel perm(p): lane half g of a B fragment owns {4g..4g+3, 8+4g..8+4g+3}
__host__ __device__ inline int skf_perm(int p) { return (p & 3) + 4 * (p >> 3) + 8 * ((p >> 2) & 1); }

// Once per call, in one launch (two took 6 us more); eight values per thread.
// Z: zt[(i*T + t)*S + 16q + p] = z[(i*S + 16q + perm(p))*T + t].
// W in fragment order: fragment (i, channel block cb of 32, output block nb of 32, half cc) holds, for lane (r, g) and
// q = 0..7, w[i][c = 32*cb + 16*cc + perm(8g + q)][n = 32*nb + r]; 512 values per fragment, lane-major.
__global__ __launch_bounds__(256) void skf_prepare_kernel(const bf16_t* __restrict__ w, const bf16_t* __restrict__ z, bf16_t* __restrict__ wp,
                                                          bf16_t* __restrict__ zt, int k, int D, int S, int T, int w_blocks) {
    bf16x8 out;
    if ((int)blockIdx.x < w_blocks) {
        const int idx = blockIdx.x * 256 + threadIdx.x;
        if (idx >= k * D * (D / 8)) return;
        const int lane = idx & 63, cc = (idx >> 6) & 1, rest = idx >> 7;  // (i * D/32 + cb) * D/32 + nb
        const int nb = rest % (D / 32), cb = (rest / (D / 32)) % (D / 32), i = rest / ((D / 32) * (D / 32));
        const bf16_t* src = w + ((int64_t)i * D + 32 * cb + 16 * cc) * D + 32 * nb + (lane & 31);
#pragma unroll
        for (int q = 0; q < 8; ++q) out[q] = src[skf_perm(8 * (lane >> 5) + q) * D];
        *(bf16x8*)(wp + (int64_t)idx * 8) = out;
    } else {
        const int idx = (blockIdx.x - w_blocks) * 256 + threadIdx.x;  // t fastest: the reads of a wave are contiguous
        if (idx >= k * T * (S / 8)) return;
        const int t = idx % T, s8 = (idx / T) % (S / 8), i = idx / (T * (S / 8));
        const bf16_t* src = z + ((int64_t)i * S + (s8 >> 1) * 16) * T + t;
#pragma unroll
        for (int q = 0; q < 8; ++q) out[q] = src[skf_perm(8 * (s8 & 1) + q) * T];
        *(bf16x8*)(zt + ((int64_t)i * T + t) * S + s8 * 8) = out;
    }
}

// SPLIT: a workgroup takes one group of examples and a range of the channel blocks (the contraction of stage 2) and leaves an
// fp32 partial sum of Y in part[range]; skf_sum_kernel adds the ranges in order.  For batches that would leave compute units
// empty, where one group's chain of D / 32 steps sets the time.
template <int NBW, int S, bool SPLIT>  // D = 128 * NBW output / input channels; S rows of X per example (128 or 256)
__global__ __launch_bounds__(64 * SKF_WAVES, 1) void sumkron_fused_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ zt,
                                                                          const bf16_t* __restrict__ wp, bf16_t* __restrict__ y,
                                                                          int B, int k, float* __restrict__ part, int blocks_per_range) {
    using L = TileLayout<SKF_CB>;  // 32-row tiles of 32 channels, the layout of the transposing reads
    constexpr int D = 128 * NBW;
    constexpr int KS = S / 16;                  // contraction steps of stage 1
    constexpr int NCB = D / SKF_CB;             // channel blocks of X
    constexpr int XBYTES = S * SKF_CB * 2;      // one example's block
        constexpr int FRAG = 1024;                  // a packed B fragment: 64 lanes x 16 bytes
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    char* const ldsX = lds;                          // [example][S/32 tiles][32 rows x 64 bytes]
    char* const ldsU = lds + SKF_EX * XBYTES;        // [example][factor 8][half 2] fragments

    int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, g = lane >> 5;
    const int ng = wave & 3, eh = wave >> 2;    // stage 2: channel group and pair of examples

    // ---- stage-1 B fragments: column t = r of Z_wave, rows in the fragment order (prepared); read once
    bf16x8 zf[KS];
    auto load_z = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            zf[ks] = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
            if (wave < k) zf[ks] = *(const bf16x8*)(zt + ((int64_t)wave * SKF_T + r) * S + 16 * ks + 8 * g);
        }
        asm volatile("" ::: "memory");
    };
    // transposing reads of an X tile: see the V^T reads of the attention kernels
    const int xrd = L::v_offset(4 * g + ((lane & 15) >> 2), (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2);

    // ---- X transport: wave e < 4 sends the block of example e straight into LDS (buffer-load-to-LDS, 16 rows of 64
    // bytes per instruction; 32-channel rows need no swizzle).  The loads are issued right after stage 1 has read the
    // old blocks, by the four waves that the SIMDs favour anyway (the older wave of each SIMD finishes stage 2 with
    // time to spare), and no registers carry them.
    const uint32_t x_voff = (uint32_t)(lane >> 2) * (uint32_t)(D * 2) + (lane & 3) * 16;
    const uint32_t ldsX0 = lds_address(ldsX);
    auto send_x = [&](int64_t group, int cb) {
        if (wave >= SKF_EX) return;
        int64_t b = group * SKF_EX + wave;
        b = b < B ? b : B - 1;  // (a missing example re-reads the last one; its results are never stored)
        u32x4 rsrc = make_rsrc_words(x + (b * S) * D + cb * SKF_CB, (uint32_t)(S - 1) * (D * 2) + SKF_CB * 2);
#pragma unroll
        for (int q = 0; q < 4; ++q) rsrc[q] = __builtin_amdgcn_readfirstlane(rsrc[q]);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ldsX0 + wave * XBYTES);
#pragma unroll
        for (int j = 0; j < S / 16; ++j) load_to_lds_b128(rsrc, x_voff, (uint32_t)j * 16 * (D * 2), dst + j * 1024);
    };

    const int64_t n_groups = ((int64_t)B + SKF_EX - 1) / SKF_EX;
    int64_t group = SPLIT ? blockIdx.x % n_groups : blockIdx.x;
    if (group >= n_groups) return;
    const int range = SPLIT ? (int)(blockIdx.x / n_groups) : 0;
    const int cb_first = SPLIT ? range * blocks_per_range : 0, cb_end = SPLIT ? cb_first + blocks_per_range : NCB;
    send_x(group, cb_first);
    load_z();
    wait_vmcnt<0>();
    // W fragments travel three fragment steps ahead of their use in a ring of four register sets that runs on from
    // one step into the next (W does not depend on the group): the first three steps of all
    const int kp = (k + 1) & ~1;                                  // factors rounded up to whole pairs
    constexpr int64_t wfactor = (int64_t)D * D;                   // values per factor
    constexpr int64_t wblock = (int64_t)(D / 32) * 2 * 512;       // values per channel block of a factor
    const bf16_t* const wlane = wp + (int64_t)NBW * ng * 2 * 512 + lane * 8;
    bf16x8 wq[4][NBW];
    auto issue = [&](int cb, int i, int cc, bf16x8 (&dst)[NBW]) {
        // factor i of block cb; i >= kp: factor i - kp of the next block (past the last real factor: it once more, unused)
        const bool next = i >= kp;
        int ii = next ? i - kp : i;
        ii = ii < k ? ii : k - 1;
        const int cbb = next ? (cb + 1 < cb_end ? cb + 1 : cb_first) : cb;
        const bf16_t* src = wlane + cbb * wblock + ii * wfactor + cc * 512;
#pragma unroll
        for (int j = 0; j < NBW; ++j) dst[j] = *(const bf16x8*)(src + j * 2 * 512);
        asm volatile("" ::: "memory");
    };
    issue(cb_first, 0, 0, wq[0]);
    issue(cb_first, 0, 1, wq[1]);
    issue(cb_first, 1, 0, wq[2]);
    for (; group < n_groups; group += SPLIT ? n_groups : gridDim.x) {
        f32x16 yacc[2][NBW];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int j = 0; j < NBW; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) yacc[e][j][v] = 0.f;
        for (int cb = cb_first; cb < cb_end; ++cb) {
            __syncthreads();  // (A) this step's X blocks are in LDS; the exchange buffer is free
            // ---- stage 1: U^T_{e, wave} of the block, example by example.  Every MFMA needs a fresh A fragment from LDS:
            // the fragments are requested four MFMAs ahead (left to the compiler they were read one at a time, each
            // MFMA behind the full latency of its own read)
            if (wave < k) {
                constexpr int AHEAD = 4, TOTAL = SKF_EX * KS;
                bf16x8 af[AHEAD];
                auto read_a = [&](int idx, bf16x8& dst) {
                    const int e = idx / KS, ks = idx % KS;
                    const char* src = ldsX + e * XBYTES + (ks >> 1) * L::TILE_BYTES + (ks & 1) * 16 * L::ROW_BYTES + xrd;
                    const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, src));
                    const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, src + 8 * L::ROW_BYTES));
                    typedef __attribute__((ext_vector_type(8))) short s16x8;
                    dst = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
                    asm volatile("" ::: "memory");
                };
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) read_a(q, af[q]);
                f32x16 uacc;
#pragma unroll
                for (int idx = 0; idx < TOTAL; ++idx) {
                    const int e = idx / KS, ks = idx % KS;
                    if (ks == 0) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) uacc[v] = 0.f;
                    }
                    const bf16x8 a = af[idx % AHEAD];
                    if (idx + AHEAD < TOTAL) read_a(idx + AHEAD, af[idx % AHEAD]);
                    uacc = mfma32(a, zf[ks], uacc);
                    if (ks == KS - 1) {
#pragma unroll
                        for (int cc = 0; cc < 2; ++cc) {
                            bf16x8 pk;
#pragma unroll
                            for (int q = 0; q < 8; ++q) pk[q] = (bf16_t)uacc[8 * cc + q];
                            *(bf16x8*)(ldsU + (((e * 8 + wave) * 2 + cc) * FRAG) + lane * 16) = pk;
                        }
                    }
                }
            }
            __syncthreads();  // (B) every U^T fragment of the step is in the exchange buffer; the X blocks are dead
            {   // the next step's blocks set out
                const bool same = cb + 1 < cb_end;
                const int64_t ng_ = same ? group : group + (SPLIT ? n_groups : gridDim.x);
                if (ng_ < n_groups) send_x(ng_, same ? cb + 1 : 0);
            }
            // ---- stage 2: Y^T_e[channels of group ng] += W_i^T[.., block] U^T_{e, i} over all factors, e = 2 eh, 2 eh + 1.  A
            // factor has two fragment steps cc (halves of the block) of NBW W fragments each; the fragments travel three
            // steps ahead of their use in a ring of four register sets, and the empty statements keep the compiler from
            // sinking the loads to their use (it would then wait for every single one).  The Z fragments of the next
            // stage 1 are requested behind the last factor, the X blocks of the step after the next at the very end.
            {
                // the U^T fragments of both examples for step (i, cc): requested one step ahead of their use
                bf16x8 ubq[2][2];
                auto fetch_u = [&](int i, int cc, bf16x8 (&dst)[2]) {
                    i = i < k ? i : k - 1;
                    dst[0] = *(const bf16x8*)(ldsU + ((((2 * eh) * 8 + i) * 2 + cc) * FRAG) + lane * 16);
                    dst[1] = *(const bf16x8*)(ldsU + ((((2 * eh + 1) * 8 + i) * 2 + cc) * FRAG) + lane * 16);
                };
                auto compute = [&](const bf16x8 (&ub)[2], const bf16x8 (&wa)[NBW]) {
#pragma unroll
                    for (int j = 0; j < NBW; ++j) {
                        yacc[0][j] = mfma32(wa[j], ub[0], yacc[0][j]);
                        yacc[1][j] = mfma32(wa[j], ub[1], yacc[1][j]);
                    }
                };
                fetch_u(0, 0, ubq[0]);
                for (int i0 = 0; i0 < k; i0 += 2) {
                    const bool two = i0 + 1 < k;
                    issue(cb, i0 + 1, 1, wq[3]);
                    fetch_u(i0, 1, ubq[1]);
                    compute(ubq[0], wq[0]);
                    issue(cb, i0 + 2, 0, wq[0]);
                    fetch_u(i0 + 1, 0, ubq[0]);
                    compute(ubq[1], wq[1]);
                    issue(cb, i0 + 2, 1, wq[1]);
                    fetch_u(i0 + 1, 1, ubq[1]);
                    if (two) compute(ubq[0], wq[2]);
                    issue(cb, i0 + 3, 0, wq[2]);
                    fetch_u(i0 + 2, 0, ubq[0]);
                    if (two) compute(ubq[1], wq[3]);
                }
            }
            // the X blocks have landed: they are older than every W fragment, and at most the three fragment steps
            // requested for the next block are still on their way
            wait_vmcnt<3 * NBW>();
        }
        // ---- output: lane holds column t = r of Y^T, rows n = 32*(NBW*ng + j) + 8*(v/4) + 4g + v%4
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int64_t b = group * SKF_EX + 2 * eh + e;
            if (SPLIT && b < B) {
                float* prow = part + (((int64_t)range * B + b) * SKF_T + r) * D + 32 * NBW * ng + 4 * g;
#pragma unroll
                for (int j = 0; j < NBW; ++j)
#pragma unroll
                    for (int vg = 0; vg < 4; ++vg) {
                        f32x4 out;
#pragma unroll
                        for (int q = 0; q < 4; ++q) out[q] = yacc[e][j][4 * vg + q];
                        *(f32x4*)(prow + 32 * j + 8 * vg) = out;
                    }
            } else if (b < B) {
                bf16_t* yrow = y + (b * SKF_T + r) * D + 32 * NBW * ng + 4 * g;
#pragma unroll
                for (int j = 0; j < NBW; ++j)
#pragma unroll
                    for (int vg = 0; vg < 4; ++vg) {
                        bf16x4 out;
#pragma unroll
                        for (int q = 0; q < 4; ++q) out[q] = (bf16_t)yacc[e][j][4 * vg + q];
                        *(bf16x4*)(yrow + 32 * j + 8 * vg) = out;
                    }
            }
        }
    }
}

// y[idx] = sum of part[range][idx] over the ranges, in order, rounded once; four values per thread
__global__ __launch_bounds__(256) void skf_sum_kernel(const float* __restrict__ part, bf16_t* __restrict__ y, int ranges, int64_t n) {
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (idx >= n) return;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < ranges; ++s) sum += *(const f32x4*)(part + (int64_t)s * n + idx);
    bf16x4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = (bf16_t)sum[q];
    *(bf16x4*)(y + idx) = o;
}

// Ranges of channel blocks: as many as fill the compute units, a divisor of D / 32.  `room`: bytes for the partial sums.
// One group takes 95 to 110 us on its compute unit however small the batch.  Forward and backward at S = 256, D = 384, k = 8,
// whole / split, us: 8 examples 139 / 68, 64: 154 / 95, 128: 182 / 120, 256: 240 / 187, 512: 341 / 318, 700: 415 / 412 (one range).
constexpr int SKF_WGS = 256;  // workgroups of a split launch, at most
static int skf_ranges(int B, int D, size_t room) {
    const int groups = (B + SKF_EX - 1) / SKF_EX, blocks = D / SKF_CB;
    int ranges = 1;
    for (int d = 2; d <= blocks; ++d)
        if (blocks % d == 0 && (int64_t)groups * d <= SKF_WGS && (size_t)d * B * SKF_T * D * sizeof(float) <= room) ranges = d;
    return ranges;
}

bool sumkron_fused_supported(int S, int T, int D, int k, int dtype) {
    return dtype == KUNLUN_BF16 && T == SKF_T && (S == 128 || S == 256) && D % 128 == 0 && D >= 128 && D <= 384 && k >= 1 && k <= SKF_WAVES;
}

size_t sumkron_fused_need(int S, int T, int D, int k) {
    return align_up((size_t)k * T * S * 2, 256) + align_up((size_t)k * D * D * 2, 256);
}
// ... with the partial sums of this batch
size_t sumkron_fused_batch_bytes(int B, int S, int T, int D, int k) {
    const int ranges = skf_ranges(B, D, ~(size_t)0);
    return sumkron_fused_need(S, T, D, k) + (ranges > 1 ? (size_t)ranges * B * SKF_T * D * sizeof(float) : 0);
}
// ... with the partial sums of any split launch (the same for every batch size, so that a kept workspace serves them all)
size_t sumkron_fused_workspace(int S, int T, int D, int k) {
    return sumkron_fused_need(S, T, D, k) + (size_t)SKF_WGS * SKF_EX * SKF_T * D * sizeof(float);
}

template <int NBW, int S, bool SPLIT>
static hipError_t launch_skf_form(const bf16_t* x, const bf16_t* zt, const bf16_t* wp, bf16_t* y, int B, int k, float* part, int ranges,
                                  hipStream_t stream) {
    constexpr int bytes = SKF_EX * S * SKF_CB * 2 + SKF_EX * 8 * 2 * 1024;
    auto kern = sumkron_fused_kernel<NBW, S, SPLIT>;
    // once per process (thread-safe initialisation of a function-local static); not a stream operation
    static const hipError_t raised = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (raised != hipSuccess) return raised;
    const int64_t n_groups = ((int64_t)B + SKF_EX - 1) / SKF_EX;
    const int64_t resident = compute_units();
    const int64_t grid = SPLIT ? n_groups * ranges : n_groups < resident ? n_groups : resident;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * SKF_WAVES), bytes, stream, x, zt, wp, y, B, k, part, 128 * NBW / SKF_CB / ranges);
    return hipGetLastError();
}
template <int NBW, int S>
static hipError_t launch_skf(const bf16_t* x, const bf16_t* zt, const bf16_t* wp, bf16_t* y, int B, int k, float* part, size_t room, hipStream_t stream) {
    const int ranges = skf_ranges(B, 128 * NBW, room);
    if (ranges == 1) return launch_skf_form<NBW, S, false>(x, zt, wp, y, B, k, nullptr, 1, stream);
    const hipError_t e = launch_skf_form<NBW, S, true>(x, zt, wp, y, B, k, part, ranges, stream);
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)B * SKF_T * 128 * NBW;
    hipLaunchKernelGGL(skf_sum_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, stream, part, y, ranges, n);
    return hipGetLastError();
}

// workspace: prepared Z, prepared W, and what is left of its bytes (at least sumkron_fused_need()) for partial sums
hipError_t launch_sumkron_fused(const void* x, const void* z, const void* w, void* y, int B, int S, int T, int D, int k, void* workspace,
                                size_t workspace_bytes, hipStream_t stream) {
    bf16_t* zt = (bf16_t*)workspace;
    bf16_t* wp = (bf16_t*)((char*)workspace + align_up((size_t)k * T * S * 2, 256));
    const int64_t nz = (int64_t)k * S * T, nw = (int64_t)k * D * D;
    const int w_blocks = (int)((nw / 8 + 255) / 256);
    hipLaunchKernelGGL(skf_prepare_kernel, dim3((unsigned)(w_blocks + (nz / 8 + 255) / 256)), dim3(256), 0, stream, (const bf16_t*)w, (const bf16_t*)z,
                       wp, zt, k, D, S, T, w_blocks);
    const size_t used = sumkron_fused_need(S, T, D, k), room = workspace_bytes > used ? workspace_bytes - used : 0;
    float* part = (float*)((char*)workspace + used);
    const bf16_t* xb = (const bf16_t*)x;
    bf16_t* yb = (bf16_t*)y;
    const int nbw = D / 128;
#define KUNLUN_SKF(NBW_) (S == 256 ? launch_skf<NBW_, 256>(xb, zt, wp, yb, B, k, part, room, stream) : launch_skf<NBW_, 128>(xb, zt, wp, yb, B, k, part, room, stream))
    switch (nbw) {
    case 1: return KUNLUN_SKF(1);
    case 2: return KUNLUN_SKF(2);
    default: return KUNLUN_SKF(3);  // (D = 512 does not fit the registers of a wave: the two-GEMM path takes it)
    }
#undef KUNLUN_SKF
}

}  // namespace kunlun
