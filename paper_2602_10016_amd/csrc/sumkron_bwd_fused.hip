// SumKronLinear backward (chain rule on Eq. (SumKronLinear)) in two kernels, for T = 32 output tokens, S in {128, 256}
// rows, D in {128, 256, 384} channels and k <= 8 factors.  With U_{b,i} = Z_i^T X_b and G_{b,i} = dY_b W_i^T (each
// computed once and rounded to bf16; 200 MB each at B = 1024, S = 256, D = 384, k = 8):
//     dX_b = sum_i Z_i G_{b,i},      dW_i = sum_b U_{b,i}^T dY_b,      dZ_i = sum_b X_b G_{b,i}^T.
//
// sumkron_gx_kernel: G and dX.  A workgroup of 8 wavefronts (one per compute unit) takes four examples, whose dY stays
// in LDS, through blocks of 32 channels c of X:
//     stage 1:  G^T[c, t] of (factor, example): W fragments straight from L2, laid out in fragment order once per call
//               (each serves all the examples of the wave), dY rows from LDS; the packed tiles go to memory in the order
//               in which the second kernel wants them, and as [t][c] images to LDS
//     stage 2:  dX^T[c, s] = sum over (i, t): images read transposed, Z_i rows in registers (16 fragments, the wave's
//               block of 32 rows s); a lane ends up with one row s and stores 16 bytes of it at a time
// Both stages run between the same two barriers (stage 2 of a block, stage 1 of the next), so waves drift apart and
// overlap them.
//
// sumkron_batch_grads_kernel: the sums over the batch.  A workgroup owns two factors (i, i + 1; four waves each) and a
// block of 64 channels c of X, and walks a range of examples; its parts of dW ([2][64][D]) and dZ ([2][S][32], over its
// channels) stay in fp32 accumulators for the whole range and leave once, as partial sums that are added in a fixed order.
// Per example, X_b[:, block] (S x 64), dY_b (32 x D) and the two G_{b,i}[:, block] (32 x 64) come by buffer-load-to-LDS
// into one of two buffers, an example ahead; then, for the wave's factor i and q = wave % 4:
//     phase 1:  U[t, c] for the 16 channels 16q..  (16x16x32 matrix instructions: Z_i^T fragments in registers, X
//               read transposed) -> bf16 exchange image [c][t] in LDS;
//               dZ rows of the S/4 rows of X that begin at q S/4: X rows and G fragments as stored
//     phase 2:  dW[64 channels, n block q of D/4] += U^T dY: U from the image, dY read transposed
// Workgroups that share X and dY rows (same examples and channels, other factors) run on one XCD.
// Measured at B = 1024, S = 256, D = 384, k = 8: 140 us (128 GFLOP) and 215 to 244 us (180 GFLOP), clocks at 2.0-2.1 GHz, in
// place of five GEMMs with U and G through HBM (100 + 121 + 100 + 147 + 134 us).  What bounds them: the writes of G and
// dX (400 MB: without the stores of dX the pair takes 55 us less; pairs of blocks stored as whole 128-byte lines, or
// non-temporal: no change); in the second kernel LDS, 328 KB per example = 2560 cycles against 1792 cycles of matrix
// instructions, and the two barriers between them (4300 cycles pass; without its loads 45 us less).
#include "lds_ring.h"

#define PIN() __builtin_amdgcn_sched_barrier(0)  // nothing is moved across by the instruction scheduler

namespace kunlun {

constexpr int SKB_T = 32;
constexpr int SKB_C = 64;  // channels per workgroup

template <int NB, int S>  // D = 128 * NB
struct SkbSmem {
    static constexpr int D = 128 * NB;
    static constexpr int X_BYTES = S * SKB_C * 2;
    static constexpr int DY_BYTES = SKB_T * D * 2;
    static constexpr int G_TILE = SKB_T * SKB_C * 2;
    static constexpr int BUF = X_BYTES + DY_BYTES + 2 * G_TILE;
    static constexpr int U_IMAGE = SKB_C * SKB_T * 2;  // [c][t] bf16, 64-byte rows
    static constexpr int TOTAL = 2 * BUF + 2 * U_IMAGE;  // 136 KB at S = 256, D = 384
};

// rows of 64 bytes, 16-byte chunk swizzled by the row
__device__ __forceinline__ int skb_u_offset(int row, int byte_in_row) {
    return row * 64 + ((((byte_in_row >> 4) ^ (row >> 2)) & 3) << 4) + (byte_in_row & 15);
}
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// channel of row m of a 32-row tile of G^T: in the C layout a lane half then holds 8 consecutive channels per 8 registers
__host__ __device__ inline int skb_channel(int m) { return (m & 16) + 8 * ((m >> 2) & 1) + 4 * ((m >> 3) & 1) + (m & 3); }

// Once per call.  W fragment (i, channel block cb of 32, contraction step kn of 16): lane (r, g) holds
// w[i][32 cb + channel(r)][16 kn + 8 g ..]: 1 KB contiguous per fragment.  zt[(i*32 + t)*S + s] = z[(i*S + s)*32 + t].
__global__ __launch_bounds__(256) void skb_prepare_kernel(const bf16_t* __restrict__ w, const bf16_t* __restrict__ z, bf16_t* __restrict__ wf,
                                                          bf16_t* __restrict__ zt, int k, int D, int S, int w_blocks) {
    if ((int)blockIdx.x < w_blocks) {
        const int idx = blockIdx.x * 256 + threadIdx.x;  // 8 values each
        if (idx >= k * D * (D / 8)) return;
        const int lane = idx & 63, frag = idx >> 6;      // (i * D/32 + cb) * D/16 + kn
        const int kn = frag % (D / 16), rest = frag / (D / 16);
        const int cb = rest % (D / 32), i = rest / (D / 32);
        const int c = 32 * cb + skb_channel(lane & 31), n = 16 * kn + 8 * (lane >> 5);
        *(u32x4*)(wf + (int64_t)idx * 8) = *(const u32x4*)(w + ((int64_t)i * D + c) * D + n);
    } else {
        const int idx = (blockIdx.x - w_blocks) * 256 + threadIdx.x;
        if (idx >= k * S * SKB_T) return;
        const int s = idx % S, t = (idx / S) % SKB_T, i = idx / (S * SKB_T);
        zt[idx] = z[((int64_t)i * S + s) * SKB_T + t];
    }
}

constexpr int SKX_EX = 4;  // examples per workgroup

// gf: G in fragment order, fragment (b, c / 64, i, (c / 16) % 4): lane (t, g) holds channels 16 (c / 16) + 8 g ..
// EXW: examples per wave in stage 1, 4 for k > 4 (a wave per factor), 2 for k in {3, 4}, 1 for k <= 2.
template <int NB, int S, int EXW>
__global__ __launch_bounds__(512, 2) void sumkron_gx_kernel(const bf16_t* __restrict__ z, const bf16_t* __restrict__ wf,
                                                            const bf16_t* __restrict__ dy, bf16_t* __restrict__ gf,
                                                            bf16_t* __restrict__ dx, int B, int k, int cb_per_wg) {
    constexpr int D = 128 * NB;
    constexpr int NCB = D / 32;
    constexpr int KN = D / 16;                       // contraction steps of stage 1
    constexpr int DY_BYTES = SKB_T * D * 2;          // one example
    constexpr int IMAGE = SKB_T * 64;                // [t][32 channels]
    constexpr int EX2 = S == 256 ? SKX_EX : SKX_EX / 2;  // examples per wave in stage 2
    using LY = TileLayout<128>;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, g = lane >> 5, s16 = lane & 15, hi16 = (lane >> 4) & 1;
    const int splits = NCB / cb_per_wg;
    const int b0 = (int)(blockIdx.x / splits) * SKX_EX;
    const int cb0 = (int)(blockIdx.x % splits) * cb_per_wg;
    const uint32_t lds0 = lds_address(smem);
    const uint32_t images = lds0 + SKX_EX * DY_BYTES;  // [example][factor]

    // ---- dY of the four examples (past the batch: the last one again; never stored)
    TileDma<128, 8, SWZ_K> ydma;
    ydma.init(lane, wave, D * 2);
#pragma unroll
    for (int e = 0; e < SKX_EX; ++e) {
        const int b = b0 + e < B ? b0 + e : B - 1;
#pragma unroll
        for (int t = 0; t < NB; ++t)
            ydma.issue((const char*)(dy + (int64_t)b * SKB_T * D + 128 * t), KT, lds0 + e * DY_BYTES + t * LY::TILE_BYTES);
    }
    // ---- stage 1 work of this wave: factor fi, examples fe ..
    const int fi = wave * EXW / SKX_EX, fe = wave * EXW % SKX_EX;
    const bool busy = fi < k;
    // ---- stage 2 work: rows 32 sb .., examples se ..; Z_i rows as B operands: column s = r, contraction t = 16 j + 8 g ..
    const int sb = S == 256 ? wave : (wave & 3), se = S == 256 ? 0 : (wave >> 2) * EX2;
    bf16x8 zf[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            zf[i][j] = *(const bf16x8*)(z + ((int64_t)(i < k ? i : k - 1) * S + 32 * sb + r) * SKB_T + 16 * j + 8 * g);
    const int y_rd = LY::k_offset(r, g);   // dY row fragment: row t = r, n = 16 kn + 8 g .. -> tile kn / 8, ^ ((kn % 8) << 5)
    const int iw0 = skb_u_offset(r, 16 * g), iw1 = skb_u_offset(r, 32 + 16 * g);  // image writes: row t = r, channels 8 g .., 16 + 8 g ..
    // image reads (A operand: row m, contraction t): rows 16 j + 8 g + 0..3 / + 4..7, columns channel(m): groups of four
    // columns in the order 0, 2, 1, 3
    const int col = 16 * hi16 + 8 * (s16 & 1) + 4 * ((s16 >> 1) & 1);
    const int irA = skb_u_offset(8 * g + (s16 >> 2), col * 2), irB = skb_u_offset(8 * g + 4 + (s16 >> 2), col * 2);
    auto tr_read = [](uint32_t a, uint32_t b) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)b);
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    constexpr int WA = 6, YA = 4;  // W fragments (L2) and dY fragments (LDS) in flight
    bf16x8 packed[EXW][2], wr[WA];
    auto w_src = [&](int cb) { return (const bf16x8*)(wf + ((int64_t)fi * NCB + cb) * KN * 512) + lane; };
    // the first fragments of a block are requested ahead of the stores of the block before: a wait for a load also
    // waits for every older store
    auto request = [&](int cb) {
        const bf16x8* wsrc = w_src(cb);
#pragma unroll
        for (int kn = 0; kn < WA; ++kn) wr[kn] = wsrc[kn * 64];
    };
    auto stage1 = [&](int cb) {
        const bf16x8* wsrc = w_src(cb);
        f32x16 acc[EXW];
        bf16x8 yr[YA];
        auto y_frag = [&](int j) {  // j = kn * EXW + e
            const int kn = j / EXW, e = j % EXW;
            return *(const __attribute__((address_space(3))) bf16x8*)(lds0 + (fe + e) * DY_BYTES + (kn / 8) * LY::TILE_BYTES + (y_rd ^ ((kn & 7) << 5)));
        };
#pragma unroll
        for (int j = 0; j < YA; ++j) yr[j] = y_frag(j);
        PIN();
#pragma unroll
        for (int j = 0; j < KN * EXW; ++j) {
            const int kn = j / EXW, e = j % EXW;
            acc[e] = mfma32(wr[kn % WA], yr[j % YA], kn == 0 ? zero16 : acc[e]);
            if (j + YA < KN * EXW) yr[j % YA] = y_frag(j + YA);
            if (e == EXW - 1 && kn + WA < KN) wr[kn % WA] = wsrc[(kn + WA) * 64];
            PIN();
        }
#pragma unroll
        for (int e = 0; e < EXW; ++e)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 8; ++v) packed[e][h][v] = (bf16_t)acc[e][8 * h + v];
    };
    wait_vmcnt<0>();
    __syncthreads();  // dY is complete
    if (busy) {
        request(cb0);
        stage1(cb0);
    }
    for (int cb = cb0; cb < cb0 + cb_per_wg; ++cb) {
        __syncthreads();  // every wave is done with the images of the block before
        if (busy) {
            if (cb + 1 < cb0 + cb_per_wg) request(cb + 1);
            PIN();
#pragma unroll
            for (int e = 0; e < EXW; ++e) {
                const uint32_t im = images + ((fe + e) * 8 + fi) * IMAGE;
                *(__attribute__((address_space(3))) bf16x8*)(im + iw0) = packed[e][0];
                *(__attribute__((address_space(3))) bf16x8*)(im + iw1) = packed[e][1];
                if (b0 + fe + e < B) {
                    bf16x8* out = (bf16x8*)(gf + ((((int64_t)(b0 + fe + e) * (D / SKB_C) + cb / 2) * k + fi) * 4 + 2 * (cb & 1)) * 512) + lane;
                    out[0] = packed[e][0];
                    out[64] = packed[e][1];
                }
            }
        }
        __syncthreads();  // the images are complete
        // ---- stage 2
#pragma unroll
        for (int e = 0; e < EX2; ++e) {
            f32x16 acc = zero16;
            const uint32_t im = images + (se + e) * 8 * IMAGE;
            bf16x8 af[4];
            auto a_frag = [&](int j) { return tr_read(im + (j >> 1) * IMAGE + irA + (j & 1) * 16 * 64, im + (j >> 1) * IMAGE + irB + (j & 1) * 16 * 64); };
#pragma unroll
            for (int j = 0; j < 4; ++j) af[j] = a_frag(j);
            PIN();
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if ((j >> 1) < k) acc = mfma32(af[j & 3], zf[j >> 1][j & 1], acc);
                if (j + 4 < 16) af[j & 3] = a_frag(j + 4);
                PIN();
            }
            bf16x8 o[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 8; ++v) o[h][v] = (bf16_t)acc[8 * h + v];
            if (b0 + se + e < B) {
                bf16_t* row = dx + ((int64_t)(b0 + se + e) * S + 32 * sb + r) * D + 32 * cb + 8 * g;
                *(bf16x8*)row = o[0];
                *(bf16x8*)(row + 16) = o[1];
            }
        }
        if (busy && cb + 1 < cb0 + cb_per_wg) stage1(cb + 1);
    }
}

// zt: Z_i^T rows, zt[(i*32 + t)*S + s].  dw_part: [split][k*D][D]; dz_part: [split][D/64][k*S][32].
template <int NB, int S>
__global__ __launch_bounds__(512, 2) void sumkron_batch_grads_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ zt,
                                                                     const bf16_t* __restrict__ dy, const bf16_t* __restrict__ gf,
                                                                     float* __restrict__ dw_part, float* __restrict__ dz_part, int B,
                                                                     int k, int splits, int per_split) {
    using SM = SkbSmem<NB, S>;
    constexpr int D = SM::D;
    constexpr int NCB = D / SKB_C;
    constexpr int KSU = S / 32;     // contraction steps of U (32 rows of X each)
    constexpr int SB = S / 128;     // 32-row blocks of dZ per wave
    using LX = TileLayout<64>;      // X and G tiles: 32 rows of 64 channels
    using LY = TileLayout<128>;     // dY tiles: 32 rows of 128 channels
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave >> 2, q = wave & 3;
    const int r = lane & 31, g = lane >> 5, r16 = lane & 15, g4 = lane >> 4;

    // workgroup -> (group = (split, channel block), pair of factors); a group's pairs follow each other on one XCD
    const int n_pairs = (k + 1) / 2;
    const int slot = blockIdx.x >> 3;
    const int group = (slot / n_pairs) * 8 + (blockIdx.x & 7);
    if (group >= splits * NCB) return;
    const int split = group / NCB, cb = group % NCB;
    const int i0 = (slot % n_pairs) * 2;
    const bool mine = i0 + half < k;          // an odd factor count leaves the second half of the last pair idle
    const int i = mine ? i0 + half : i0;      // (it computes the first factor again and stores nothing)
    const int b0 = split * per_split, b1 = b0 + per_split < B ? b0 + per_split : B;

    const uint32_t lds0 = lds_address(smem);
    const uint32_t image = lds0 + 2 * SM::BUF + half * SM::U_IMAGE;
    const int64_t kD = (int64_t)k * D;

    // ---- transport: X tiles by 8 / (S/32) waves each, dY tiles by all eight, the factor's G tile by its four waves
    constexpr int WX = 8 / (S / 32);
    TileDma<64, WX, SWZ_U> xdma;
    TileDma<128, 8, SWZ_V> ydma;
    xdma.init(lane, wave % WX, D * 2);
    ydma.init(lane, wave, D * 2);
    auto issue = [&](int b, int buf) {
        const uint32_t dst = lds0 + buf * SM::BUF;
        const int xt = wave / WX;
        xdma.issue((const char*)(x + ((int64_t)b * S + 32 * xt) * D + cb * SKB_C), KT, dst + xt * LX::TILE_BYTES);
#pragma unroll
        for (int t = 0; t < NB; ++t)
            ydma.issue((const char*)(dy + (int64_t)b * SKB_T * D + 128 * t), KT, dst + SM::X_BYTES + t * LY::TILE_BYTES);
        u32x4 grsrc = make_rsrc_words(gf + ((((int64_t)b * NCB + cb) * k + i) * 4 + q) * 512, 1024);
#pragma unroll
        for (int j = 0; j < 4; ++j) grsrc[j] = __builtin_amdgcn_readfirstlane(grsrc[j]);
        load_to_lds_b128(grsrc, lane * 16, 0, __builtin_amdgcn_readfirstlane(dst + SM::X_BYTES + SM::DY_BYTES + half * SM::G_TILE + q * 1024));
    };
    if (b0 < b1) issue(b0, 0);

    // Z_i^T fragments (A operands of 16x16x32): row t = 16 th + r16, contraction s = 32 ks + 8 g4 ..
    bf16x8 zf[KSU][2];
#pragma unroll
    for (int ks = 0; ks < KSU; ++ks)
#pragma unroll
        for (int th = 0; th < 2; ++th)
            zf[ks][th] = *(const bf16x8*)(zt + ((int64_t)i * SKB_T + 16 * th + r16) * S + 32 * ks + 8 * g4);

    f32x16 dw[2][NB], dz[SB];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) dw[c][n][v] = 0.f;
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 16; ++v) dz[sb][v] = 0.f;

    // ---- LDS offsets of this lane
    const int s16 = lane & 15, hi16 = (lane >> 4) & 1;
    // U, B operand from X tile ks: rows 8 g4 + 0..3 / + 4..7, channels 16 q + r16
    const int xuA = LX::u_offset(8 * g4 + (s16 >> 2), (16 * q + 4 * (s16 & 3)) * 2);
    const int xuB = LX::u_offset(8 * g4 + 4 + (s16 >> 2), (16 * q + 4 * (s16 & 3)) * 2);
    // dZ, A operand: row r of X block q SB + sb, channels 16 kc + 8 g ..; B operand: G fragment kc, the same channels
    int xr = q * SB * LX::TILE_BYTES + LX::u_offset(r, 16 * g);
    const int gr = SM::X_BYTES + SM::DY_BYTES + half * SM::G_TILE + lane * 16;
    // dW, A operand: image row c = 32 cc + r, t = 16 j + 8 g ..
    int ur = skb_u_offset(r, 16 * g);
    // dW, B operand from dY: rows t = 16 j + 8 g + 0..3 / + 4..7, channel block n = q NB + nb of 32
    const int yrow = 8 * g + (s16 >> 2), ycol = 16 * hi16 + 4 * (s16 & 3);
    int yA[NB], yB[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = 32 * (q * NB + nb);
        yA[nb] = SM::X_BYTES + (n / 128) * LY::TILE_BYTES + LY::v_offset(yrow, (n % 128 + ycol) * 2);
        yB[nb] = SM::X_BYTES + (n / 128) * LY::TILE_BYTES + LY::v_offset(yrow + 4, (n % 128 + ycol) * 2);
    }
    // image writes: U[t = 16 th + 4 g4 + 0..3, c = 16 q + r16] -> row c
    const int uw0 = skb_u_offset(16 * q + r16, 8 * g4), uw1 = skb_u_offset(16 * q + r16, 32 + 8 * g4);
    auto row_read = [](uint32_t a) { return *(const __attribute__((address_space(3))) bf16x8*)a; };
    auto tr_read = [](uint32_t a, uint32_t b) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)b);
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    for (int b = b0; b < b1; ++b) {
        const int buf = (b - b0) & 1;
        const uint32_t base = lds0 + buf * SM::BUF;
        wait_vmcnt<0>();
        __syncthreads();  // the example's tiles are complete; every wave is done with the other buffer and the image
        if (b + 1 < b1) issue(b + 1, buf ^ 1);
        // The order of the LDS reads and matrix instructions is pinned: fragments are read a few instructions ahead of
        // their use, those of the next step behind the last instructions of the one before.
        auto x_frag = [&](int ks) { return tr_read(base + xuA + ks * LX::TILE_BYTES, base + xuB + ks * LX::TILE_BYTES); };
        auto g_frag = [&](int kc) { return row_read(base + gr + kc * 1024); };
        auto xr_frag = [&](int kc, int sb) { return row_read(base + (xr ^ (kc << 5)) + sb * LX::TILE_BYTES); };
        auto y_frag = [&](int j, int nb) { return tr_read(base + yA[nb] + j * 16 * LY::ROW_BYTES, base + yB[nb] + j * 16 * LY::ROW_BYTES); };
        auto u_frag = [&](int j, int c) { return row_read(image + (ur ^ (j << 5)) + c * 32 * 64); };
        // ---- U of the wave's 16 channels
        f32x4 u0 = {0.f, 0.f, 0.f, 0.f}, u1 = {0.f, 0.f, 0.f, 0.f};
        bf16x8 xf[3];
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) xf[ks] = x_frag(ks);
        PIN();
        bf16x8 gf[2], xs[2][SB];
#pragma unroll
        for (int ks = 0; ks < KSU; ++ks) {
            u0 = mfma16(zf[ks][0], xf[ks % 3], u0);
            u1 = mfma16(zf[ks][1], xf[ks % 3], u1);
            if (ks + 3 < KSU) xf[ks % 3] = x_frag(ks + 3);
            if (ks == KSU - 1) {  // the first step of dZ
                gf[0] = g_frag(0);
#pragma unroll
                for (int sb = 0; sb < SB; ++sb) xs[0][sb] = xr_frag(0, sb);
            }
            PIN();
        }
        bf16x4 p0, p1;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p0[e] = (bf16_t)u0[e]; p1[e] = (bf16_t)u1[e]; }
        *(__attribute__((address_space(3))) bf16x4*)(image + uw0) = p0;
        *(__attribute__((address_space(3))) bf16x4*)(image + uw1) = p1;
        PIN();
        // ---- dZ of the wave's rows of X
        bf16x8 yf[NB];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            if (kc + 1 < 4) {
                gf[(kc + 1) & 1] = g_frag(kc + 1);
#pragma unroll
                for (int sb = 0; sb < SB; ++sb) xs[(kc + 1) & 1][sb] = xr_frag(kc + 1, sb);
            } else {  // the first half of dW's dY fragments
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) yf[nb] = y_frag(0, nb);
            }
            PIN();
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) dz[sb] = mfma32(xs[kc & 1][sb], gf[kc & 1], dz[sb]);
            PIN();
        }
        __syncthreads();  // the images are complete
        // ---- dW of the wave's n block
        bf16x8 uf[4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 2; ++c) uf[2 * j + c] = u_frag(j, c);
        PIN();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                for (int c = 0; c < 2; ++c) dw[c][nb] = mfma32(uf[2 * j + c], yf[nb], dw[c][nb]);
                if (j == 0) yf[nb] = y_frag(1, nb);
                PIN();
            }
    }
    if (!mine) return;
    // ---- partial sums: lane = column (n, or t) r, registers = rows 8 (v / 4) + 4 g + v % 4
    float* pw = dw_part + (int64_t)split * kD * D + ((int64_t)i * D + cb * SKB_C) * D + 32 * q * NB + r;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) pw[(int64_t)(32 * c + c_row(v, g)) * D + 32 * nb] = dw[c][nb][v];
    float* pz = dz_part + ((int64_t)group * k * S + (int64_t)i * S + 32 * q * SB) * SKB_T + r;
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int v = 0; v < 16; ++v) pz[(32 * sb + c_row(v, g)) * SKB_T] = dz[sb][v];
}

// out[idx] = sum over `parts` of partial[part][idx], in order, rounded once; four values per thread.  Both sums in one launch
// (one after the other took 8 us more: the sum for dZ is a chain of reads by few workgroups): the first `z_blocks`
// workgroups add up dZ, the longer chain, the others dW.
struct SumParts {
    const float* partial;
    bf16_t* out;
    int parts;
    int64_t n;
};
__global__ __launch_bounds__(256) void sum_parts_kernel(SumParts dz, SumParts dw, int z_blocks) {
    const bool first = (int)blockIdx.x < z_blocks;
    const SumParts p = first ? dz : dw;
    const int64_t idx = ((int64_t)(blockIdx.x - (first ? 0 : z_blocks)) * 256 + threadIdx.x) * 4;
    if (idx >= p.n) return;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int s = 0; s < p.parts; ++s) sum += *(const f32x4*)(p.partial + (int64_t)s * p.n + idx);
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16_t)sum[e];
    *(bf16x4*)(p.out + idx) = o;
}

bool sumkron_bwd_fused_supported(int S, int T, int D, int k, int dtype) {
    return dtype == KUNLUN_BF16 && T == SKB_T && (S == 128 || S == 256) && (D == 128 || D == 256 || D == 384) && k >= 1 && k <= 8;
}

// Ranges of examples: one workgroup per compute unit, none with fewer than four examples.
static void skb_plan(int B, int D, int k, int& splits, int& per_split) {
    const int pairs = (k + 1) / 2 * (D / SKB_C);
    int want = 256 / pairs;
    if (want > B / 4) want = B / 4;
    if (want < 1) want = 1;
    if (B < 1) { splits = per_split = 1; return; }  // (the workspace query of an empty batch)
    per_split = (B + want - 1) / want;
    splits = (B + per_split - 1) / per_split;
}

struct SkbLayout {
    size_t zt, wf, gf, dw_part, dz_part, total;
};
static SkbLayout skb_layout(int B, int S, int D, int k) {
    int splits, per_split;
    skb_plan(B, D, k, splits, per_split);
    SkbLayout l;
    l.zt = 0;
    l.wf = l.zt + align_up((size_t)k * S * SKB_T * 2, 256);
    l.gf = l.wf + align_up((size_t)k * D * D * 2, 256);
    l.dw_part = l.gf + align_up((size_t)B * SKB_T * k * D * 2, 256);
    l.dz_part = l.dw_part + align_up((size_t)splits * k * D * D * sizeof(float), 256);
    l.total = l.dz_part + align_up((size_t)splits * (D / SKB_C) * k * S * SKB_T * sizeof(float), 256);
    return l;
}
size_t sumkron_bwd_fused_workspace(int B, int S, int D, int k) { return skb_layout(B, S, D, k).total; }

template <int NB, int S, int EXW>
static hipError_t launch_gx(const bf16_t* z, const bf16_t* wf, const bf16_t* dy, bf16_t* gf, bf16_t* dx, int B, int k, hipStream_t stream) {
    constexpr int D = 128 * NB, NCB = D / 32;
    constexpr int bytes = SKX_EX * (SKB_T * D * 2 + 8 * SKB_T * 64);
    auto kern = sumkron_gx_kernel<NB, S, EXW>;
    // once per process (thread-safe initialisation of a function-local static); not a stream operation
    static const hipError_t raised = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (raised != hipSuccess) return raised;
    // small batches: the channel blocks of a group of examples are spread over workgroups (each loads the group's dY)
    const int groups = (B + SKX_EX - 1) / SKX_EX;
    int splits = 1;
    for (int d = 2; d <= NCB; ++d)
        if (NCB % d == 0 && (int64_t)groups * d <= 256) splits = d;
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups * splits)), dim3(512), bytes, stream, z, wf, dy, gf, dx, B, k, NCB / splits);
    return hipGetLastError();
}

template <int NB, int S>
static hipError_t launch_skb(const bf16_t* x, const bf16_t* z, const bf16_t* w, const bf16_t* dy, bf16_t* dx, bf16_t* dz, bf16_t* dw, int B,
                             int k, char* ws, hipStream_t stream) {
    constexpr int D = 128 * NB;
    constexpr int bytes = SkbSmem<NB, S>::TOTAL;
    auto kern = sumkron_batch_grads_kernel<NB, S>;
    if (bytes > 64 * 1024) {
        static const hipError_t raised = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (raised != hipSuccess) return raised;
    }
    const SkbLayout l = skb_layout(B, S, D, k);
    bf16_t *zt = (bf16_t*)(ws + l.zt), *wf = (bf16_t*)(ws + l.wf), *gf = (bf16_t*)(ws + l.gf);
    float *dw_part = (float*)(ws + l.dw_part), *dz_part = (float*)(ws + l.dz_part);
    const int64_t nw = (int64_t)k * D * D, nz = (int64_t)k * S * SKB_T;
    const int w_blocks = (int)((nw / 8 + 255) / 256);
    hipLaunchKernelGGL(skb_prepare_kernel, dim3((unsigned)(w_blocks + (nz + 255) / 256)), dim3(256), 0, stream, w, z, wf, zt, k, D, S, w_blocks);
    const hipError_t e = k > 4   ? launch_gx<NB, S, 4>(z, wf, dy, gf, dx, B, k, stream)
                         : k > 2 ? launch_gx<NB, S, 2>(z, wf, dy, gf, dx, B, k, stream) : launch_gx<NB, S, 1>(z, wf, dy, gf, dx, B, k, stream);
    if (e != hipSuccess) return e;
    int splits, per_split;
    skb_plan(B, D, k, splits, per_split);
    const int groups = splits * (D / SKB_C);
    hipLaunchKernelGGL(kern, dim3((unsigned)((groups + 7) / 8 * 8 * ((k + 1) / 2))), dim3(512), bytes, stream, x, zt, dy, gf, dw_part, dz_part, B, k,
                       splits, per_split);
    const int z_blocks = (int)((nz / 4 + 255) / 256);
    hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)(z_blocks + (nw / 4 + 255) / 256)), dim3(256), 0, stream, SumParts{dz_part, dz, groups, nz},
                       SumParts{dw_part, dw, splits, nw}, z_blocks);
    return hipGetLastError();
}

hipError_t launch_sumkron_bwd_fused(const void* x, const void* z, const void* w, const void* dy, void* dx, void* dz, void* dw, int B, int S,
                                    int D, int k, void* workspace, hipStream_t stream) {
    auto run = [&](auto launch) {
        return launch((const bf16_t*)x, (const bf16_t*)z, (const bf16_t*)w, (const bf16_t*)dy, (bf16_t*)dx, (bf16_t*)dz, (bf16_t*)dw, B, k,
                      (char*)workspace, stream);
    };
    if (S == 256) return D == 384 ? run(launch_skb<3, 256>) : D == 256 ? run(launch_skb<2, 256>) : run(launch_skb<1, 256>);
    return D == 384 ? run(launch_skb<3, 128>) : D == 256 ? run(launch_skb<2, 128>) : run(launch_skb<1, 128>);
}

}  // namespace kunlun
