// One-pass bf16 matrix-core backward for 65..256 queries per example at head dimension 128 (the seed direction
// with many seeds): dQ, dK, dV of <O, dO>, every score computed once.
//
// One workgroup of 8 wavefronts (two per SIMD, the whole register file of a compute unit) = one (example, head) or
// one range of its key tiles.  Per 32-key tile:
//     score phase: wave w owns query block w (32 queries; Q_w^T and dO_w^T fragments live in registers):
//         S^T = K Q_w^T,  dP^T = V dO_w^T,  P_w^T and dS_w^T in registers,  dQ_w^T += K^T dS_w^T  (64 accumulators)
//         bf16 copies of P_w and dS_w go to the tile's [query][key] LDS images
//     gradient phase, one tile later: wave w owns one of the 8 output blocks, dV^T or dK^T of 32 channels:
//         dV^T[block] = dO^T[block] P,   dK^T[block] = Q^T[block] dS,   over all 256 queries;
//         the dO^T / Q^T operand of a block does not change over the key tiles: its 16 fragments stay in registers
// Blocks of 32 queries that an example does not have take no part: their waves compute no scores, and the gradient phase
// skips their share of the contraction (65 queries, H = 8, GELU, 256 histories of 64..256 keys 184 -> 154 us, log-normal
// 915 -> 657 us; the two-pass kernels 157 and 987 us).
// The P / dS images are double-buffered, so the gradient phase of a tile and the score phase of the next lie
// between the same two barriers (one barrier per tile).
// K/V tiles travel by buffer-load-to-LDS through a ring of three stages (lds_ring.h), two tiles ahead.
//
// What bounds it: 256 shared seeds over 256 log-normal histories (H = 8, 71 700 key tiles, 793 GFLOP) take 890 us =
// 890 TFLOP/s, where the vendor GEMM reaches 1160 on this device; the two-pass kernels (attn_bwd_tiled_mfma.hip),
// which serve longer query sequences and compute S and dP twice, took 1640 us.  Per tile and compute unit the 320
// matrix instructions need 2560 cycles and about 4700 pass; the clock is at 1.8 GHz (power), so that removing the
// exponentials, the stores or the alternation of the phases between the two waves of a SIMD changes the time by
// 1 to 5 % only.  The fragment reads are pinned several matrix instructions ahead of their use: left to itself, at
// this register pressure, the compiler waits out the LDS latency for every one of them (908 -> 868 us).
#include "lds_ring.h"
#include "tile_map.h"

namespace kunlun {

#define PIN() __builtin_amdgcn_sched_barrier(0)  // nothing is moved across by the instruction scheduler

constexpr float LOG2E_W = 1.4426950408889634f;

struct WideSmem {
    static constexpr int D = 128;
    static constexpr int NQ = 256;                       // queries of a workgroup
    static constexpr int TILE = KT * D * 2;              // K tile, V tile
    static constexpr int STAGE = 2 * TILE;
    static constexpr int RING = 3 * STAGE;               // 48 KB
    static constexpr int P_BYTES = NQ * KT * 2;          // P image, dS image ([query][key])
    static constexpr int IMAGES = 4 * P_BYTES;           // both, double-buffered: 64 KB; the prologue stages Q and dO here
    static constexpr int OUT_WAVE = KT * 64;             // a wave's output block: 32 rows of 32 channels
    static constexpr int OUT = 8 * OUT_WAVE;             // 16 KB
    // Q_w^T fragments that a wave parks in LDS, lane by lane: dQ accumulators, dO_w^T and output-block fragments leave
    // too few registers for all eight, and values spilled to scratch memory would be reloaded with vector-memory
    // loads, which wait for the tile loads in flight
    static constexpr int Q_PARK = 3;
    static constexpr int PARK_WAVE = Q_PARK * 64 * 16;
    static constexpr int TOTAL = RING + IMAGES + OUT + 8 * PARK_WAVE;  // 152 KB
    static constexpr int DQ_STRIDE = D * 2 + 16;         // dQ staging rows of the epilogue (padded)
    static_assert(NQ * D * 2 <= IMAGES, "the staged queries must fit the images");
    static_assert(8 * KT * DQ_STRIDE <= RING + IMAGES, "dQ staging must fit");
};

static bool wide_applies(int d, int max_q, int max_kv) { return d == WideSmem::D && max_q > 64 && max_q <= WideSmem::NQ && max_kv > KT; }

// kt0 .. kt1-1: key tiles of the item.  dq_part: null = the item covers all tiles, dQ rows go out rounded;
// else the fp32 dQ partial sums of this range go there, lane by lane (launch_wide_dq_sum adds them).
template <int ACT>
__device__ __forceinline__ void attn_bwd_wide_item(const AttnParams& p, char* smem, int h, int64_t q_row0, int nq, int64_t k0,
                                                   int n_kv, int kt0, int kt1, float* __restrict__ dq_part) {
    using SM = WideSmem;
    constexpr int D = SM::D;
    using L = TileLayout<D>;
    constexpr bool SOFTMAX = ACT == KUNLUN_ACT_SOFTMAX;
    constexpr int KC = D / 16, DB = D / 32;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // opaque per item: nothing derived from it is kept across the persistent loop
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, g = lane >> 5;
    const int64_t hd = (int64_t)p.H * D;
    const uint32_t row_bytes = (uint32_t)(hd * 2);
    const int64_t tile_bytes = (int64_t)KT * row_bytes;
    const char* Qg = (const char*)((const bf16_t*)p.q + q_src_row(p, q_row0) * hd + (int64_t)h * D);
    const char* DOg = (const char*)((const bf16_t*)p.d_o + q_row0 * hd + (int64_t)h * D);
    const char* Kg = (const char*)((const bf16_t*)p.k + (k0 * p.H + h) * D);
    const char* Vg = (const char*)((const bf16_t*)p.v + (k0 * p.H + h) * D);
    const int out_which = wave >> 2, out_db = wave & 3;  // gradient phase: 0 = dV, 1 = dK; 32-channel block
    char* OUTg = (char*)((bf16_t*)(out_which == 0 ? p.dv : p.dk) + (k0 * p.H + h) * D + out_db * 32);
    const uint32_t lds0 = lds_address(smem);
    char* images = smem + SM::RING;  // [buffer][P, dS]
    const uint32_t out_stage = lds0 + SM::RING + SM::IMAGES + wave * SM::OUT_WAVE;
    char* park = smem + SM::RING + SM::IMAGES + SM::OUT + wave * SM::PARK_WAVE + lane * 16;  // + 1024 per fragment
    constexpr int Q_REG = KC - SM::Q_PARK;

    TileDma<D, 8, SWZ_U> dma;  // (V is read as row fragments only, but shares K's read offsets this way)
    dma.init(lane, wave, row_bytes);
    static_assert(TileDma<D, 8, SWZ_U>::IPW == 1, "one load per wave, tile and tensor");
    auto issue = [&](int kt, int stage) {
        const uint32_t dst = lds0 + stage * SM::STAGE;
        dma.issue(Kg + kt * tile_bytes, n_kv - kt * KT, dst);
        dma.issue(Vg + kt * tile_bytes, n_kv - kt * KT, dst + SM::TILE);
    };
    const int n_steps = kt1 - kt0;
    if (n_steps > 0) issue(kt0, 0);

    // ---- prologue: the queries' rows pass through the image region, dO first, then Q (rows past nq read as zero:
    // they add nothing to dK and dV, and their dQ rows are never stored).  Every wave picks the row fragments of its
    // query block (B operands of S^T and dP^T), and the transposed fragments of its output block over all queries.
    const int s16 = lane & 15, hi16 = (lane >> 4) & 1;
    const int colb = (16 * hi16 + 4 * (s16 & 3)) * 2;  // transposing reads: 4 rows x 16 columns per 16 lanes
    int rr0 = L::u_offset(r, g * 16);                  // row fragment: row r, channels 16*kc + 8g .. -> ^ (kc << 5)
    bf16x8 qf[Q_REG], dof[KC], outf[16];
    {
        // queries 16j + 8g + 0..3 and + 4..7, channels of the wave's output block
        const int qtA = L::u_offset(8 * g + (s16 >> 2), colb) ^ (out_db << 6);
        const int qtB = L::u_offset(8 * g + 4 + (s16 >> 2), colb) ^ (out_db << 6);
        auto stage = [&](const char* src) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, (nq - 1) * (int)row_bytes + D * 2, 0x00020000);
            const int row0 = tid >> 4, ch = tid & 15;
            u32x4 st[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                st[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (uint32_t)row0 * row_bytes + ch * 16, i * 32 * row_bytes, 0);
#pragma unroll
            for (int i = 0; i < 8; ++i) *(u32x4*)(images + i * SM::TILE + L::u_offset(row0, ch * 16)) = st[i];
        };
        auto row_frag = [&](int kc) { return *(const bf16x8*)(images + wave * SM::TILE + (rr0 ^ (kc << 5))); };
        auto pick_block = [&]() {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const char* a = images + (j >> 1) * SM::TILE + (j & 1) * 16 * L::ROW_BYTES;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a + qtA));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, a + qtB));
                typedef __attribute__((ext_vector_type(8))) short s16x8;
                outf[j] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        stage(DOg);
        __syncthreads();
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) dof[kc] = row_frag(kc);
        if (out_which == 0) pick_block();
        __syncthreads();
        stage(Qg);
        __syncthreads();
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            if (kc < Q_REG) qf[kc < Q_REG ? kc : 0] = row_frag(kc);
            else *(bf16x8*)(park + (kc - Q_REG) * 1024) = row_frag(kc);
        }
        if (out_which != 0) pick_block();
    }
    if (n_steps > 1) issue(kt0 + 1, 1);
    // softmax statistics of this lane's query: lse in log2 units, delta = <dO, O>
    float lse2 = INFINITY, delta = 0.f;
    if (SOFTMAX) {
        const int qi = 32 * wave + r;
        float part = 0.f;
        if (qi < nq) {
            lse2 = p.lse[(int64_t)h * p.total_q + q_row0 + qi] * LOG2E_W;
            const bf16_t* Or = (const bf16_t*)p.o + (q_row0 + qi) * hd + (int64_t)h * D;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const bf16x8 of = *(const bf16x8*)(Or + 16 * kc + 8 * g);
#pragma unroll
                for (int e = 0; e < 8; ++e) part = fmaf((float)of[e], (float)dof[kc][e], part);
            }
        }
        delta = halves_sum(part);
    }

    // LDS offsets of this lane
    int ktA = L::u_offset(4 * g + (s16 >> 2), colb);      // K^T: keys 16c + 4g + 0..3, channel block db -> ^ (db << 6)
    int ktB = L::u_offset(8 + 4 * g + (s16 >> 2), colb);  //      keys 16c + 8 + 4g + 0..3
    const int ptA = w64_offset(8 * g + (s16 >> 2), colb);        // image columns: queries 16j + 8g + 0..3
    const int ptB = w64_offset(8 * g + 4 + (s16 >> 2), colb);    //                queries 16j + 8g + 4..7
    int pw0 = w64_offset(32 * wave + r, 8 * g);            // image writes: query 32 wave + r, keys 8 vg + 4g .. -> ^ (vg << 4)
    int ow0 = w64_offset(r, 8 * g);                        // output block: key r, channels 8 vg + 4g .. -> ^ (vg << 4)
    const int orow = lane >> 2, och = lane & 3;                  // its rows out: rows orow, orow + 16, chunk och
    const int or0 = w64_offset(orow, och * 16);
    const uint32_t goff = (uint32_t)orow * row_bytes + och * 16;
    // (LDS reads by address: the compiler then folds what is constant between two reads into their offset fields)
    auto row_read = [](uint32_t a) { return *(const __attribute__((address_space(3))) bf16x8*)a; };
    auto tr_read = [](uint32_t a, uint32_t b) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)b);
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto put8 = [](uint32_t a, bf16x4 x) { *(__attribute__((address_space(3))) bf16x4*)a = x; };

    f32x16 dqacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) dqacc[db][v] = 0.f;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const float sc = SOFTMAX ? p.scale * LOG2E_W : p.scale;

    const float neg_lse = SOFTMAX ? -lse2 : 0.f, neg_delta = -delta * p.scale;
    auto score_phase = [&](uint32_t kv, uint32_t img, int kt) {
        // (opaque per tile: the XORed addresses are computed where they are used, not kept in 40 registers)
        asm volatile("" : "+v"(rr0), "+v"(ktA), "+v"(ktB), "+v"(pw0));
        // S^T, then dP^T: the matrix instructions of dP^T run beside the exponentials of S^T.  Each
        // fragment is read AHEAD matrix instructions before its use.
        constexpr int AHEAD = 3;
        const int key_base = kt * KT;
        f32x16 sacc, dpacc;
        float pv[16], dsv[16];
        bf16x8 fr[AHEAD], qb = qf[0];
        auto frag = [&](int j) {  // K row fragments, then V row fragments
            const int kc = j < KC ? j : j - KC;
            return row_read((uint32_t)(rr0 ^ (kc << 5)) + kv + (j < KC ? 0 : SM::TILE));
        };
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) fr[j] = frag(j);
        PIN();
#pragma unroll
        for (int j = 0; j < 2 * KC; ++j) {
            if (j < KC) sacc = mfma32(fr[j % AHEAD], j < Q_REG ? qf[j < Q_REG ? j : 0] : qb, j == 0 ? zero16 : sacc);
            else dpacc = mfma32(fr[j % AHEAD], dof[j < KC ? 0 : j - KC], j == KC ? zero16 : dpacc);
            if (j + 1 >= Q_REG && j + 1 < KC) qb = *(const bf16x8*)(park + (j + 1 - Q_REG) * 1024);
            if (j + AHEAD < 2 * KC) fr[j % AHEAD] = frag(j + AHEAD);
            if (j >= KC) {  // two weights per matrix instruction
#pragma unroll
                for (int v = 2 * (j - KC); v < 2 * (j - KC) + 2; ++v) {
                    if (SOFTMAX) {
                        pv[v] = fast_exp2(fmaf(sacc[v], sc, neg_lse));
                    } else {
                        act_fast_vd<ACT>(sacc[v] * sc, pv[v], dsv[v]);
                        dsv[v] *= p.scale;
                    }
                }
            }
            PIN();
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) dsv[v] = SOFTMAX ? pv[v] * fmaf(dpacc[v], p.scale, neg_delta) : dpacc[v] * dsv[v];
        auto kt_frag = [&](int j) {  // channel block j / 2, keys 16 (j % 2) ..
            const int db = j >> 1, c = j & 1;
            return tr_read((uint32_t)(ktA ^ (db << 6)) + kv + c * 16 * L::ROW_BYTES, (uint32_t)(ktB ^ (db << 6)) + kv + c * 16 * L::ROW_BYTES);
        };
        if (key_base + KT > n_kv || 32 * wave + 32 > nq) {  // keys past the history, and the queries that pad the block
            const int keys_left = r < nq - 32 * wave ? n_kv - key_base - 4 * g : 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool ok = 8 * (v >> 2) + (v & 3) < keys_left;
                pv[v] = ok ? pv[v] : 0.f;
                dsv[v] = ok ? dsv[v] : 0.f;
            }
        }
        bf16x8 pf[2], dsf[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) { pf[c][e] = (bf16_t)pv[8 * c + e]; dsf[c][e] = (bf16_t)dsv[8 * c + e]; }
        PIN();
        bf16x8 kfr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) kfr[j] = kt_frag(j);
        PIN();
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
            const int c = vg >> 1;
            const uint32_t a = (uint32_t)(pw0 ^ (vg << 4)) + img;
            put8(a, (vg & 1) ? __builtin_shufflevector(pf[c], pf[c], 4, 5, 6, 7) : __builtin_shufflevector(pf[c], pf[c], 0, 1, 2, 3));
            put8(a + SM::P_BYTES, (vg & 1) ? __builtin_shufflevector(dsf[c], dsf[c], 4, 5, 6, 7) : __builtin_shufflevector(dsf[c], dsf[c], 0, 1, 2, 3));
        }
        PIN();
#pragma unroll
        for (int j = 0; j < 2 * DB; ++j) {
            dqacc[j >> 1] = mfma32(kfr[j & 3], dsf[j & 1], dqacc[j >> 1]);
            if (j + 4 < 2 * DB) kfr[j & 3] = kt_frag(j + 4);
            PIN();
        }
    };
    auto gradient_phase = [&](uint32_t img, int kt) {
        asm volatile("" : "+v"(ow0));
        const uint32_t src = img + out_which * SM::P_BYTES;
        f32x16 acc;
        bf16x8 fr[4];  // four matrix instructions ahead
        auto frag = [&](int j) { return tr_read(ptA + src + j * 16 * 64, ptB + src + j * 16 * 64); };
        if (nq > SM::NQ - 32) {
#pragma unroll
            for (int j = 0; j < 4; ++j) fr[j] = frag(j);
            PIN();
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                acc = mfma32(outf[j], fr[j & 3], j == 0 ? zero16 : acc);
                if (j + 4 < 16) fr[j & 3] = frag(j + 4);
                PIN();
            }
        } else {  // the blocks that hold queries, two matrix instructions each
            acc = zero16;
#pragma unroll
            for (int j = 0; j < 14; j += 2) {
                if (16 * j >= nq) break;
                fr[0] = frag(j);
                fr[1] = frag(j + 1);
                acc = mfma32(outf[j], fr[0], acc);
                acc = mfma32(outf[j + 1], fr[1], acc);
            }
        }
        // lane: key r, channels 8 vg + 4g + 0..3 of the block -> whole rows of the block, 16 bytes per lane (the
        // region is the wave's own, and the LDS operations of a wave complete in order)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
            bf16x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (bf16_t)acc[4 * vg + e];
            put8((uint32_t)(ow0 ^ (vg << 4)) + out_stage, out);
        }
        const int rows = (n_kv - kt * KT) < KT ? (n_kv - kt * KT) : KT;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(OUTg + kt * tile_bytes), 0, (rows - 1) * (int)row_bytes + 64, 0x00020000);
        const u32x4 x0 = *(const __attribute__((address_space(3))) u32x4*)(out_stage + or0);
        const u32x4 x1 = *(const __attribute__((address_space(3))) u32x4*)(out_stage + or0 + 16 * 64);
        __builtin_amdgcn_raw_buffer_store_b128(x0, rs, goff, 0, 0);  // rows past the history are dropped
        __builtin_amdgcn_raw_buffer_store_b128(x1, rs, goff, 16 * row_bytes, 0);
    };

    // ---- main loop.  Iteration i: scores of tile i, gradients of tile i-1.  The loads of tile i are followed by the
    // two stores of iteration i-2, the two loads of tile i+1 and the two stores of iteration i-1 (iteration 0 has no
    // stores); a wave's vector-memory operations complete in order.
    __syncthreads();  // every wave has its fragments: the images may be written
    int stage = 0;
    for (int i = 0; i <= n_steps; ++i) {
        if (i + 1 < n_steps) {
            if (i >= 3) wait_vmcnt<6>();
            else wait_vmcnt<2>();
        } else if (i < n_steps) {
            wait_vmcnt<0>();
        }
        __syncthreads();  // tile i is complete, the images of tile i-1 are; stage (i-1) % 3 and the images of tile i-2 are free
        if (i + 2 < n_steps) issue(kt0 + i + 2, stage == 0 ? 2 : stage - 1);
        const uint32_t kv = lds0 + stage * SM::STAGE;
        const uint32_t img = lds0 + SM::RING + (i & 1) * 2 * SM::P_BYTES;
        const uint32_t img_prev = lds0 + SM::RING + ((i & 1) ^ 1) * 2 * SM::P_BYTES;
        stage = stage == 2 ? 0 : stage + 1;
        if (i < n_steps && 32 * wave < nq) score_phase(kv, img, kt0 + i);
        PIN();
        if (i > 0) gradient_phase(img_prev, kt0 + i - 1);
    }

    // ---- dQ
    if (dq_part) {
        if (32 * wave >= nq) return;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int vg = 0; vg < 4; ++vg) {
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = dqacc[db][4 * vg + e];
                *(f32x4*)(dq_part + (size_t)(((wave * DB + db) * 4 + vg) * 64 + lane) * 4) = x;
            }
        return;
    }
    __syncthreads();  // every wave is done with the ring and the images
    char* dq_stage = smem + wave * KT * SM::DQ_STRIDE;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
            bf16x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (bf16_t)dqacc[db][4 * vg + e];
            *(bf16x4*)(dq_stage + r * SM::DQ_STRIDE + (32 * db + 8 * vg + 4 * g) * 2) = out;
        }
    const int nq_w = nq - 32 * wave;
    bf16_t* DQg = (bf16_t*)p.dq + (q_row0 + 32 * wave) * hd + (int64_t)h * D;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = i * 4 + (lane >> 4), ch = lane & 15;
        const u32x4 val = *(const u32x4*)(dq_stage + row * SM::DQ_STRIDE + ch * 16);
        if (row < nq_w) __builtin_nontemporal_store(val, (u32x4*)(DQg + row * hd + ch * 8));
    }
}

// The key rows kr0 .. kr1-1 of one head get zero gradients (an example without queries).
__device__ __forceinline__ void zero_key_gradients(const AttnParams& p, int h, int64_t kr0, int n_rows) {
    constexpr int D = WideSmem::D;
    const int64_t hd = (int64_t)p.H * D;
    const u32x4 z = {0, 0, 0, 0};
    for (int idx = threadIdx.x; idx < n_rows * (D / 8); idx += 512) {
        const int row = idx / (D / 8), c8 = idx % (D / 8);
        *(u32x4*)((bf16_t*)p.dk + (kr0 + row) * hd + (int64_t)h * D + c8 * 8) = z;
        *(u32x4*)((bf16_t*)p.dv + (kr0 + row) * hd + (int64_t)h * D + c8 * 8) = z;
    }
}

#define KUNLUN_WIDE_SWITCH(ACTV, CALL)                                  \
    switch (ACTV) {                                                     \
    case KUNLUN_ACT_SOFTMAX: { constexpr int A = KUNLUN_ACT_SOFTMAX; CALL; } break;     \
    case KUNLUN_ACT_IDENTITY: { constexpr int A = KUNLUN_ACT_IDENTITY; CALL; } break;   \
    case KUNLUN_ACT_RELU: { constexpr int A = KUNLUN_ACT_RELU; CALL; } break;           \
    case KUNLUN_ACT_GELU: { constexpr int A = KUNLUN_ACT_GELU; CALL; } break;           \
    case KUNLUN_ACT_GELU_TANH: { constexpr int A = KUNLUN_ACT_GELU_TANH; CALL; } break; \
    case KUNLUN_ACT_SILU: { constexpr int A = KUNLUN_ACT_SILU; CALL; } break;           \
    default: { constexpr int A = KUNLUN_ACT_GELU_POLY; CALL; } break;                   \
    }

// Work items = (example, head) in scheduler order on a persistent launch with a work counter, as in the pair kernel
// (attn_bwd_pair_mfma.hip).
__global__ __launch_bounds__(512, 2) void gdpa_bwd_wide_kernel(AttnParams p, int n_items) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    // hand-over word of the next item: the last word of the last wave's parked fragments, dead between items
    volatile int* const next_word = (volatile int*)(smem + WideSmem::TOTAL - 4);
    int item = blockIdx.x;
    while (item < n_items) {
        int claimed = 0;
        if (threadIdx.x == 0) claimed = atomicAdd(p.queue, 1);
        const int slot = item & 7;
        const int64_t j = item >> 3;
        const int h = (int)(j % p.H);
        const int64_t e = (j / p.H) * 8 + slot;
        if (e < p.B) {
            const int b = p.order[e];
            const int64_t q0 = q_begin(p, b);
            const int nq = (int)(q_end(p, b) - q0);
            const int64_t k0 = p.kv_off[b];
            const int n_kv = p.kv_off[b + 1] - (int)k0;
            if (nq <= 0) zero_key_gradients(p, h, k0, n_kv);
            else KUNLUN_WIDE_SWITCH(p.head_act[h], (attn_bwd_wide_item<A>(p, smem, h, q0, nq, k0, n_kv, 0, (n_kv + KT - 1) / KT, nullptr)));
        }
        __syncthreads();  // the item's last LDS reads (dQ rows) are done
        if (threadIdx.x == 0) *next_word = claimed + (int)gridDim.x;
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(*next_word);  // (next written in the next item's prologue, where the last wave parks its fragments behind the barriers of the staging)
    }
}

// The same on ranges of `chunk` key tiles: one workgroup per (example, range, head), fp32 dQ partial sums per range.
// Work mapping of tile_map.h with tiles of 32 * chunk keys.
__global__ __launch_bounds__(512, 2) void gdpa_bwd_wide_range_kernel(AttnParams p, const int32_t* __restrict__ tile_start,
                                                                     const int32_t* __restrict__ tile_example, int chunk,
                                                                     float* __restrict__ partial, int part_floats) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int b, h, t;
    if (!locate_tile(tile_start, tile_example, p.B, p.H, blockIdx.x, b, h, t)) return;
    const int64_t q0 = q_begin(p, b);
    const int nq = (int)(q_end(p, b) - q0);
    const int64_t k0 = p.kv_off[b];
    const int n_kv = p.kv_off[b + 1] - (int)k0;
    const int n_tiles = (n_kv + KT - 1) / KT;
    const int kt0 = t * chunk, kt1 = kt0 + chunk < n_tiles ? kt0 + chunk : n_tiles;
    if (nq <= 0) {
        const int row1 = kt1 * KT < n_kv ? kt1 * KT : n_kv;
        zero_key_gradients(p, h, k0 + kt0 * KT, row1 - kt0 * KT);
        return;
    }
    float* out = partial + ((size_t)(tile_start[b] + t) * p.H + h) * part_floats;
    KUNLUN_WIDE_SWITCH(p.head_act[h], (attn_bwd_wide_item<A>(p, smem, h, q0, nq, k0, n_kv, kt0, kt1, out)));
}

// dQ rows = the partial sums of the example's ranges, added in range order, rounded once; four channels per thread, in
// the order in which the lanes of the kernel above left them.
__global__ __launch_bounds__(256) void wide_dq_sum_kernel(AttnParams p, const int32_t* __restrict__ tile_start,
                                                          const float* __restrict__ partial, int part_floats) {
    constexpr int D = WideSmem::D;
    const int per_item = part_floats / 4;  // multiple of 1024
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int idx = (int)(gid % per_item);
    const int64_t item = gid / per_item;
    const int b = (int)(item / p.H), h = (int)(item % p.H);
    const int lane = idx & 63, vg = (idx >> 6) & 3, db = (idx >> 8) & 3, w = idx >> 10;
    const int row = 32 * w + (lane & 31), ch = 32 * db + 8 * vg + 4 * (lane >> 5);
    const int64_t q0 = q_begin(p, b);
    if (row >= (int)(q_end(p, b) - q0)) return;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int t = tile_start[b]; t < tile_start[b + 1]; ++t)
        sum += *(const f32x4*)(partial + ((size_t)t * p.H + h) * part_floats + (size_t)idx * 4);
    bf16x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = (bf16_t)sum[e];
    *(bf16x4*)((bf16_t*)p.dq + (q0 + row) * (int64_t)p.H * D + (int64_t)h * D + ch) = out;
}

bool mfma_bwd_wide_supported(const AttnParams& p, int dtype) {
    return dtype == KUNLUN_BF16 && !p.windowed && wide_applies(p.d, p.max_q, p.max_kv);
}

// Key tiles per range, 0 = whole histories.  A tile takes a workgroup about 2.2 us whatever else runs, so a launch
// lasts at least as long as its longest history; ranges lift that for the price of the partial sums (128 KB written
// and read per range and head).  Whole backward and forward call with 256 queries, H = 4, whole against ranges: 64
// histories of 64..1024 keys (longest = 1.9 times the mean work of a compute unit) 132 / 153 us, 16 x 8 heads of them
// (3.8 times) 120 / 108 us, 64 log-normal histories up to 4096 (3.7 times) 392 / 307 us; with 100 queries,
// where half of the waves have no scores to compute, the backward alone of 128 log-normal histories (1.9 times) takes
// 252 / 219 us, of 64 histories of 64..1024 keys (1.9 times) 62 / 73 us.
// Two ranges per compute unit, of at least 8 tiles.
static int wide_chunk(int B, int H, int max_q, int max_kv, int64_t total_kv) {
    const int64_t tiles = total_kv * H / KT;
    const int64_t longest = (max_kv + KT - 1) / KT;
    if ((int64_t)B * H >= 1024 || longest * 256 <= (max_q > 128 ? 2 * tiles : 3 * tiles / 2)) return 0;
    const int64_t c = tiles / 512;
    return (int)(c < 8 ? 8 : c);
}
static int wide_part_floats(int max_q) { return (max_q + 31) / 32 * 32 * WideSmem::D; }

size_t mfma_bwd_wide_workspace(int B, int H, int d, int max_q, int max_kv, int64_t total_kv) {
    if (!wide_applies(d, max_q, max_kv)) return 0;
    const int c = wide_chunk(B, H, max_q, max_kv, total_kv);
    return c == 0 ? 0 : align_up((size_t)(total_kv / (c * KT) + B) * H * wide_part_floats(max_q) * sizeof(float), 256);
}

hipError_t launch_mfma_bwd_wide(const AttnParams& params, void* counters, void* order, void* tables, void* partial, hipStream_t stream) {
    AttnParams p = params;
    constexpr int bytes = WideSmem::TOTAL;
    const int chunk = wide_chunk(p.B, p.H, p.max_q, p.max_kv, p.total_kv);
    if (chunk > 0) {
        // once per process (thread-safe initialisation of a function-local static); not a stream operation
        static const hipError_t raised =
            hipFuncSetAttribute((const void*)gdpa_bwd_wide_range_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (raised != hipSuccess) return raised;
        int32_t* tile_start = (int32_t*)tables;
        int32_t* tile_example = tile_example_of(tile_start, p.B);
        const int part_floats = wide_part_floats(p.max_q);
        hipLaunchKernelGGL(tile_prefix_kernel<2>, dim3(1), dim3(1024), 0, stream, p.kv_off, 0, p.B, tile_start, tile_example, chunk * KT);
        const int64_t per_xcd = ((p.total_kv / (chunk * KT) + p.B) * p.H + 7) / 8;  // an upper bound of the range count sizes the grid
        hipLaunchKernelGGL(gdpa_bwd_wide_range_kernel, dim3((unsigned)((per_xcd + 1) * 8)), dim3(512), bytes, stream, p, tile_start, tile_example,
                           chunk, (float*)partial, part_floats);
        hipLaunchKernelGGL(wide_dq_sum_kernel, dim3((unsigned)((int64_t)p.B * p.H * (part_floats / 1024))), dim3(256), 0, stream, p, tile_start,
                           (const float*)partial, part_floats);
        return hipGetLastError();
    }
    static const hipError_t raised =
        hipFuncSetAttribute((const void*)gdpa_bwd_wide_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (raised != hipSuccess) return raised;
    p.order = (const int32_t*)order;
    p.queue = (int32_t*)counters;
    const hipError_t e = launch_schedule(p.kv_off, p.B, p.max_kv, (int32_t*)order, p.queue, stream);
    if (e != hipSuccess) return e;
    const int64_t n_items = (((int64_t)p.B + 7) / 8) * 8 * p.H;
    const int64_t resident = compute_units();
    hipLaunchKernelGGL(gdpa_bwd_wide_kernel, dim3((unsigned)(n_items > resident ? resident : n_items)), dim3(512), bytes, stream, p, (int)n_items);
    return hipGetLastError();
}

}  // namespace kunlun
