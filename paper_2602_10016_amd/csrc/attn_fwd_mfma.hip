// bf16 matrix-core forward kernel for gfx950, streaming launches: GDPA (Eq. (GDPA)) and softmax
// attention of a few seed / context queries (up to 64 per example) over a jagged history
// (Eq. (PMA), Eq. (seed-level attention)).  Longer query sequences and the sliding window are
// served by the query-tiled kernel (attn_fwd_ring_mfma.hip).
//
// A workgroup owns one work item = (example, head), or a pair of heads of 32 channels (HP = 2); a wave owns 32*NQB of its
// queries for the whole item.  Either NW waves with different queries stream the 32-key K/V tiles of the item together:
// every thread fetches its share of tile t+1 (and t+2) into registers (whole rows, coalesced,
// non-temporal) while tile t, already in LDS, is being consumed; tiles are double-buffered in
// LDS, so there is one barrier per tile.  Or KS waves with the same queries take the tiles in turn, without a barrier, and
// merge their results at the end (mfma_fwd_plan() says which).  These operators do only Nq flops per byte of K/V (a
// key/value byte is used by the queries of its own example and head and by nobody else), far
// below the matrix-core ridge, so the design goal is bytes in flight and enough resident waves
// to hide latency, not MFMA occupancy.
//
// Per 32-key tile and wave:
//     S^T = K Q^T              (MFMA; Q^T fragments resident in registers)
//     P^T = score function of S^T * scale, in registers, zero past the end of the history,
//           packed to bf16
//     O^T += V^T P^T           (MFMA; V^T via transposing LDS reads)
// Softmax keeps a running maximum and sum per query (one query per lane column) and rescales
// O^T when the maximum grows; the activation path has no such stage.
#include "attn_fwd_score.h"

namespace kunlun {

// LDS tiles of the forward kernels: 32 rows, row-major, each row padded so that every access
// pattern is free of bank conflicts and every offset is affine in (row, column):
//   K rows + 16 bytes: the 16 lanes that read the same 16-byte chunk of 16 consecutive rows
//                      (A-operand reads) fall into 16 different 16-byte bank slots;
//   V rows + 64 bytes: the 4 consecutive rows of a transposing read fall into 4 different
//                      64-byte bank groups.
template <int D>
struct FwdSmem {
    static constexpr int K_STRIDE = D * 2 + 16;
    static constexpr int V_STRIDE = D == 32 ? 64 : D * 2 + 64;  // (D = 32: four rows of 64 bytes already cover all banks)
    static constexpr int K_TILE = KT * K_STRIDE;
    static constexpr int V_TILE = KT * V_STRIDE;
    static constexpr int BUF_BYTES = K_TILE + V_TILE;  // K tile, then V tile
    static constexpr int TOTAL = 2 * BUF_BYTES;        // double buffer (workgroups of several waves)
    // A wave that streams alone needs no second buffer (it writes a tile, reads it, and writes the next one in
    // program order); the key-split launches use that to fit four waves' buffers, the others keep two buffers
    // (the store of the next tile can then be scheduled before the reads of the current one end).  With both query
    // blocks in a wave (nqb = 2) its partial results, which pass through the same bytes, are what takes the room.
    static constexpr int bytes(int ks, int nqb) { return ks == 1 ? TOTAL : nqb == 1 ? BUF_BYTES : D / 32 * nqb * 4096 + 2048; }
};

// Cooperative global -> register -> LDS staging of one 32-row tile by a workgroup of 64*NW
// threads: slot = i*64*NW + tid covers (row, 16-byte chunk) pairs row-major, so whole rows
// coalesce.  A thread's chunks sit ROWS_PER_LOAD rows apart, so every address is "uniform
// base + one per-thread offset + constant" and the key loop spends no vector arithmetic on it.
template <int D, int NW>
struct CoopTile {
    using SM = FwdSmem<D>;
    static constexpr int CHUNKS = D / 8;  // 16-byte chunks per row
    static constexpr int SLOTS = KT * CHUNKS;
    static constexpr int LOADS = SLOTS / (64 * NW);
    static constexpr int ROWS_PER_LOAD = 64 * NW / CHUNKS;
    static_assert(LOADS >= 1 && SLOTS % (64 * NW) == 0, "tile does not split evenly over the workgroup");

    uint32_t goff;   // byte offset of this thread's first chunk inside a tile of the [tokens,H,D] tensor
    int kw, vw;      // LDS byte offsets of the same chunk in the K / V tiles
    int row0, chunk;
    uint32_t row_bytes;

    __device__ __forceinline__ void init(int tid, uint32_t row_stride_bytes) {
        row0 = tid / CHUNKS;
        chunk = tid % CHUNKS;
        row_bytes = row_stride_bytes;
        goff = (uint32_t)row0 * row_stride_bytes + chunk * 16;
        kw = row0 * SM::K_STRIDE + chunk * 16;
        vw = row0 * SM::V_STRIDE + chunk * 16;
    }
    // Loads go through a buffer resource that covers exactly the valid rows of the tile: rows
    // past the end of a history read as zero (and get zero weight later), with no address
    // clamping in the loop.  voffset = the thread's constant offset, soffset = uniform.
    // STREAM: the data is read once by this workgroup and by nobody else (GDPA keys/values):
    // non-temporal loads keep it from displacing useful lines in the caches.  Not at D = 32: a row piece is then
    // half a 128-byte line, the other half belongs to the neighbouring head, and a streaming load fetches the
    // whole line for one use (measured on the bench batch: 2.06 GB fetched against 1.80 GB with plain loads, which
    // the neighbouring head's workgroup can hit in L2 when it runs on the same XCD; the operands are 1.2 GB).
    template <bool STREAM>
    __device__ __forceinline__ void load(u32x4 (&st)[LOADS], const char* __restrict__ tile_base, int rows_valid) const {
        const int rows = rows_valid < KT ? rows_valid : KT;
        const int bytes = (rows - 1) * (int)row_bytes + D * 2;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)tile_base, 0, bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            st[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff, i * ROWS_PER_LOAD * row_bytes, STREAM && D != 32 ? 2 : 0);
    }
    __device__ __forceinline__ void store(char* ldsK, char* ldsV, const u32x4 (&ks)[LOADS], const u32x4 (&vs)[LOADS]) const {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) *(u32x4*)(ldsK + kw + i * ROWS_PER_LOAD * SM::K_STRIDE) = ks[i];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) *(u32x4*)(ldsV + vw + i * ROWS_PER_LOAD * SM::V_STRIDE) = vs[i];
    }
};

// SMALL: GELU in its short form where the scores of a tile allow it (short_gelu()).
// HP = 2: the item is a PAIR of neighbouring heads of D / 2 channels each, whose row pieces are one piece of D channels; the
// wave forms the scores and outputs of both from the same tiles.
// One work item.  q_row0 / nq_wg: first query row (global) and query count of the workgroup's tile.
// KS > 1 (with NW = 1): the workgroup has KS waves that own the SAME queries and take the key tiles of the
// item in turn (wave s: tiles s, s + KS, ...), each with its own tile buffers and no barrier in the key loop;
// their partial results are merged in LDS at the end, in wave order.  For launches with few work items, where
// one wave per item would leave the time to the longest history.
template <int D, int HP, int NQB, int NW, int ACT, int AHEAD, int KS, bool SMALL>
__device__ __forceinline__ void attn_fwd_item(const AttnParams& p, char* lds, int h, int64_t q_row0, int nq_wg,
                                              int64_t k0, int n_kv) {
    using SM = FwdSmem<D>;
    using CT = CoopTile<D, NW>;
    static_assert(KS == 1 || NW == 1, "key splitting is for single-wave query groups");
    constexpr bool SOFTMAX = ACT == KUNLUN_ACT_SOFTMAX;
    constexpr int DH = D / HP;          // head dimension
    constexpr int KC = DH / 16;         // contraction steps of S^T = K Q^T
    constexpr int DB = DH / 32;         // 32-channel blocks of O^T
    static_assert(DB >= 1, "a head has at least 32 channels");
    constexpr int QW = 32 * NQB;  // queries per wave
    // (the thread index goes through an opaque move per item: what is derived from it is computed where the item
    // uses it, and not kept in registers across the loop of a persistent launch for all six score functions)
    int tid_wg = threadIdx.x;
    asm volatile("" : "+v"(tid_wg));
    const int split = KS > 1 ? __builtin_amdgcn_readfirstlane(tid_wg >> 6) : 0;  // this wave's turn in the key tiles
    const int tid = KS > 1 ? (tid_wg & 63) : tid_wg;
    constexpr int LDS_BYTES = SM::bytes(KS, NQB);  // of one query-owning group of waves
    char* const lds_all = lds;
    lds += split * LDS_BYTES;
    const int lane = tid & 63, wave = tid >> 6;
    const int r = lane & 31, g = lane >> 5;
    const int64_t hd = (int64_t)p.H * DH;
    const uint32_t row_bytes = (uint32_t)(hd * 2);
    const int64_t tile_bytes = (int64_t)KT * row_bytes;
    const bf16_t* Q = (const bf16_t*)p.q;
    const char* K = (const char*)((const bf16_t*)p.k + (k0 * p.H + h) * DH);
    const char* V = (const char*)((const bf16_t*)p.v + (k0 * p.H + h) * DH);

    // this wave's queries
    const int q_lo_w = wave * QW;
    int nq = nq_wg - q_lo_w;
    nq = nq < 0 ? 0 : (nq > QW ? QW : nq);
    const bool wave_active = nq > 0;
    const int kt_end = (n_kv + KT - 1) / KT;  // key tiles of the item
    const int n_local = kt_end > split ? (kt_end - split + KS - 1) / KS : 0;  // ... of this wave: split + i*KS

    CT ct;
    ct.init(tid, row_bytes);
    // LDS read offsets of this lane.  K fragment of contraction step kc (A operand: row r,
    // channels 16*kc + 8g ..): kr + 32*kc.  V^T fragment of channel block db for the keys in
    // registers 8c..8c+7 of the score layout (keys 16c + 4g + 0..3 and 16c + 8 + 4g + 0..3): two
    // transposing reads at vr + 64*db + 16c rows (+ 8 rows); in each, the 16 lanes of a group
    // address a 4 (keys) x 16 (channels) block - lane s points at key s/4, channels 4*(s%4) .. -
    // and lane i receives channel i of the four keys.
    const int kr = r * SM::K_STRIDE + g * 16;
    const int vr = (4 * g + ((lane & 15) >> 2)) * SM::V_STRIDE + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;

    // Q^T fragments (B operand): column = query 32*qb + r, contraction = channels 16*kc + 8g..
    // The workgroup's query tile is fetched with whole-row coalesced loads (rows past the tile
    // read as zero), staged in LDS in the K-tile row layout, and each wave picks its fragments.
    constexpr int QT = QW * NW;
    constexpr int Q_LOADS = QT * CT::CHUNKS / (64 * NW);
    static_assert(QT * SM::K_STRIDE <= LDS_BYTES, "query tile must fit the tile buffers");
    bf16x8 qf[NQB][HP * KC];
    {
        const char* qbase = (const char*)(Q + q_src_row(p, q_row0) * hd + (int64_t)h * DH);
        const __amdgpu_buffer_rsrc_t qrsrc =
            __builtin_amdgcn_make_buffer_rsrc((void*)qbase, 0, (nq_wg - 1) * (int)row_bytes + D * 2, 0x00020000);
        u32x4 qst[Q_LOADS];
#pragma unroll
        for (int i = 0; i < Q_LOADS; ++i)
            qst[i] = __builtin_amdgcn_raw_buffer_load_b128(qrsrc, ct.goff, i * CT::ROWS_PER_LOAD * row_bytes, 0);
#pragma unroll
        for (int i = 0; i < Q_LOADS; ++i) *(u32x4*)(lds + ct.kw + i * CT::ROWS_PER_LOAD * SM::K_STRIDE) = qst[i];
        if (NW > 1) __syncthreads();
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
            for (int kc = 0; kc < HP * KC; ++kc)
                qf[qb][kc] = *(const bf16x8*)(lds + (q_lo_w + 32 * qb) * SM::K_STRIDE + kr + 32 * kc);
        if (NW > 1) __syncthreads();  // the tile buffers are reused for K/V from here on
    }

    // key k is visible iff (unsigned)k <= key_span (every key of the history; none if it is empty)
    const int key_lo = n_kv > 0 ? 0 : 0x3fffffff;
    const unsigned key_span = n_kv > 0 ? (unsigned)(n_kv - 1) : 0u;

    f32x16 oacc[HP][DB][NQB];
    float m_ref[HP][NQB], l_run[HP][NQB];  // softmax: reference maximum (log2 units) and running sum
#pragma unroll
    for (int hh = 0; hh < HP; ++hh)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
            m_ref[hh][qb] = -INFINITY;
            l_run[hh][qb] = 0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[hh][db][qb][v] = 0.f;
        }
    const float sc = SOFTMAX ? p.scale * LOG2E : p.scale;

    // AHEAD tiles ahead of the one being consumed are in flight in registers (AHEAD register sets,
    // used in turn): one tile costs a full memory round trip, so a wave that walks its history alone
    // moves AHEAD tiles per round trip.
    static_assert(AHEAD == 1 || AHEAD % 2 == 0, "the LDS double buffer alternates with the tile index");
    u32x4 kst[AHEAD][CT::LOADS], vst[AHEAD][CT::LOADS];
    auto fetch = [&](u32x4 (&ks)[CT::LOADS], u32x4 (&vs)[CT::LOADS], int i) {
        const int kt = split + i * KS;
        if (kt < kt_end) {
            const int rows = n_kv - kt * KT;
            ct.template load<true>(ks, K + kt * tile_bytes, rows);
            ct.template load<true>(vs, V + kt * tile_bytes, rows);
        }
    };
    auto compute = [&](const char* ldsK, const char* ldsV, int i) {
        if (!wave_active) return;
        const int kt = split + i * KS;
        // ---- S^T = K Q^T
        f32x16 sacc[HP][NQB];
#pragma unroll
        for (int hh = 0; hh < HP; ++hh) {
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
                for (int v = 0; v < 16; ++v) sacc[hh][qb][v] = 0.f;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const bf16x8 a = *(const bf16x8*)(ldsK + kr + 32 * (hh * KC + kc));
#pragma unroll
                for (int qb = 0; qb < NQB; ++qb) sacc[hh][qb] = mfma32(a, qf[qb][hh * KC + kc], sacc[hh][qb]);
            }
        }
        // ---- score function, masking, packing
        const int key_base = kt * KT;
        const bool need_mask = key_base + KT > n_kv;  // only the last tile of a history has invisible keys
        bf16x8 pf[HP][NQB][2];
#pragma unroll
        for (int hh = 0; hh < HP; ++hh)
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb)
                score_to_weights<ACT, DB, NQB, false, SMALL>(sacc[hh][qb], need_mask, (unsigned)(key_base + 4 * g - key_lo), key_span, sc,
                                                             m_ref[hh][qb], l_run[hh][qb], oacc[hh], qb, pf[hh][qb]);
        // ---- O^T += V^T P^T
#pragma unroll
        for (int hh = 0; hh < HP; ++hh)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const char* src = ldsV + vr + 64 * (hh * DB + db) + c * 16 * SM::V_STRIDE;
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, src));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, src + 8 * SM::V_STRIDE));
                    typedef __attribute__((ext_vector_type(8))) short s16x8;
                    const bf16x8 a = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                    for (int qb = 0; qb < NQB; ++qb) oacc[hh][db][qb] = mfma32(a, pf[hh][qb][c], oacc[hh][db][qb]);
                }
            }
    };
    auto step = [&](u32x4 (&ks)[CT::LOADS], u32x4 (&vs)[CT::LOADS], int i, int buf) {
        char* ldsK = lds + (KS > 1 ? 0 : buf) * SM::BUF_BYTES;
        char* ldsV = ldsK + SM::K_TILE;
        ct.store(ldsK, ldsV, ks, vs);
        // the tile is complete in LDS; every wave is also done with the other buffer (the tile before)
        if (NW > 1) __syncthreads();
        fetch(ks, vs, i + AHEAD);
        compute(ldsK, ldsV, i);
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) fetch(kst[j], vst[j], j);
    if (AHEAD == 1) {
        for (int i = 0; i < n_local; i += 2) {
            step(kst[0], vst[0], i, 0);
            if (i + 1 < n_local) step(kst[0], vst[0], i + 1, 1);
        }
    } else {
        for (int i = 0; i < n_local; i += AHEAD) {
#pragma unroll
            for (int j = 0; j < AHEAD; ++j)
                if (i + j < n_local) step(kst[j], vst[j], i + j, j & 1);
        }
    }

    if (KS > 1) {
        // ---- merge of the KS partial results (wave 0 collects, in wave order): every other wave leaves its
        // accumulators, lane by lane, in its own idle tile buffers, with the softmax reference and sum
        // (su: head of the pair and query block)
        constexpr int STAT = HP * DB * NQB * 4 * 1024;  // byte offset of the statistics behind the accumulators
        static_assert(STAT + HP * NQB * 2 * 256 <= LDS_BYTES, "partial results must fit the tile buffers");
        if (split > 0) {
#pragma unroll
            for (int hh = 0; hh < HP; ++hh)
#pragma unroll
                for (int qb = 0; qb < NQB; ++qb) {
                    const int su = hh * NQB + qb;
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int vg = 0; vg < 4; ++vg) {
                            f32x4 x;
#pragma unroll
                            for (int e = 0; e < 4; ++e) x[e] = oacc[hh][db][qb][4 * vg + e];
                            *(f32x4*)(lds + (((hh * DB + db) * NQB + qb) * 4 + vg) * 1024 + lane * 16) = x;
                        }
                    if (SOFTMAX) {
                        *(float*)(lds + STAT + (2 * su) * 256 + lane * 4) = m_ref[hh][qb];
                        *(float*)(lds + STAT + (2 * su + 1) * 256 + lane * 4) = l_run[hh][qb];
                    }
                }
        }
        __syncthreads();
        if (split > 0) return;
#pragma unroll 1
        for (int w = 1; w < KS; ++w) {
            const char* part = lds_all + w * LDS_BYTES;
#pragma unroll
            for (int hh = 0; hh < HP; ++hh)
#pragma unroll
                for (int qb = 0; qb < NQB; ++qb) {
                    const int su = hh * NQB + qb;
                    float cw = 1.f;
                    if (SOFTMAX) {
                        const float mw = *(const float*)(part + STAT + (2 * su) * 256 + lane * 4);
                        const float lw = *(const float*)(part + STAT + (2 * su + 1) * 256 + lane * 4);
                        const float m_new = fmaxf(m_ref[hh][qb], mw);
                        const float c0 = m_ref[hh][qb] == -INFINITY ? 0.f : fast_exp2(m_ref[hh][qb] - m_new);
                        cw = mw == -INFINITY ? 0.f : fast_exp2(mw - m_new);
                        l_run[hh][qb] = l_run[hh][qb] * c0 + lw * cw;
                        m_ref[hh][qb] = m_new;
#pragma unroll
                        for (int db = 0; db < DB; ++db)
#pragma unroll
                            for (int v = 0; v < 16; ++v) oacc[hh][db][qb][v] *= c0;
                    }
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int vg = 0; vg < 4; ++vg) {
                            const f32x4 x = *(const f32x4*)(part + (((hh * DB + db) * NQB + qb) * 4 + vg) * 1024 + lane * 16);
#pragma unroll
                            for (int e = 0; e < 4; ++e) oacc[hh][db][qb][4 * vg + e] = fmaf(x[e], cw, oacc[hh][db][qb][4 * vg + e]);
                        }
                }
        }
    }

    // ---- epilogue: lane holds query 32*qb + r, channels 32*db + 8*(v/4) + 4g + (v%4).  The wave
    // transposes its O tile through LDS (its own region of the now idle tile buffers) and
    // writes whole rows, 16 bytes per lane.
    if (NW > 1) __syncthreads();  // every wave is done with the K/V tiles
    if (!wave_active) return;
    char* stage = lds + wave * (QW * SM::K_STRIDE);
#pragma unroll
    for (int hh = 0; hh < HP; ++hh)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
            const int qi = 32 * qb + r;  // inside this wave's block
            float inv = 1.f;
            if (SOFTMAX) {
                const float l_tot = halves_sum(l_run[hh][qb]);
                inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
                if (p.lse && g == 0 && qi < nq)
                    p.lse[(int64_t)(h + hh) * p.total_q + q_row0 + q_lo_w + qi] =
                        l_tot > 0.f ? (m_ref[hh][qb] + __builtin_amdgcn_logf(l_tot)) * (1.f / LOG2E) : -INFINITY;
            }
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    bf16x4 out;
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[e] = (bf16_t)(oacc[hh][db][qb][4 * vg + e] * inv);
                    *(bf16x4*)(stage + qi * SM::K_STRIDE + (32 * (hh * DB + db) + 8 * vg + 4 * g) * 2) = out;
                }
        }
    {
        bf16_t* obase = (bf16_t*)p.o + (q_row0 + q_lo_w) * hd + (int64_t)h * DH;
        constexpr int O_STORES = QW * CT::CHUNKS / 64;
        const int chunk = lane % CT::CHUNKS, rsub = lane / CT::CHUNKS;
#pragma unroll
        for (int i = 0; i < O_STORES; ++i) {
            const int row = i * (64 / CT::CHUNKS) + rsub;
            const u32x4 val = *(const u32x4*)(stage + row * SM::K_STRIDE + chunk * 16);
            if (row < nq) __builtin_nontemporal_store(val, (u32x4*)(obase + row * hd + chunk * 8));  // written once, not read back
        }
    }
}

template <int D, int HP, int NQB, int NW, int AHEAD, int KS, bool SMALL>
__device__ __forceinline__ void attn_fwd_dispatch(const AttnParams& p, char* lds, int act, int h, int64_t q_row0,
                                                  int nq, int64_t k0, int n_kv) {
    switch (act) {
    case KUNLUN_ACT_SOFTMAX: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_SOFTMAX, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    case KUNLUN_ACT_IDENTITY: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_IDENTITY, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    case KUNLUN_ACT_RELU: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_RELU, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    case KUNLUN_ACT_GELU: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_GELU, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    case KUNLUN_ACT_GELU_TANH: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_GELU_TANH, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    case KUNLUN_ACT_SILU: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_SILU, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    default: attn_fwd_item<D, HP, NQB, NW, KUNLUN_ACT_GELU_POLY, AHEAD, KS, SMALL>(p, lds, h, q_row0, nq, k0, n_kv); break;
    }
}

// GDPA / cross attention: work items = (example, query tile, head), examples in scheduler order (longest
// history first).  Item i belongs to "lane" i % 8: consecutive entries (example, query tile) go to consecutive
// lanes and each lane walks through all heads of its entries - on a grid of one workgroup per item, where
// workgroup i runs on XCD i % 8, every L2 so sees all address residues modulo the token stride H*D*2 (one head
// per XCD would use only a fraction of the L2 channels).
// With a work counter (p.queue: launches with more items than resident workgroups) the launch is persistent:
// as many workgroups as fit the device, each starts with the item of its index and then takes the next
// unclaimed one, which is the dispatcher's longest-first list scheduling without its cost (measured on the
// jagged benchmark batch: with cheap score functions the dispatcher kept a third of the workgroup slots empty).
// The counter is asked for the next item while the current one starts.
template <int D, int HP, int NQB, int NW, int OCC, int AHEAD, int KS, bool SMALL>
__global__ __launch_bounds__(64 * NW * KS, OCC) void gdpa_fwd_mfma_kernel(AttnParams p, int n_qtiles, int n_items) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];  // KS * FwdSmem<D>::bytes(KS, NQB) bytes
    constexpr int QT = 32 * NQB * NW;
    // hand-over word for the next item: the last word of the tile buffers, dead between items
    volatile int* const next_word = (volatile int*)(lds + KS * FwdSmem<D>::bytes(KS, NQB) - 4);
    const int64_t n_entries = (int64_t)p.B * n_qtiles;
    int item = blockIdx.x;
    while (item < n_items) {
        int claimed = 0;
        if (KS == 1 && p.queue && threadIdx.x == 0) claimed = atomicAdd(p.queue, 1);
        const int slot = item & 7;
        const int64_t j = item >> 3;
        const int groups = p.H / HP;
        const int h = (int)(j % groups) * HP;
        const int64_t e = (j / groups) * 8 + slot;
        if (e < n_entries) {
            const int qt = (int)(e % n_qtiles);
            const int b = p.order ? p.order[e / n_qtiles] : (int)(e / n_qtiles);
            const int64_t qb0 = q_begin(p, b);
            const int64_t nq_all = q_end(p, b) - qb0;
            const int64_t q_first = (int64_t)qt * QT;
            if (q_first < nq_all) {
                const int nq = (int)((nq_all - q_first) < QT ? (nq_all - q_first) : QT);
                const int64_t k0 = p.kv_off[b];
                const int n_kv = p.kv_off[b + 1] - (int)k0;
                attn_fwd_dispatch<D, HP, NQB, NW, AHEAD, KS, SMALL>(p, lds, p.head_act[h], h, qb0 + q_first, nq, k0, n_kv);
            }
        }
        if (KS > 1 || !p.queue) break;
        __syncthreads();  // the item's last LDS reads (output rows) are done
        if (threadIdx.x == 0) *next_word = claimed + (int)gridDim.x;
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(*next_word);  // (next written by the second key tile of the next item, behind barriers)
    }
}

bool mfma_fwd_supported(const AttnParams& p, int dtype) {
    if (dtype != KUNLUN_BF16 || (p.d != 32 && p.d != 64 && p.d != 128)) return false;
    // the online softmax takes the row maximum before scaling: it needs scale > 0
    // (other scales are served by the generic kernels)
    for (int h = 0; h < p.H; ++h)
        if (p.head_act[h] == KUNLUN_ACT_SOFTMAX && !(p.scale > 0.f)) return false;
    return true;
}

template <bool SMALL, int D, int HP, int NQB, int NW, int OCC, int AHEAD, int KS>
static hipError_t launch_gdpa(const AttnParams& p, hipStream_t stream) {
    constexpr int QT = 32 * NQB * NW;
    constexpr int bytes = KS * FwdSmem<D>::bytes(KS, NQB);
    auto kern = gdpa_fwd_mfma_kernel<D, HP, NQB, NW, OCC, AHEAD, KS, SMALL>;
    if (bytes > 64 * 1024) {
        // once per process (thread-safe initialisation of a function-local static); not a stream operation
        static const hipError_t raised = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (raised != hipSuccess) return raised;
    }
    const int n_qtiles = (p.max_q + QT - 1) / QT;
    const int64_t n_items = (((int64_t)p.B * n_qtiles + 7) / 8) * 8 * (p.H / HP);
    int64_t grid = n_items;
    if (KS == 1 && p.queue) {
        // workgroups of this kernel that fit the device (once per process, like the attribute above)
        static const int per_cu = [&] {
            int n = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)kern, 64 * NW * KS, bytes) != hipSuccess || n < 1) n = 1;
            return n;
        }();
        // Fewer workgroups than would fit: every workgroup is a walk of its own through memory, and the memory system
        // moves the bytes of few walks faster than those of many, as long as the score function keeps up: exponential
        // forms and the short form of GELU do, its general form does not.  GELU on small scores, 8 heads, log-normal
        // histories, us with 2 / 3 / 4 / all that fit workgroups per compute unit:
        //   d = 128, 64 queries, 400 examples 348 / 376 / 390 / 390;  d = 32 (single heads), 900: 368 / 290 / 273 / 285
        // At d = 128 two are the best alone (bench batch 855 / 865 / 873 us), but not next to kernels that draw the clock
        // down, where two waves of a compute unit cannot keep up: in the benchmark step 887 / 833 / 838 us.
        // At d = 32 with 33..64 queries (heads that do not pair) the tanh and the polynomial form need all that fit: single heads, 900
        // examples of 64..1024 keys 157 / 161 us.
        const bool needs_waves = (!SMALL && has_act(p, KUNLUN_ACT_GELU)) ||
                                 (D == 32 && NW == 2 && (has_act(p, KUNLUN_ACT_GELU_TANH) || has_act(p, KUNLUN_ACT_GELU_POLY)));
        const int walkers = needs_waves ? per_cu : D == 32 ? 4 : 3;
        const int64_t resident = (int64_t)(per_cu < walkers ? per_cu : walkers) * compute_units();
        if (grid > resident) grid = resident;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW * KS), bytes, stream, p, n_qtiles, (int)n_items);
    return hipGetLastError();
}

bool mfma_fwd_is_qtiled(const AttnParams& p) { return p.windowed || p.max_q > 64; }

// How a launch is cut.  One wave per block of 32 queries leaves the time to the longest history and to the score function of a
// single wave when items are few, and makes many thin walks through memory when they are many; so waves share the key tiles of
// an item: four or eight when items are few, two or four when they are many (the four waves of an item read one stretch of
// memory together).  33..64 queries: the blocks of an item are either two items that read K and V once each (the second time
// out of the L2; few items), or both in the registers of one wave (`both`; not at d = 128, where the accumulators alone are 128
// registers: there a workgroup of two waves walks the whole history, items handed out by a counter).
// Longest first (one more kernel, 4 us): when the items do not all fit the device at once, and earlier with long histories.
// us, 8 heads, histories of 64..512 (t), 64..1024 (u), 256..2048 (v) and log-normal up to 4096 keys (l):
//   (at d = 32 a walk over the 64-byte pieces of one head, half memory lines, reads 3.75 TB/s; over the pieces of two 6.3)
//   Many items, softmax: one wave (33..64 queries: a workgroup of two) per item from a counter, single heads / the plan below:
//     d = 32   32 queries  4096 items t 72 / 37, u 96 / 60, v 162 / 111, l 168 / 116;  2048 l 72 / 64
//              64 queries  4096 items t 74 / 44, u 97 / 67, v 163 / 124, l 170 / 126;  2048 l 104 / 71
//     d = 64   32 queries  4096 items t 82 / 64, u 121 / 112, v 221 / 217, l 238 / 221
//              64 queries  4096 items t 84 / 70, u 126 / 115, v 229 / 224, l 247 / 231;  1024 u 41 / 38, v 79 / 63, l 109 / 74;
//                          256 u 22 / 14, v 38 / 23, l 47 / 38 (two items per (example, head); 171 l 34 / 40)
//     d = 128  20 queries  4096 items t 126 / 117, u 213 / 203, v 410 / 400;  3072 l 342 / 313
//   `both`, two / four / eight waves, unsorted, then sorted, d = 64, 64 queries:
//     1024 items l 99 / 87 / 89, 91 / 74 / 77;  v 78 / 70 / 76, 74 / 63 / 72;  512 v 42 / 43 / 44, 42 / 42 / 41, l 67 / 63 / 59, 63 / 52 / 48;
//     2048 u 67 / 65 / 92, 62 / 67 / 95
//   Few items, one wave per item / 4 waves / 8 waves, unsorted, then sorted:
//     64 queries  d = 128  softmax  256 items u 31 / 36 / 38, 35 / 35 / 36;  l 110 / 104 / 98, 111 / 80 / 73;  GELU 512 l 149 / 149 / 132, 153 / 117 / 117;
//                                   512 v, whole histories 76 / by four 122, by eight sorted 119: with even histories the split pays up to 256 items only
//                 d = 32   softmax  384 u 18 / 14 / 15;  768 u 20 / 23 / 25, 29 / 23 / 27;  1024 l 67 / 68 / 61, 73 / 52 / 54 (pairs, sorted, 47)
//     32 queries  d = 128 (one / 2 / 4 / 8)  softmax  512 u 36 / 34 / 35 / 38, 43 / 34 / 35 / 35;  768 t 27 / 27 / 29 / 36, 36 / 27 / 30 / 38;
//                          768 u 50 / 50 / 54 / 55, 58 / 48 / 47 / 53;  256 t 17 / 12 / 12 / 13
//                 d = 64   softmax  256 l 76 / 29 / 31, 82 / 33 / 34;  384 l 79 / 44 / 37, 85 / 39 / 37
//                 d = 32   ReLU     256 l 41 / 16 / 15, 47 / 19 / 18;  384 l 43 / 20 / 20, 50 / 21 / 21;  512 l 43 / 26 / 27, 51 / 23 / 23
//                          pairs / singles, softmax  512 l 32 / 26, 1024 l 43 / 41, 2048 u 34 / 32: pairs pay above
//   The lines themselves come from 800 random calls beside them, new form over old in time, by items (E: the longest history less than
//   2.5 times the mean; the three forms of GELU, "general" its exact form on scores that may be large):
//     pairs, up to 32 queries, long histories   E 1040..1720 1.03..1.12;  l 1036..1112 0.88..1.00, 1144..1270 softmax and SiLU 1.03..1.10, GELU 0.93..1.03,
//                                               1300..1450 GELU 0.91..1.07, 1464..1760 all 1.02..1.16
//     pairs, 33..64 queries                     long 1008..2256 1.13..1.66, general GELU to 1956 0.98..1.00;  short 1552..1800 1.06..1.22, tanh 0.93..1.02
//     `both` at d = 64                          E 212..464 1.3..1.7;  l 200..252 0.70..1.06, 256..508 1.05..1.44 but general GELU to 300 0.77, 416 1.04;
//                                               short 130..138 0.91..1.06, 142..300 1.02..1.53 but general GELU to 162 0.88..1.03, 168..288 0.96..1.21
//     one walk instead of eight waves, d = 128  33..64 queries, E 280..472 1.09..1.47 but GELU on small scores 274 0.94, in general 268..272 0.76, 368 0.95
//     four waves instead of eight, d = 128      up to 32 queries, E 784..1003 1.03..1.11;  l 776..928 0.90..0.99, 944..1017 1.00..1.03
FwdPlan mfma_fwd_plan(const AttnParams& p) {
    const bool cheap = !has_act(p, KUNLUN_ACT_GELU), general_gelu = !cheap && !small_scores_expected(p);
    const bool tanh_gelu = has_act(p, KUNLUN_ACT_GELU_TANH), any_gelu = !cheap || tanh_gelu || has_act(p, KUNLUN_ACT_GELU_POLY);
    const bool even = histories_are_even(p);
    const int d = p.d;
    const int64_t items = (int64_t)p.B * p.H, blocks = items * ((p.max_q + 31) / 32);
    const bool long_histories = p.max_kv > 1024;
    const bool all_fit = schedule_is_moot(items, 4);
    FwdPlan plan = {1, false, false, !all_fit || (long_histories && !schedule_is_moot(blocks, 1))};
    if (p.max_q <= 32) {
        plan.pair = heads_pair(p) && items > (!long_histories ? 2048 : even ? 1024 : any_gelu ? 1456 : 1216);
        if (blocks > 2048 && (plan.pair || d != 32)) {
            plan.key_split = long_histories ? 4 : 2;
            return plan;
        }
        if (blocks > 2048) return plan;
        plan.key_split = long_histories && blocks <= (d != 128 ? 1024 : even ? 768 : 936) ? 8 : 4;
        if (d == 128 && !long_histories) {
            const bool worth = p.max_kv > 512 && blocks > 512;  // (four waves crowd each other out below)
            plan.key_split = worth || blocks <= 256 ? 4 : 2;
            plan.sorted = plan.sorted || worth;
        }
        if (cheap && long_histories && (d == 64 ? blocks <= 256 : d == 32 && blocks > 256 && blocks <= 384)) {
            plan.key_split = 4;
            plan.sorted = false;
        }
        return plan;
    }
    plan.pair = heads_pair(p) && items > (general_gelu ? 2048 : long_histories ? 1000 : tanh_gelu ? 1800 : 1500);
    if (d == 64 && p.max_kv <= 256 && items > 512 && all_fit) return plan;  // (952 items of 64..256 keys, a workgroup of two / `both`: 12.5 / 13.7)
    const int both_limit = !long_histories ? (general_gelu ? 170 : 140) : even ? 192 : general_gelu ? 400 : 256;
    if (plan.pair || (d == 64 && items > both_limit)) {
        const int64_t units = plan.pair ? items / 2 : items;
        plan.both = true;
        if (long_histories)
            plan.key_split = units <= 256 ? 4 : units <= (p.max_kv > 2048 ? 768 : 512) ? 8 : units <= 2048 ? 4 : 2;
        else
            plan.key_split = units <= (p.max_kv > 512 ? 1024 : 512) ? 4 : 2;
        plan.sorted = !all_fit || (long_histories && units > 256);
        return plan;
    }
    const int64_t dear_limit = d == 32 ? 4096 : d == 64 ? (long_histories ? 2048 : 1024) : (long_histories ? (!even ? 1024 : general_gelu ? 800 : 600) : 512);
    const int64_t cheap_limit = d == 32 ? (long_histories || !all_fit ? 4096 : 768) : d == 64 ? (long_histories ? 1024 : 512) : (long_histories ? (even ? 512 : 1024) : 256);
    if (blocks <= (cheap ? cheap_limit : dear_limit))
        plan.key_split = long_histories && blocks <= (d == 32 ? 1536 : 2048) ? 8 : 4;
    else
        plan.sorted = !all_fit || (long_histories && (d == 128 ? items > 896 && !even : !cheap));
    return plan;
}

template <bool SMALL>
static hipError_t launch_streaming(const AttnParams& p, const FwdPlan& plan, hipStream_t stream) {
    // 32 queries per wave (64 where a wave has both blocks), up to 256 registers per wave, two or three waves per SIMD.
    const int ks = plan.key_split;
    if (p.d == 128) {
        if (ks == 8) return launch_gdpa<SMALL, 128, 1, 1, 1, 2, 1, 8>(p, stream);
        if (ks == 4) return launch_gdpa<SMALL, 128, 1, 1, 1, 2, 1, 4>(p, stream);
        if (ks == 2) return launch_gdpa<SMALL, 128, 1, 1, 1, 2, 1, 2>(p, stream);
        return launch_gdpa<SMALL, 128, 1, 1, 2, 2, 2, 1>(p, stream);
    }
    // Both blocks: one tile in flight per wave (a second takes 32 registers: spills with pairs, no gain without)
    if (plan.both && plan.pair) {
        if (ks == 8) return launch_gdpa<SMALL, 64, 2, 2, 1, 2, 1, 8>(p, stream);
        if (ks == 4) return launch_gdpa<SMALL, 64, 2, 2, 1, 2, 1, 4>(p, stream);
        return launch_gdpa<SMALL, 64, 2, 2, 1, 2, 1, 2>(p, stream);
    }
    if (plan.pair) {
        if (ks == 4) return launch_gdpa<SMALL, 64, 2, 1, 1, 2, 2, 4>(p, stream);
        return launch_gdpa<SMALL, 64, 2, 1, 1, 2, 2, 2>(p, stream);
    }
    if (plan.both) {
        if (ks == 8) return launch_gdpa<SMALL, 64, 1, 2, 1, 2, 1, 8>(p, stream);
        if (ks == 4) return launch_gdpa<SMALL, 64, 1, 2, 1, 2, 1, 4>(p, stream);
        return launch_gdpa<SMALL, 64, 1, 2, 1, 2, 1, 2>(p, stream);
    }
    if (p.d == 64) {
        if (ks == 8) return launch_gdpa<SMALL, 64, 1, 1, 1, 2, 2, 8>(p, stream);
        if (ks == 2) return launch_gdpa<SMALL, 64, 1, 1, 1, 2, 2, 2>(p, stream);
        if (ks == 1) return launch_gdpa<SMALL, 64, 1, 1, 2, 2, 2, 1>(p, stream);
        // Four waves: with the short form of GELU a kernel of 177 registers, two workgroups per compute unit; without it 162
        // and three, which is what counts for short histories (GELU, 768 items of 32 queries, 64..512 keys 17.2 / 15.9 us;
        // 1536 of 64..1024 keys 43.9 / 45.4 us)
        if (SMALL && p.max_kv > 512) return launch_gdpa<SMALL, 64, 1, 1, 1, 2, 2, 4>(p, stream);
        return launch_gdpa<false, 64, 1, 1, 1, 2, 2, 4>(p, stream);
    }
    if (ks == 8) return launch_gdpa<SMALL, 32, 1, 1, 1, 2, 2, 8>(p, stream);
    if (ks == 4) return launch_gdpa<SMALL, 32, 1, 1, 1, 2, 2, 4>(p, stream);
    return p.max_q <= 32 ? launch_gdpa<SMALL, 32, 1, 1, 1, 2, 2, 1>(p, stream) : launch_gdpa<SMALL, 32, 1, 1, 2, 2, 2, 1>(p, stream);
}

hipError_t launch_mfma_fwd(const AttnParams& p, hipStream_t stream) {
    // Query-tiled launches use 128-query tiles (4 waves): fewer K/V tile loads per query.
    if (mfma_fwd_is_qtiled(p)) return launch_mfma_fwd_qtiled(p, stream);
    const FwdPlan plan = mfma_fwd_plan(p);
    return short_gelu(p) ? launch_streaming<true>(p, plan, stream) : launch_streaming<false>(p, plan, stream);
}

}  // namespace kunlun
