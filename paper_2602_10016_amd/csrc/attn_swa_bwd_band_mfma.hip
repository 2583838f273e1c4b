// One-pass bf16 matrix-core backward of sliding-window self-attention (Eq. (sliding window)) at head dimension 128, for windows that
// put at most nine key tiles of 32 under a query tile: dQ, dK, dV of <O, dO>, every score computed once, every row loaded once.
//
// One workgroup of 8 wavefronts (one per compute unit) walks a sequence of one head from front to back, one 32-query tile per
// step.  Wave w owns the key tiles j = w mod 8, one at a time, while they are under the window: K_j^T and V_j^T fragments and
// the dK_j, dV_j accumulators live in its registers.  Step i:
//     the half of the waves that takes up no key tile in this step adds up dQ of step i - 1, one 32-channel block per wave:
//         dQ_{i-1}^T = sum over the key tiles under the window of K_j^T dS_{i-1,j}   (both operands from LDS, where the K tiles under the
//         window stay in a ring of ten) -> dQ rows, done
//     every wave, for its key tile:  S = Q K^T,  dP = dO V^T,  P and dS in registers (one key per lane),
//         dV^T += dO^T P,  dK^T += Q^T dS,  and behind a barrier (dQ_{i-1} is done) a bf16 image of dS, [key][query], to LDS
//     two waves of the other half have sent the loads of step i + 1 at the start (buffer-load-to-LDS, lds_ring.h) and wait for them
//         here; they compute delta = rowsum(dO * O) of the rows that they loaded themselves;  barrier
// Every sum is made in the order of the two-pass kernels, so that a sequence has the same gradients to the bit whatever batch it comes in.
// A window of nine tiles (256 rows) makes one wave a step hand its key tile over: it finishes tile i - L, sends out its rows and
// takes tile i + R (L, R: tiles to the left and right) within the step.
//
// What bounds it: the chain of a step, not bytes or flops.  Previous 256, 128 sequences of 256..2048 rows, 4 heads: 73 steps per
// compute unit in the mean, 4.7 us each (at nine tiles the longest chain is that of the wave that finishes one key tile, sends out its
// rows and takes the next): 340 to 359 us = 3.5 TB/s and 490 TFLOP/s (ten flops per pair and channel).  The two-pass kernels
// (attn_bwd_tiled_mfma.hip), which compute S and dP twice and load every row of the window for each tile of 64, take 470 to 485.  Windows of
// two to five tiles: 266 to 278 against 352 to 388.  Tried with sums in another order (2 % faster in the whole kernel): at d = 64 the same
// kernel gains nothing (230 against 260 us at nine tiles, 205 against 208 at five), at d = 32 it loses, as the chain does not shrink with
// the bytes; rows through LDS instead of straight from registers (whole rows per store instruction) and the masks beside the matrix
// instructions changed less than 2 %.
#include <type_traits>

#include "lds_ring.h"
#include "tile_map.h"

namespace kunlun {

#define PIN() __builtin_amdgcn_sched_barrier(0)  // nothing is moved across by the instruction scheduler

constexpr float LOG2E_B = 1.4426950408889634f;
constexpr int SWB_WAVES = 8;
constexpr int SWB_LOADERS = 2;  // waves that load a step's query tiles
constexpr int SWB_MAX_TILES = SWB_WAVES + 1;  // key tiles under a query tile

struct SwbSmem {
    static constexpr int D = 128;
    static constexpr int TILE = KT * D * 2;
    static constexpr int RING = SWB_MAX_TILES + 1;  // K tiles under the window, and the next one on its way
    static constexpr int IMAGE = KT * KT * 2;
    static constexpr int STATS = 2 * KT * 4;        // of a query tile: -lse log2 e, then delta
    static constexpr int V = RING * TILE;           // two tiles: read by its owner when it takes up the key tile
    static constexpr int QD = V + 2 * TILE;         // two stages of a Q and a dO tile
    static constexpr int O = QD + 4 * TILE;
    static constexpr int IMAGES = O + TILE;         // dS, the slots of the K ring
    static constexpr int ST = IMAGES + RING * IMAGE;  // two stages of statistics
    static constexpr int LSE = ST + 2 * STATS;      // lse as loaded, for each loading wave
    static constexpr int TOTAL = LSE + SWB_LOADERS * 256;  // d = 128: 157 KB
};

// A 32 x 32 block in the C layout (lane: output row r, registers: channels 8*(v/4) + 4g + v%4) to bf16 rows of the buffer, 16
// bytes per lane: the lane halves exchange the channels that make them whole.  voff: r * row_bytes + channel block + 16 g bytes.
__device__ __forceinline__ void store_block_rows(const f32x16& acc, const __amdgpu_buffer_rsrc_t rsrc, uint32_t voff) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        bf16x4 a, b;
#pragma unroll
        for (int e = 0; e < 4; ++e) { a[e] = (bf16_t)acc[8 * p + e]; b[e] = (bf16_t)acc[8 * p + 4 + e]; }
        const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
        const auto s0 = __builtin_amdgcn_permlane32_swap(ua[0], ub[0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(ua[1], ub[1], false, false);
        const u32x4 x = {s0[0], s1[0], s0[1], s1[1]};
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, voff, 32 * p, 0);
    }
}

__device__ __forceinline__ void swa_bwd_band_item(const AttnParams& p, char* lds, int h, int64_t row0, int n, int L_tiles, int R_tiles) {
    using SM = SwbSmem;
    constexpr int D = SM::D;
    using L = TileLayout<D>;
    constexpr int KC = D / 16, DB = D / 32;
    // Accumulators and fragments leave no registers for all of K_j^T: the last fragments are read from the ring.
    constexpr int K_REG = KC - 3;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t hd = (int64_t)p.H * D;
    const uint32_t row_bytes = (uint32_t)(hd * 2);
    const int64_t tile_bytes = (int64_t)KT * row_bytes;
    const int64_t base = (row0 * p.H + h) * D * 2;
    const char* Q = (const char*)p.q + base;
    const char* K = (const char*)p.k + base;
    const char* V = (const char*)p.v + base;
    const char* O = (const char*)p.o + base;
    const char* DO = (const char*)p.d_o + base;
    const uint32_t lds0 = lds_address(lds);
    const int nt = (n + KT - 1) / KT;
    L_tiles = L_tiles < nt - 1 ? L_tiles : nt - 1;  // (a reach past the sequence's other end would only add steps without a key tile)
    R_tiles = R_tiles < nt - 1 ? R_tiles : nt - 1;
    const float sc = p.scale * LOG2E_B;

    const u32x4 lse_rsrc = make_rsrc_words(p.lse + (int64_t)h * p.total_q + row0, (uint32_t)n * 4);
    using DmaQ = TileDma<D, SWB_LOADERS, SWZ_U>;
    constexpr int ROWS = DmaQ::RPI * DmaQ::IPW;  // rows of a query tile that a wave loads, one after the other
    using DmaK = TileDma<D, SWB_WAVES / 2, SWZ_U>;
    // Q, dO, O and lse of query tile i, by SWB_LOADERS waves
    auto issue_queries = [&](int i, int part) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // (what the addresses derive from it is computed here and not kept across the loop)
        DmaQ dma;
        dma.init(lane, part, row_bytes);
        const uint32_t qd = lds0 + SM::QD + (i & 1) * 2 * SM::TILE;
        dma.issue(Q + i * tile_bytes, n - i * KT, qd);
        dma.issue(DO + i * tile_bytes, n - i * KT, qd + SM::TILE);
        dma.issue(O + i * tile_bytes, n - i * KT, lds0 + SM::O);
        const int qi = i * KT + lane;
        load_to_lds_b32(lse_rsrc, (uint32_t)(qi < n ? qi : n - 1) * 4, 0, lds0 + SM::LSE + part * 256);
    };
    // K and V of key tile j, by four waves
    auto issue_keys = [&](int j) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        DmaK dma;
        dma.init(lane, wave & 3, row_bytes);
        dma.issue(K + j * tile_bytes, n - j * KT, lds0 + (j % SM::RING) * SM::TILE);
        dma.issue(V + j * tile_bytes, n - j * KT, lds0 + SM::V + (j & 1) * SM::TILE);
    };
    // statistics of the rows of query tile i that this wave loaded (its own loads have arrived)
    auto row_stats = [&](int i, int part) {
        asm volatile("" : : : "memory");  // (no LDS read moves up across the wait for the loads)
        PIN();
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const char* dot = lds + SM::QD + (i & 1) * 2 * SM::TILE + SM::TILE;
        float* st = (float*)(lds + SM::ST + (i & 1) * SM::STATS);
        // Two neighbouring lanes per row and half (every other 8 channels): each multiplies half of the channels, and the even one adds all
        // of them up in the order of the two-pass kernels (a product of two bf16 is exact).
        const int row = part * ROWS + (lane >> 1) % ROWS, odd = lane & 1, at = L::u_offset(row, (lane >> 5) * 16) ^ (odd * (KC / 2) << 5);
        const float lse = *(const float*)(lds + SM::LSE + part * 256 + row * 4);
        float term[KC / 2 * 8], sum = 0.f;
#pragma unroll
        for (int kc = 0; kc < KC / 2; ++kc) {
            const bf16x8 of = *(const bf16x8*)(lds + SM::O + (at ^ (kc << 5)));
            const bf16x8 df = *(const bf16x8*)(dot + (at ^ (kc << 5)));
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += term[kc * 8 + e] = (float)of[e] * (float)df[e];
        }
#pragma unroll
        for (int x = 0; x < KC / 2 * 8; ++x)  // quad_perm [1,0,3,2]: the neighbour's
            sum += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, term[x]), 0xB1, 0xf, 0xf, true));
        sum = halves_sum(sum);
        if (lane < 2 * ROWS && !odd) {
            st[row] = lse * -LOG2E_B;
            st[KT + row] = sum;
        }
    };

    f32x16 dkacc[DB], dvacc[DB];
    bf16x8 kf[K_REG], vf[KC];
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    const int i0 = -R_tiles;  // (the steps before the first query tile only take up key tiles)
    int cur = -1;             // key tile of this wave
    int next = wave;          // and the one after it
    constexpr int LOADS = 3 * DmaQ::IPW + 1, STORES = 4 * DB;  // of a query tile; of dK and dV rows (dQ rows are two)
    int behind = 0;           // vector-memory operations of this wave behind its last loads of a key tile (-1: it has none in flight)
    // In every step the waves meet where dQ of the last step is done and its images are free, and the key tile that the widest
    // window takes up in this step has arrived.
    auto meet = [&]() {
        if (behind == 2) wait_vmcnt<2>();
        else if (behind == LOADS) wait_vmcnt<LOADS>();
        else if (behind == STORES) wait_vmcnt<STORES>();
        else if (behind >= 0) wait_vmcnt<0>();
        __syncthreads();
    };
    bf16x8 dsf[2];
    // one query tile under this wave's key tile; dS stays in dsf
    auto unit = [&](int i, auto first) {
        const char* ldsQ = lds + SM::QD + (i & 1) * 2 * SM::TILE;
        const char* ldsDO = ldsQ + SM::TILE;
        const float* stats = (const float*)(lds + SM::ST + (i & 1) * SM::STATS);
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int r = lane & 31, g = lane >> 5;
        UFrag<D> uf;
        uf.init(lane);
        const int slot = cur % SM::RING;
        const char* ldsK = lds + slot * SM::TILE;
        // S = Q K^T, then dP = dO V^T: lane = key column, registers = queries of the tile.
        // The matrix instructions of dP run beside the exponentials of S; fragments are read AHEAD instructions before their use.
        constexpr int AHEAD = 3;
        f32x16 sacc, dpacc;
        bf16x8 fr[AHEAD], kr = kf[0];
        f32x4 lse[2], del[4];
        auto stat = [&](int vg, int which) { return *(const f32x4*)(stats + which * KT + 8 * vg + 4 * g); };
        auto frag = [&](int j) { return j < KC ? uf.row(ldsQ, j) : uf.row(ldsDO, j - KC); };
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) fr[j] = frag(j);
        PIN();
        float pv[16], dsv[16];
#pragma unroll
        for (int j = 0; j < 2 * KC; ++j) {
            if (j < KC) sacc = mfma32(fr[j % AHEAD], j < K_REG ? kf[j < K_REG ? j : 0] : kr, j == 0 ? zero16 : sacc);
            else dpacc = mfma32(fr[j % AHEAD], vf[j < KC ? 0 : j - KC], j == KC ? zero16 : dpacc);
            if (j + 1 >= K_REG && j + 1 < KC) kr = uf.row(ldsK, j + 1);
            if (j + AHEAD < 2 * KC) fr[j % AHEAD] = frag(j + AHEAD);
            if (j >= KC) {
                constexpr int W = 16 / KC;  // weights beside each matrix instruction
#pragma unroll
                for (int v = W * (j - KC); v < W * (j - KC) + W; ++v) pv[v] = fast_exp2(fmaf(sacc[v], sc, lse[(v >> 2) & 1][v & 3]));
            }
            if (j >= KC - 2 && j % 2 == 0 && j < 2 * KC - 2) lse[((j - KC + 2) >> 1) & 1] = stat((j - KC + 2) >> 1, 0);
            if (j >= 2 * KC - 3) del[j - 2 * KC + 3] = stat(j - 2 * KC + 3, 1);
            PIN();
        }
        del[3] = stat(3, 1);
        PIN();
#pragma unroll
        for (int v = 0; v < 16; ++v) dsv[v] = pv[v] * (dpacc[v] - del[v >> 2][v & 3]) * p.scale;
        // Interior tiles - every (query, key) pair inside the sequence and the window - skip the visibility test.
        // (Padding key lanes repeat the last key and are never stored.)
        const int q_base = i * KT, k_lo = cur * KT, k_hi = k_lo + KT - 1;
        bool need_mask = q_base + KT > n || k_hi >= n;
        if (p.right >= 0 && q_base < k_hi - p.right) need_mask = true;
        if (p.left >= 0 && q_base + KT - 1 > k_lo + p.left) need_mask = true;
        if (need_mask) {
            const int kp = k_lo + r;  // queries that see this lane's key: q_lo .. q_hi
            int q_lo = 0, q_hi = n - 1;
            if (p.right >= 0 && kp - p.right > 0) q_lo = kp - p.right;
            if (p.left >= 0 && kp + p.left < q_hi) q_hi = kp + p.left;
            const bool empty = q_hi < q_lo || kp >= n;
            const unsigned rel0 = (unsigned)(q_base + 4 * g - (empty ? 0x3fffffff : q_lo));
            const unsigned q_span = empty ? 0u : (unsigned)(q_hi - q_lo);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool ok = rel0 + (unsigned)(8 * (v >> 2) + (v & 3)) <= q_span;
                pv[v] = ok ? pv[v] : 0.f;
                dsv[v] = ok ? dsv[v] : 0.f;
            }
        }
        bf16x8 pf[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) { pf[c][e] = (bf16_t)pv[8 * c + e]; dsf[c][e] = (bf16_t)dsv[8 * c + e]; }
        PIN();
        // dV^T += dO^T P and dK^T += Q^T dS (contraction over the queries of the tile)
        constexpr int TA = 6;
        auto tfrag = [&](int j) { return uf.transposed((j & 1) ? ldsQ : ldsDO, j >> 2, (j >> 1) & 1); };
        bf16x8 tf[TA];
#pragma unroll
        for (int j = 0; j < TA; ++j) tf[j] = tfrag(j);
        PIN();
#pragma unroll
        for (int j = 0; j < 4 * DB; ++j) {
            const int db = j >> 2, c = (j >> 1) & 1;
            const bool zero = decltype(first)::value && c == 0;  // nothing in the accumulators yet
            if (j & 1) dkacc[db] = mfma32(tf[j % TA], dsf[c], zero ? zero16 : dkacc[db]);
            else dvacc[db] = mfma32(tf[j % TA], pf[c], zero ? zero16 : dvacc[db]);
            if (j + TA < 4 * DB) tf[j % TA] = tfrag(j + TA);
            PIN();
        }
    };
    auto put_image = [&](int tile) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        char* image = lds + SM::IMAGES + (tile % SM::RING) * SM::IMAGE;
        const int iw0 = w64_offset(lane & 31, 8 * (lane >> 5));  // key r, queries 8 vg + 4g .. -> ^ (vg << 4)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
            const int c = vg >> 1;
            *(bf16x4*)(image + (iw0 ^ (vg << 4))) =
                (vg & 1) ? __builtin_shufflevector(dsf[c], dsf[c], 4, 5, 6, 7) : __builtin_shufflevector(dsf[c], dsf[c], 0, 1, 2, 3);
        }
    };
    // dK and dV rows of this wave's key tile
    auto retire = [&]() {
        const int k_lo = cur * KT;
        const int rows = n - k_lo < KT ? n - k_lo : KT;
        int out_lane = threadIdx.x & 63;
        asm volatile("" : "+v"(out_lane));
        const uint32_t voff = (uint32_t)(out_lane & 31) * row_bytes + (out_lane >> 5) * 16;
        const uint32_t bytes = (uint32_t)(rows - 1) * row_bytes + D * 2;  // rows past the sequence are dropped
        const __amdgpu_buffer_rsrc_t rdv = __builtin_amdgcn_make_buffer_rsrc((char*)p.dv + base + cur * tile_bytes, 0, bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rdk = __builtin_amdgcn_make_buffer_rsrc((char*)p.dk + base + cur * tile_bytes, 0, bytes, 0x00020000);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            store_block_rows(dvacc[db], rdv, voff + db * 64);
            store_block_rows(dkacc[db], rdk, voff + db * 64);
        }
        cur = -1;
    };

    // dQ rows of query tile i, a channel block per wave
    auto query_gradient = [&](int i) {
        static_assert(DB == 4, "a channel block per helping wave");
        const int db = wave & 3;
        const int j0 = i - L_tiles > 0 ? i - L_tiles : 0, j1 = i + R_tiles < nt - 1 ? i + R_tiles : nt - 1;
        int dq_lane = threadIdx.x & 63;
        asm volatile("" : "+v"(dq_lane));
        const int s16 = dq_lane & 15, r = dq_lane & 31, g = dq_lane >> 5;
        const int colb = (16 * ((dq_lane >> 4) & 1) + 4 * (s16 & 3)) * 2;
        // (the keys of a matrix instruction in the order of the two-pass kernels, which have them from the C layout)
        int ka = L::u_offset(4 * g + (s16 >> 2), colb) ^ (db << 6), kb = L::u_offset(8 + 4 * g + (s16 >> 2), colb) ^ (db << 6);
        int ia = w64_offset(4 * g + (s16 >> 2), colb), ib = w64_offset(8 + 4 * g + (s16 >> 2), colb);
        // two matrix instructions per key tile; their operands are read two tiles ahead (past the window: slots that
        // are not used)
        bf16x8 kfr[4], ifr[4];
        int slot = j0 % SM::RING;
        auto fetch = [&](int x) {
            const int c = x & 1;
            const char* kt = lds + slot * SM::TILE + c * 16 * L::ROW_BYTES;
            const char* im = lds + SM::IMAGES + slot * SM::IMAGE + c * 16 * 64;
            kfr[x] = tr_pair(kt + ka, kt + kb);
            ifr[x] = tr_pair(im + ia, im + ib);
            if (c == 1) slot = slot == SM::RING - 1 ? 0 : slot + 1;
        };
        f32x16 acc = zero16;
#pragma unroll
        for (int x = 0; x < 4; ++x) fetch(x);
        PIN();
#pragma unroll 1
        for (int left = j1 - j0 + 1; left > 0; left -= 2) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (x < 2 || left > 1) acc = mfma32(kfr[x], ifr[x], acc);
                fetch(x);
                PIN();
            }
        }
        const int rows = n - i * KT < KT ? n - i * KT : KT;
        const __amdgpu_buffer_rsrc_t rdq =
            __builtin_amdgcn_make_buffer_rsrc((char*)p.dq + base + i * tile_bytes, 0, (uint32_t)(rows - 1) * row_bytes + D * 2, 0x00020000);
        store_block_rows(acc, rdq, (uint32_t)r * row_bytes + g * 16 + db * 64);
    };

    // Key tiles are loaded a step before they are taken up; where the widest window has no slot for that yet, at the end of it, which
    // is soon enough: its waves take them up late in their step.
    const bool early = L_tiles + R_tiles + 1 < SWB_MAX_TILES;
    if (wave >= SWB_WAVES / 2) issue_keys(0);
    if (wave < SWB_LOADERS && i0 >= 0) issue_queries(i0, wave);
    wait_vmcnt<0>();
    if (wave < SWB_LOADERS && i0 >= 0) row_stats(i0, wave);
    __syncthreads();
    for (int i = i0; i < nt; ++i) {
        // the half of the waves without the one that takes up a key tile computes dQ of the last step
        const int taker = (i + R_tiles) & (SWB_WAVES - 1);
        const bool helper = (wave ^ taker) >> 2;
        // two of its neighbours load for the next step.  (Helpers, loaders and the taker are different waves, and the wave that sends out
        // its rows in front of the meeting is the taker, so that `behind` counts one kind of operation.)
        const int part = i + 1 >= 0 && i + 1 < nt && !helper ? ((wave - taker) & 3) - 1 : -1;
        const bool loader = part >= 0 && part < SWB_LOADERS;
        const bool keys = helper && i + 1 + R_tiles < nt;
        behind = !helper && early ? -1 : loader ? LOADS : 0;
        if (loader) issue_queries(i + 1, part);
        if (helper) {
            if (keys && early) issue_keys(i + 1 + R_tiles);
            if (i > 0) {
                query_gradient(i - 1);
                behind = 2;
            }
        }
        const int tile = cur;
        const bool under = cur >= 0 && i >= 0 && cur + L_tiles >= i;
        if (under) unit(i, std::false_type{});
        if (!early && cur >= 0 && cur + L_tiles <= i) {
            retire();
            if (behind >= 0) behind += STORES;
        }
        const bool takes = next == i + R_tiles && next < nt;
        bool met = false;
        if (under || !takes || !early) {
            meet();
            met = true;
            if (under) put_image(tile);
            if (early && cur >= 0 && cur + L_tiles <= i) retire();
        }
        if (takes) {
            cur = next;
            next += SWB_WAVES;
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));
            UFrag<D> uf;
            uf.init(lane);
            const char* kt = lds + (cur % SM::RING) * SM::TILE;
            const char* vt = lds + SM::V + (cur & 1) * SM::TILE;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                if (kc < K_REG) kf[kc < K_REG ? kc : 0] = uf.row(kt, kc);
                vf[kc] = uf.row(vt, kc);
            }
            if (i >= 0) {
                unit(i, std::true_type{});
                if (!met) meet();
                met = true;
                put_image(cur);
            } else {
#pragma unroll
                for (int db = 0; db < DB; ++db) { dkacc[db] = zero16; dvacc[db] = zero16; }
            }
        }
        if (!met) meet();
        if (keys && !early) issue_keys(i + 1 + R_tiles);
        if (loader) {
            wait_vmcnt<0>();
            row_stats(i + 1, part);
        }
        __syncthreads();  // the dS images are complete, and step i + 1 is in LDS
    }
    if (wave < DB) query_gradient(nt - 1);
    if (cur >= 0) retire();  // (the key tiles that are still under the window of the last query tile)
}

// One workgroup per (sequence, head), longest sequence first; the heads of a sequence on one XCD (workgroup i runs on XCD i % 8).
__global__ __launch_bounds__(64 * SWB_WAVES, 2) void swa_bwd_band_kernel(AttnParams p, int L_tiles, int R_tiles) {
    extern __shared__ __attribute__((aligned(1024))) char swb_lds[];
    const unsigned slot = blockIdx.x >> 3;
    const int h = (int)(slot % (unsigned)p.H);
    const int64_t e = dealt_rank(slot / (unsigned)p.H, blockIdx.x & 7);
    if (e >= p.B) return;
    const int b = p.order[e];
    const int64_t row0 = p.kv_off[b];
    const int n = p.kv_off[b + 1] - (int)row0;
    if (n <= 0) return;
    swa_bwd_band_item(p, swb_lds, h, row0, n, L_tiles, R_tiles);
}

static int64_t band_items(const AttnParams& p) { return (((int64_t)p.B + 7) / 8) * 8 * p.H; }
static int64_t tiles_reached(int reach, int max_len) { return ((int64_t)(reach < 0 || reach > max_len ? max_len : reach) + KT - 1) / KT; }

// A step takes as long whatever the other compute units do, so a launch lasts as long as the compute unit with the most steps, where the
// two-pass kernels spread the tiles of every sequence.  In units of the mean: the longest sequence, or, for lengths that are nearly
// equal, the rounds that they leave incomplete.  One pass against two, 220 random launches: with up to 1.2 times the mean 1.14 to 1.39
// times as fast, at 1.35 1.14 (three tiles), at 1.45 1.17 (nine) and 1.06 (three to five), at 1.6 0.95 (two) and 1.09 (nine), at 1.9
// 0.8 to 0.95.
bool swa_bwd_band_applies(const AttnParams& p, int dtype) {
    if (!p.windowed || dtype != KUNLUN_BF16 || p.d != SwbSmem::D) return false;
    const int64_t tiles = tiles_reached(p.left, p.max_kv) + tiles_reached(p.right, p.max_kv) + 1;
    if (tiles > SWB_MAX_TILES || band_items(p) > largest_grid(64 * SWB_WAVES)) return false;
    const float units = (float)compute_units(), items = (float)p.B * p.H / units;
    const float longest = (float)p.max_kv, each = (float)p.total_q / p.B, mean = items * each;
    // Sequences of a few tiles: a workgroup of 157 KB is a prologue to most of its item, and the steps in front of the first query tile, one for
    // each tile that the window reaches to the right, are a good part of its steps (`lead`).  One pass over two, 1191 random launches over
    // sequences of up to 320 rows:
    //     up to 128 rows, and the two passes run as small launches                                     0.85 (0.63 to 1.12)
    //     up to 128 rows, 9 to 16 items per compute unit of 48 rows and more, 13 to 20 of 33 to 47     0.99 (0.89 to 1.16)
    //     lead of 0.3 and more, 9 to 21 and 13 to 25 of these items                                    0.96 (0.84 to 1.16)
    //     lead of 0.6 and more                                                                         0.93 (0.79 to 1.25)
    //     any lead, 5 to 8 items of 80 rows and more                                                   0.95 (0.84 to 1.12)
    //     the others                                                                                   1.15 (30 of 928 below 0.97)
    if (p.max_kv <= 8 * KT) {
        const int64_t first = tiles_reached(p.right, p.max_kv), tiles_each = tiles_reached((int)each, p.max_kv);
        const float lead = tiles_each > 0 ? (float)(first < tiles_each - 1 ? first : tiles_each - 1) / tiles_each : 0.f;
        const float from = each < 48 ? 12.f : 8.f, to = (each < 48 ? 20.f : 16.f) + (lead >= 0.3f ? 5.f : 0.f);
        const bool between = each >= 33 && items > from && items <= to;
        if (p.max_kv <= 4 * KT && (between || mfma_bwd_tiled_small_window(p))) return false;
        if (lead >= 0.6f || (lead >= 0.3f && between) || (lead > 0 && each >= 80 && items > 4 && items <= 8)) return false;
    }
    // the rounds that equal lengths leave incomplete
    const float shortest = fmaxf(0.f, 2.f * each - longest);
    const float whole = fmaxf(longest, mean + shortest * (ceilf(items) - items));
    return whole <= (tiles >= SWB_WAVES ? 1.5f : 1.35f) * mean;
}

// p.order: the sequences, longest first.
hipError_t launch_swa_bwd_band(const AttnParams& p, hipStream_t stream) {
    constexpr int bytes = SwbSmem::TOTAL;
    // once per process (thread-safe initialisation of a function-local static); not a stream operation
    static const hipError_t raised = hipFuncSetAttribute((const void*)swa_bwd_band_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (raised != hipSuccess) return raised;
    hipLaunchKernelGGL(swa_bwd_band_kernel, dim3((unsigned)band_items(p)), dim3(64 * SWB_WAVES), bytes, stream, p,
                       (int)tiles_reached(p.left, p.max_kv), (int)tiles_reached(p.right, p.max_kv));
    return hipGetLastError();
}

}  // namespace kunlun
