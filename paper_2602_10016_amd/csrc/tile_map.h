// Work mapping of the tiled launches (query tiles of the forward kernel and of the backward
// dQ pass, key tiles of the backward dK/dV pass): grid = H * (tiles of all examples), cut into
// 8 contiguous ranges, one per XCD (workgroup i runs on XCD i % 8), so that the tiles of one
// (example, head) - which share their operands - meet in the same L2.  Items are ordered by
// example, then tile, then head.  tile_start[b] = number of tiles before example b and
// tile_example[t] = example of tile t (both written by the prefix kernel), so a workgroup finds
// its item with two dependent loads.
// Inside its range an XCD takes the items in order: a tile and its successor, H items further on, run side by side.  (Cut into
// `runs` contiguous runs that are issued in turn, a tile starts when its predecessor is one tile width into its window, and both
// read the rows they share at the same time.  That costs up to 8 % in large launches: sliding-window forward, 128 sequences of
// 256..2048, 4 heads, d = 128, previous 64: in order 120 us, 32 slots apart 131; 512 log-normal sequences, 8 heads, previous 64: 875 /
// 948, 255 to both sides 1656 / 1689.  In order over in turn, 3000 random forward calls: d = 32 1.02 at every size, d = 64 1.00 up to 2000
// tile-heads and 1.02 beyond, d = 128 1.02 up to 512, 0.99 from there to 1800 and 1.02 beyond; what is lost is lost in narrow windows over
// long sequences, 2.5 % in the mean and up to 6 from 1024 to 1792 tile-heads, and tile_runs() cuts those.)
#pragma once
#include "common.h"

namespace kunlun {

enum { BY_TABLES, BY_ORDER, BY_OFFSETS };  // how a workgroup finds its tile

constexpr int TILE_ROWS = 128;  // rows (queries or keys) per tile of every tiled launch: 4 waves x 32

inline size_t tile_table_bytes(int B, int64_t total_rows) {
    return align_up((size_t)(B + 1) * sizeof(int32_t), 256) +
           align_up((size_t)(total_rows / TILE_ROWS + B) * sizeof(int32_t), 256);
}
inline int32_t* tile_example_of(int32_t* tile_start, int B) {
    return (int32_t*)((char*)tile_start + align_up((size_t)(B + 1) * sizeof(int32_t), 256));
}
// grid size (an upper bound of the tile count sizes it; surplus workgroups exit at once)
inline unsigned tile_grid(int B, int H, int64_t total_rows, int runs = 1) {
    const int64_t per_xcd = ((total_rows / TILE_ROWS + B) * H + 7) / 8;
    return (unsigned)((per_xcd + runs) * 8);
}
// tiles times heads: half a tile more per example than its rows fill
inline int64_t tiles_expected(const AttnParams& p) { return (p.total_q / TILE_ROWS + (p.B + 1) / 2) * p.H; }
// The launches that number their tiles by the offsets instead (locate_spread_tile below).
// The numbers without a tile are up to one per example, and not the same share of every XCD: where the tiles fill so many rounds of
// `slots` workgroups and the numbers one more, some compute units get a round more than others.  Backward, by offsets over by tables: 34 to 64
// keys, 231 examples, 1 head (231 key tiles, 314 numbers) 119 / 97 us; few keys, 13 x 4 (496 chunks, 520) 27.0 / 24.3; windows 49.8 / 47.
// From the fifth round on it is not seen.
inline bool spread_keeps_rounds(int B, int H, int64_t total_rows, int max_rows, int tile_rows, int slots) {
    const int64_t numbers = (total_rows / tile_rows + B) * H;
    const int64_t tiles = (max_rows <= tile_rows ? B : total_rows / tile_rows + (B + 1) / 2) * H;
    return tiles > 4 * (int64_t)slots || (numbers + slots - 1) / slots <= (tiles - tiles / 32 + slots - 1) / slots;
}
inline unsigned spread_grid(int B, int H, int64_t total_rows, int tile_rows) {
    return (unsigned)((((total_rows / tile_rows + B) * H + 7) / 8 + 1) * 8);
}
// Runs per XCD of a forward launch: with about 96 workgroups resident there, a tile and its successor start 48 slots apart.
inline int tile_runs(const AttnParams& p) {
    const int64_t tiles = tiles_expected(p);
    if (!p.windowed || p.d != 128 || p.left < 0 || p.right < 0 || (int64_t)p.left + p.right > TILE_ROWS) return 1;
    if (tiles <= 1024 || tiles > 1792 || p.total_q < (int64_t)512 * p.B) return 1;
    const int want = 48 / p.H;
    return want < 1 ? 1 : (want > 32 ? 32 : want);
}
// Dense queries over histories of their own lengths (every example has the same number of query tiles, a tile takes as long as its
// history): examples in the issue order of the scheduler kernel, longest history first, dealt over the XCDs; the tiles of an
// (example, head), which read the same keys, next to each other on one XCD.  In the order of the tile tables every XCD has the
// histories of an eighth of the batch, whatever their sum, and a long one may start last.
inline int64_t dense_tiles(const AttnParams& p) { return (p.max_q + TILE_ROWS - 1) / TILE_ROWS; }
inline int64_t dense_tile_grid(const AttnParams& p) { return ((int64_t)p.B + 7) / 8 * 8 * p.H * dense_tiles(p); }
// Up to two workgroups per compute unit run at the same time in whatever order they are listed; short or even histories leave
// nothing to order, and the sorting kernel is a microsecond longer than that of the tile tables.  320 random calls with 65..400
// shared seeds, tables over sorted: log-normal histories 1.1 to 1.75 (forward) and 1.0 to 1.47 (backward at d = 32 and 64), 64..1024 keys up to
// 1.45 and 1.18, 900..1024 keys 0.96 to 1.0, 30..120 keys 0.91 to 0.97.  256 seeds over 256 log-normal histories, 8 heads, d = 128: forward 500 / 440 us.
inline bool dense_tiles_sorted(const AttnParams& p) {
    return !p.windowed && !p.q_off && p.max_kv > 256 && (int64_t)p.max_kv * p.B > 5 * p.total_kv / 4 && dense_tile_grid(p) > 2 * compute_units() &&
           dense_tile_grid(p) <= largest_grid(256);
}
// The forward at d = 128: more than 18 workgroups per compute unit, one for each example, over histories of up to eleven key tiles balance
// themselves in any order.  Tables over sorted, 850 random calls of up to 100000 examples: 0.93 to 1.05 (0.97 in the mean) up to 352 keys where the
// longest is at most 2.5 times the mean or there are more than 28 per compute unit (30000 examples of 66 seeds, 1 to 280 keys, 1 head: 551 / 595
// us), the others 0.98 to 1.7.
inline bool dense_tiles_sorted_fwd(const AttnParams& p) {
    const bool many_short = p.d == 128 && p.max_q <= TILE_ROWS && p.max_kv <= 352 && dense_tile_grid(p) > 18 * (int64_t)compute_units() &&
                            (2 * (int64_t)p.max_kv * p.B <= 5 * p.total_kv || dense_tile_grid(p) > 28 * (int64_t)compute_units());
    return dense_tiles_sorted(p) && !many_short;
}
#ifdef __HIPCC__
// Rank in the issue order of item group k (one example) of an XCD: dealt forth and back, so that no XCD has the longer one of every
// eight.
__device__ __forceinline__ int64_t dealt_rank(unsigned k, unsigned xcd) { return (int64_t)k * 8 + ((k & 1) ? 7 - xcd : xcd); }
__device__ __forceinline__ bool locate_dense_tile(const int32_t* __restrict__ order, int B, int H, int max_q, unsigned block, int& b, int& h, int& t) {
    const unsigned tiles = (unsigned)(max_q + TILE_ROWS - 1) / TILE_ROWS, slot = block >> 3;
    t = (int)(slot % tiles);
    h = (int)(slot / tiles % (unsigned)H);
    const int64_t e = dealt_rank(slot / tiles / (unsigned)H, block & 7);
    if (e >= B) return false;
    b = order[e];
    return true;
}
__device__ __forceinline__ bool locate_tile(const int32_t* __restrict__ tile_start,
                                            const int32_t* __restrict__ tile_example, int B, int H, unsigned block,
                                            int& b, int& h, int& t, int runs = 1) {
    const int64_t n_items = (int64_t)tile_start[B] * H;
    const int64_t per_xcd = (n_items + 7) / 8;
    const int xcd = block & 7;
    int64_t in_xcd = block >> 3;
    if (runs > 1) {
        const unsigned slot = block >> 3, run_len = ((unsigned)per_xcd + runs - 1) / runs;
        if (slot >= run_len * runs) return false;
        in_xcd = (slot % runs) * run_len + slot / runs;
    }
    if (in_xcd >= per_xcd) return false;
    const int64_t item = xcd * per_xcd + in_xcd;
    if (item >= n_items) return false;
    const int tile = (int)(item / H);
    h = (int)(item % H);
    b = tile_example[tile];
    t = tile - tile_start[b];
    return true;
}

// The same mapping without tables, for long sequences: tile numbers are dealt by the offsets themselves, example b beginning at
// off[b] / tile_rows + b (never fewer numbers than it has tiles; a number without a tile ends its workgroup).  Every wave finds the
// example by itself, 64 probes of the offsets at a time: as many dependent loads as the tables take up to 4096 examples, and no
// launch in front.
constexpr int SPREAD_STEPS = 3;  // 64^3 examples; launches with as many as 8192 take this path (half a tile each in tiles_expected())
__device__ __forceinline__ int spread_tile(const int32_t* __restrict__ off, int b, int tile_rows) { return off[b] / tile_rows + b; }
__device__ __forceinline__ bool locate_spread_tile(const int32_t* __restrict__ off, int B, int H, int64_t total, int tile_rows, unsigned block,
                                                   int& b, int& h, int& t) {
    const int64_t n_items = (total / tile_rows + B) * H;
    const int64_t per_xcd = (n_items + 7) / 8;
    const int64_t in_xcd = block >> 3, item = (block & 7) * per_xcd + in_xcd;
    if (in_xcd >= per_xcd || item >= n_items) return false;
    const int tile = (int)(item / H);
    h = (int)(item % H);
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = B;  // the example is in [lo, hi)
    // Steps of a known number, and the result as scalars: with a loop of unknown length in front of the item the forward kernels take
    // 191 / 133 / 108 registers (d = 128 / 64 / 32) instead of 160 / 102 / 77, two, three and four workgroups per compute unit instead of
    // three, four and six.
#pragma unroll
    for (int i = 0; i < SPREAD_STEPS; ++i) {
        if (hi - lo <= 1) break;
        const int step = (hi - lo + 63) / 64, probe = lo + lane * step;
        const int before = __builtin_popcountll(__builtin_amdgcn_ballot_w64(probe < hi && spread_tile(off, probe < hi ? probe : lo, tile_rows) <= tile));
        lo += (before > 0 ? before - 1 : 0) * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    b = __builtin_amdgcn_readfirstlane(lo);
    t = __builtin_amdgcn_readfirstlane(tile) - spread_tile(off, b, tile_rows);
    h = __builtin_amdgcn_readfirstlane(h);
    return t >= 0 && (int64_t)t * tile_rows < off[b + 1] - off[b];
}

// Exclusive prefix sum of ceil(len_b / tile_rows) over the examples, and the example of every
// tile; single workgroup of 1024 threads.  off == null: every example has `dense_len` rows.
// tile_rows is TILE_ROWS or a multiple of it (a workgroup that walks several tiles).
// (A template only so that every translation unit that launches it carries its own copy.)
template <int UNUSED>
__global__ __launch_bounds__(1024) void tile_prefix_kernel(const int32_t* __restrict__ off, int dense_len, int B,
                                                           int32_t* __restrict__ tile_start,
                                                           int32_t* __restrict__ tile_example, int tile_rows) {
    __shared__ int totals[16];
    const int tid = threadIdx.x;
    const int per = (B + 1023) / 1024;
    const int b0 = tid * per, b1 = (b0 + per < B) ? b0 + per : B;
    auto tiles_of = [&](int b) { return ((off ? off[b + 1] - off[b] : dense_len) + tile_rows - 1) / tile_rows; };
    int sum = 0;
    for (int b = b0; b < b1; ++b) sum += tiles_of(b);
    const int upto = scan1024(sum, totals);
    int run = upto - sum;
    for (int b = b0; b < b1; ++b) {
        tile_start[b] = run;
        const int n = tiles_of(b);
        for (int t = 0; t < n; ++t) tile_example[run + t] = b;
        run += n;
    }
    if (tid == 1023) tile_start[B] = upto;
}
#endif  // __HIPCC__

}  // namespace kunlun
