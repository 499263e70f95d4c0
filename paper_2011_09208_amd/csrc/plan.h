// Which kernels a call takes, how its work is cut and what scratch it wants: functions of its sizes alone.  Host code, in a header
// of its own so that the tests can compile it without the kernels.
#pragma once
#include <algorithm>
#include <stddef.h>
#include <stdint.h>

#include "gemm_block.h"
#include "gemm_core.h"
#include "gemm_small.h"
#include "gemm_stream.h"
#include "gemm_tiles.h"

namespace ws {

// n / d is the high half of n * inverse(d) as long as n * d < 2^32 and d > 1; there is no such number for 1, and 0 stands for it.
static inline uint32_t inverse(uint32_t d) { return d > 1 ? (uint32_t)((((uint64_t)1 << 32) + d - 1) / d) : 0; }
__host__ __device__ inline uint32_t quotient(uint32_t n, uint32_t inv) { return inv == 0 ? n : (uint32_t)(((uint64_t)n * inv) >> 32); }

// How the list kernels cut the logits: each of `ranges` columns of workgroups (one for every batch tile) takes every ranges-th of
// the first full * ranges whole class tiles and one part of the rest, `per` units of 32 classes, the first `more` of them one more
// (whole k-steps of the dX contraction in all).  What the kernels divide by comes as its inverse.
struct RangePlan {
    int ranges, full, per, more;
    uint32_t inv_block, inv_rest;        // of a block of batch tiles (`ranges` times four of them), of the batch tiles of the last block
    uint32_t inv_ranges;
};

constexpr int64_t INFINITY_CACHE_BYTES = (int64_t)256 << 20;
static inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
static inline int xcd_grid(int n_tiles) { return 8 * ((n_tiles + 7) / 8); }

// Full tiles fill whole rounds of the 256 compute units; the tiles of a last round are run as thin ones (four per full
// tile) if they are at most `max_thin_tail`.
static TilePlan plan_tiles(int n_tiles, int max_thin_tail) {
    TilePlan t;
    const int tail = n_tiles % 256;
    const bool thin = tail > 0 && tail <= max_thin_tail;
    t.n_full = thin ? n_tiles - tail : n_tiles;
    t.n_thin = thin ? 4 * tail : 0;
    t.thin_first = xcd_grid(t.n_full);
    return t;
}
// Logits: as many as fit one round.  A thin tile takes about half as long as a full one, so two rounds of them are no
// faster: forward, B = 256, D = 2048, 256 tiles and a tail of 32, 64, 65, 128 tiles: thin 79, 101, 120, 138 us; full, whatever
// the tail, 101-108.
static const int LOGITS_MAX_THIN_TAIL = 64;
// dW: as many as fit one round if there is no round before (fewer if they are short: they then wait for the side jobs' compute
// units), and behind full rounds, where the first of them share the chip with the last full tiles, fewer, and none if they
// are short.  A single round, us of the launch on full and thin tiles: 30 tiles (D = 256, C = 7600): 11 k-steps 21.5 and 14.7, 40: 52
// and 33; 40: 5: 13.9 and 12.5, 24: 34 and 23; 52 (D = 1024, C = 3300): 2: 10.7 and 12.5, 11: 22.3 and 20.1, 40: 51 and 39; 64
// (C = 4000): 2: 11.2 and 15.0, 11: 23.3 and 23.7, 24: 35.7 and 30.0.  Backward calls of 1 and 3 full rounds, speed of thin
// over full last rounds, tails up to 32 / 48 / 64 / 80 / 128: 48 k-steps 1.01, 0.99, 0.97, 0.97, 0.93; 64: 1.02, 1.00, 0.97, 0.97,
// 0.93; 128: 1.05, 1.03, 0.99, 0.98, 0.94; 32: 1.01, 0.98, 0.96; 16 and 24: 1.00, 0.98, 0.96 (six shapes each, D = 256, 1024, 2048).
static int dw_max_thin_tail(int n_tiles, int k_steps) { return n_tiles < 256 ? (k_steps < 12 ? 40 : 64) : k_steps < 48 ? 0 : k_steps < 96 ? 32 : 48; }
// dW in 64 x 64 tiles: as long as they are few enough for the two that a compute unit holds, and the contraction long enough to
// pay for their traffic once there is more than one.  us of the launch, 256-wide tiles (thin ones where that is
// allowed) and these: 8 of them (D = 64, C = 500): 24 k-steps 17.6 and 10.0, 125: 66 and 30; 128 (D = 256, C = 2000): 5: 8.8 and
// 8.2, 24: 21.6 and 14.8, 125: 72 and 36; 252 (D = 256, C = 4000): 11: 13.7 and 14.4, 24: 22.1 and 17.5, 125: 71 and 40; 384 (D = 1024, C =
// 1500): 5: 11.9 and 12.3, 24: 22.6 and 20.1, 125: 67.6 and 63.0; 476 (D = 256, C = 7600): 11: 14.4 and 17.9, 24: 23.5 and 23.0,
// 63: 43 and 35; 640 (D = 1024, C = 2500): 24: 22.5 and 27.2, 63: 38 and 50.
static bool dw_blocks(int D, int C, int k_steps) {
    const int64_t n = (int64_t)(D / BLOCK) * ((C + BLOCK - 1) / BLOCK);
    return n <= 192 || (n <= 512 && k_steps >= 20);
}
// dW runs as a stream where a workgroup has a second tile to overlap with the first and neighbouring tiles share a dz
// panel (more than 256 features).  Whole backward calls, one workgroup per tile and stream, us: up to 256 tiles (B = 384,
// D = 256, C = 50 000) 88.2 and 99.3; one feature tile (B = 4096, D = 256, C = 100 000) 817 and 835; more than one round of
// tiles, geometric means over 34 shapes of up to 16 k-steps 1.01 to 1.04 faster as a stream, the same beyond.
static bool dw_streams(int nDT, int n_full, int k_steps, int64_t lddw) {
    return nDT > 1 && n_full > STREAM_WGS && k_steps >= STREAM_MIN_K_STEPS && lddw < ((int64_t)1 << 22);   // 256 rows of a
}                                                                          // store tile stay within 32-bit byte offsets
// It prefetches dz if bwd_dx, which runs in between, has read more than the 256 MiB Infinity Cache holds (dz and W: B =
// 1024 and C = 12 500, 76 MB: 66.8 us without, 68.0 with; C = 100 000, 615 MB: 372 and 345), unless its tiles are so
// long that writes are rare, and where at least four workgroups share the work.  Backward calls without / with, by feature
// tiles: 8: 1.06 at 4 k-steps, 1.02 at 16, 1.006 at 24, 0.98 at 32, 0.99 at 64; 5: 1.04 at 6, 1.01 at 16, 1.005 at 24, 0.99 at 32;
// 3: 1.00 at 10 to 16; 2: 0.98 to 1.00; 1: 0.91 to 0.94.
static bool dw_prefetches(int nDT, int64_t dz_and_w_bytes, int k_steps) {
    return nDT >= 4 && k_steps <= 24 && dz_and_w_bytes > INFINITY_CACHE_BYTES;
}
// Workgroups appended to a GEMM launch for its small side job (X^T, the final reductions).
static const int SIDE_BLOCKS = 128;

// Small batches: rows that fit the registers of gemm_small.h.
struct SmallPlan {
    int rows, range, ranges;
    SmallPlan(int32_t B, int32_t C) {
        rows = B <= 16 ? 16 : 32;
        const int even = (int)round_up(round_up(C, SMALL_MAX_RANGES) / SMALL_MAX_RANGES, 8);   // whole 16-byte stores
        range = std::max(even, SMALL_C);
        ranges = (int)(round_up(C, range) / range);
    }
};
// Whether a call takes them: up to 16 rows always (forward, us, 256-wide tiles and here: C = 14 000, D = 2048: 39 and 17; arg-max, 64 x 64
// tiles and here: B = 1, D = 2048, C = 4000: 13.3 and 9.9, C = 70 000: 52.4 and 50.7).  Up to 32 where a workgroup has one turn of
// 32 classes (forward + dz, 64 x 64 tiles and here: B = 24, D = 2048, C = 4000: 12.9 + 13.2 and 12.0 + 12.1; C = 16 000: 13.9 + 14.9 and
// 17.5 + 18.3; B = 32, D = 256, C = 50 000: 11.5 + 12.2 and 12.4 + 17.3), and the arg-max again where it has four, whose 64 x 64 tiles leave four times
// as many candidates to merge (B = 24, D = 1024: C = 16 000: 10.9 and 12.0, C = 33 000: 20.3 and 18.9).
// The forward and the backward call of a shard decide alike: the backward call's logits are the forward call's.  The forward call alone would
// be quicker here from the second round of 64 x 64 tiles on up to some 1024 features, but dz loses more (B = 24, forward and backward calls, us, 64 x
// 64 tiles and here, D = 256: C = 33 000: 10.9 + 21.1 and 10.3 + 24.3, C = 100 000: 20.2 + 44.7 and 18.1 + 52.3; D = 512: 26.1 + 71.6 and 22.2 + 78.3;
// D = 2048: C = 33 000: 31.4 + 87.9 and 30.8 + 88.7, C = 100 000: 79.9 + 239.3 and 79.7 + 248.3).
enum SmallUse { SMALL_STEP, SMALL_PROBS, SMALL_TOP1 };
static bool small_batch(int32_t B, int32_t D, int32_t C, SmallUse use) {
    if (B > SMALL_MAX_ROWS || D > SMALL_MAX_STEPS * TILE_K) return false;
    return B <= 16 || C <= 32 * SMALL_MAX_RANGES || (use == SMALL_TOP1 && C > 128 * SMALL_MAX_RANGES);
}
// Small layers, and batches of up to 64 rows that are not small: the logits kernels in 64 x 64 tiles.  The wide tiles need all of a
// compute unit for 256 rows, the thin ones for 256 classes, and either a barrier's wait per k-step; two of these share one.  us of forward + dz
// on wide or thin tiles and here, by their number: 16 (B = 40, D = 1408, C = 1000) 17.4 + 18.4 and 10.6 + 10.8; 188 (B = 100, D = 2048, C =
// 6000) 22.9 + 24.4 and 13.0 + 13.6; 376 (B = 200, C = 6000) 22.5 + 24.4 and 16.9 + 16.9; 470 (B = 100, D = 256, C = 15 000) 11.2 + 11.4 and
// 7.8 + 9.0; 553 (B = 400, D = 256, C = 5000) 9.7 + 11.8 and 10.3 + 12.2; 611 (B = 800, D = 1408, C = 3000) 18.3 + 20.0 and 20.4 + 20.3.
// Probabilities and arg-max, which have neither thin tiles nor lists: 782 (B = 80, D = 2048, C = 25 000) 38.4, 40.2 and 25.9, 29.5; 939 (B =
// 150, D = 256, C = 20 000) 12.2, 13.4 and 8.9, 12.4; 1316 (B = 400, D = 1024, C = 12 000) 24.1, 25.0 and 23.6, 26.6.  Up to 64 rows, forward +
// dz: 125 (D = 4096, C = 8000) 45.2 + 46.8 and 19.8 + 20.2; 1094 (D = 1024, C = 70 000) 38.9 + 53.1 and 27.5 + 29.5; 1954 (D = 64, C = 125 000)
// 18.6 + 29.6 and 15.2 + 17.2, D = 2048: 105.7 + 107.9 and 95.3 + 107.5, but D = 3072: 141.9 + 154.6 and 147.5 + 162.7, where two full
// rounds of wide tiles read W as fast.  Arg-max of the same: D = 1024: 50.2 and 46.4, D = 256: 25.8 and 25.2, but D = 64: 16.6 and 19.8,
// four times the candidates to merge; likewise within one round of wide tiles, from the fourth block of a compute unit on: 64 rows, D =
// 64, 760 blocks 10.6 and 10.8, 820 10.6 and 11.7, 1024 10.7 and 12.1, but 1150 15.9 and 14.1; D = 192: 900 12.8 and 13.0; D = 256: 13.8 and
// 13.5; 128 rows, D = 64: 820 10.2 and 10.5, 1024 10.4 and 11.0, D = 128: 11.6 and 11.5.
static bool logits_blocks(int32_t B, int32_t D, int32_t C, SmallUse use) {
    const int64_t rows = round_up(B, BLOCK) / BLOCK, tiles = rows * (round_up(C, BLOCK) / BLOCK);
    if (use == SMALL_TOP1 && tiles > 768 && tiles <= 1024 && D < (rows == 1 ? 256 : 128)) return false;
    if (rows == 1) return tiles <= 1280 || (D <= 2048 && (use != SMALL_TOP1 || D >= 256));
    return tiles <= (use == SMALL_STEP ? 512 : 1024);
}

struct BwdPlan {
    int64_t Bpad, Cpad;
    int nBT, nCT, nDT;
    int steps_total, splits, steps_per_split;
    bool dx_small, dw_small;             // dX, dW in 64 x 64 tiles
    size_t dz_bytes, xt_bytes, dbp_bytes, parts_bytes;
    bool one_launch() const { return dx_small && dw_small && splits == 1; }      // for dX and dW (not with the fused update)
    size_t bytes() const { return dz_bytes + xt_bytes + dbp_bytes + parts_bytes; }
};

// dX: its tiles, 256 x 256 or 64 x 64, and the splits of its contraction: what takes the shortest time, in ns, of up to as many
// splits as fill the compute units once (two workgroups each of the small tiles), rounded up.
//   A wide tile takes 1.3 us per k-step and 6 for its start and its end, whatever part of it is there; a small one 0.32 for each
//   of those that share a compute unit.  The partial sums are written and read once (4.5 TB/s), and the side job takes 16 splits
//   per us and turn of its threads.
// Rounded up alone a split too many costs a second round; bwd_dx, us, rounded up / one round: B = 777, D = 1088 (20 tiles), C =
// 14 450, 13 splits (260 workgroups) 56.8, 12 splits 36.3; B = 5000, D = 1024, C = 20 000 (80 tiles), 4: 212.7, 3: 154.9.  A split for
// every k-step or two leaves the sum more to do than it saves: step, us, B = 100, D = 64, C = 30 000: 235 splits 61.2, 59 50.3.
// Without splits small tiles run in the launch of a dW of small tiles, which is worth ONE_LAUNCH_NS (step, two launches and one: B = 32,
// D = 256, C = 500 27.9 and 25.6; B = 900, D = 128, C = 700 29.9 and 26.4; B = 8000, D = 64, C = 500 55.7 and 51.3).
// Wide and small tiles, dX / step: B = 32, D = 256, C = 8000 12.4 / 30.6 and 7.0 / 27.3; B = 400, D = 128, C = 12 000 17.8 / 56.3 and
// 9.2 / 47.6; B = 1500, D = 256, C = 8000 20.2 / 75.8 and 19.3 / 67.3; B = 3000, D = 256, C = 8000 28.0 / 118.5 and 38.1 / 116.2; B = 800, D =
// 2048, C = 3000 22.6 / 93.4 and 29.8 / 94.7; B = 800, D = 256, C = 40 000 30.0 / 134.2 and 45.2 / 143.3.
// A W that the 256 MiB Infinity Cache does not hold comes from HBM, and the 128 bytes that a small tile takes of each of its rows cost more
// there: wide tiles (backward call, us, wide and small, D = 2048: B = 64, C = 62 000, 254 MB 158.1 and 152.3, C = 70 000, 287 MB 172.2 and 180.4;
// B = 24, C = 80 000: 181.7 and 192.7, with the fused update 250.7 and 277.0; D = 1536, B = 32, C = 80 000, 246 MB 136.1 and 133.1, C = 90 000, 276 MB
// 155.3 and 159.8).  Unless more than 1 / 32 of the wide tiles is padding, which cuts their reading short as well (275 to 430 MB, wide over small, backward
// call and fused update: D = 1088, a fifth tile for 64 features, 1.03 to 1.09 and 1.01 to 1.07; 1600, a seventh, 1.02 to 1.10 and 1.00 to 1.05; 1728, 192
// of a seventh, 1.00 to 1.08 and 0.99 to 1.04; 1984, 192 of an eighth, 0.97 to 1.05 and 0.93 to 1.00; whole tiles, D = 1024 to 2048, 0.93 to 1.03 and
// 0.91 to 1.02, but 1280 features, 41 and 64 rows, 275 MB 1.07).
constexpr int ONE_LAUNCH_NS = 4000;
static void dx_splits(BwdPlan& p, int32_t B, int32_t D, int32_t C) {
    const int64_t sum_turns = ((int64_t)B * (D / 4) + SIDE_BLOCKS * NTHREADS - 1) / (SIDE_BLOCKS * NTHREADS);   // of the side job's threads
    const int64_t sum_cost = 2 * ((int64_t)B * D * 4) / 4500 + sum_turns * 1000 / 16;                            // of a split
    const bool wide_only = (int64_t)C * D * 2 > INFINITY_CACHE_BYTES && 32 * (TILE_N * (int64_t)p.nDT - D) <= TILE_N * (int64_t)p.nDT;
    int64_t best = -1;
    for (int small = 0; small < (wide_only ? 1 : 2); ++small) {
        const int64_t tiles = small ? (int64_t)(D / BLOCK) * (round_up(B, BLOCK) / BLOCK) : (int64_t)p.nDT * p.nBT;
        const int room = small ? 512 : 256, most = std::min(tiles >= room ? 1 : (int)((room + tiles - 1) / tiles), p.steps_total);
        // from one number of splits to the next that makes them shorter, as long as their sum alone does not cost more
        for (int splits = 1, steps = p.steps_total; splits <= most && (splits == 1 || splits * sum_cost < best);) {
            const int64_t turns = (tiles * splits + 255) / 256;
            const int64_t cost = (small ? turns * 320 * steps + 1500 : turns * (1300 * (int64_t)steps + 6000)) + splits * sum_cost -
                                 (small && splits == 1 && p.dw_small ? ONE_LAUNCH_NS : 0);
            if (best < 0 || cost < best) {
                best = cost;
                p.steps_per_split = steps;
                p.splits = splits;
                p.dx_small = small;
            }
            // every number of splits up to the root of the k-steps makes them shorter, and every length below it is some number's
            if ((int64_t)splits * (splits + 1) <= p.steps_total) {
                ++splits;
                steps = (p.steps_total + splits - 1) / splits;
            } else if (--steps > 0) {
                splits = (p.steps_total + steps - 1) / steps;
            } else {
                break;
            }
        }
    }
}

static bool shape_ok(int32_t B, int32_t D, int32_t C) { return B > 0 && D > 0 && C > 0 && D % 64 == 0; }

// The kernels address an operand with 32-bit byte offsets, tiles may hang 256 rows over its end.
static bool fits_32bit_offsets(int64_t rows, int64_t ld) { return (rows + 256) * ld * 2 < ((int64_t)1 << 32); }

static BwdPlan plan_bwd(int32_t B, int32_t D, int32_t C) {
    BwdPlan p;
    p.Bpad = round_up(B, 256);
    p.Cpad = round_up(C, 256);
    p.nBT = (int)(p.Bpad / 256);
    p.nCT = (int)(p.Cpad / 256);
    p.nDT = (int)(round_up(D, 256) / 256);
    p.steps_total = (int)(round_up(C, TILE_K) / TILE_K);
    p.dw_small = dw_blocks(D, C, (B + TILE_K - 1) / TILE_K);
    dx_splits(p, B, D, C);
    p.dz_bytes = (size_t)p.Bpad * p.Cpad * 2;
    p.xt_bytes = (size_t)D * p.Bpad * 2;
    p.dbp_bytes = (size_t)4 * p.nBT * p.Cpad * 4;        // one db partial per 64-row wave column
    p.parts_bytes = (size_t)p.splits * B * D * 4;
    return p;
}

// The list kernels' cut: the number of ranges (and with it of workgroups per compute unit, m) that takes the shortest time, in
// cycles: a k-step of a whole tile is bound by its matrix instructions, one of a lower tile by the slots of its loads, too.
constexpr int LIST_MAX_ITEMS = 4;
static RangePlan plan_ranges(int32_t D, int32_t C, int nBT) {
    const int units = (int)(2 * (round_up(C, TILE_K) / TILE_K)), k_steps = D / TILE_K;
    RangePlan best = {1, 0, 0, 0, 0, 0, 0};
    int64_t best_cost = -1;
    for (int m = 1; m <= LIST_MAX_ITEMS; ++m) {
        const int ranges = std::min(std::max(1, LIST_WGS * m / nBT), (units + 1) / 2);
        const int per_item = (units + ranges - 1) / ranges;
        const int64_t items = ((int64_t)ranges * nBT + LIST_WGS - 1) / LIST_WGS, full = per_item / MAX_UNITS, u = per_item % MAX_UNITS;
        const int64_t cost = items * (full * (k_steps * 2700 + 10000) + (u > 0 ? k_steps * (1200 + 180 * u) + 3000 + 1000 * u : 0));
        if (best_cost >= 0 && cost >= best_cost) continue;
        best_cost = cost;
        best.ranges = ranges;
    }
    best.full = units / (MAX_UNITS * best.ranges);
    const int rest = units - best.full * MAX_UNITS * best.ranges;
    best.per = rest / best.ranges;
    best.more = rest - best.per * best.ranges;
    best.inv_block = inverse(4 * best.ranges);
    best.inv_ranges = inverse(best.ranges);
    best.inv_rest = inverse(nBT % 4);
    return best;
}
// Whether the logits of a step (more than a small batch) run as lists or as a workgroup per tile, us of forward and dz:
//   up to 64 tiles of 256 x 256 thin tiles fill more of the chip (B = 300, D = 1024, C = 800: tiles 15.1 + 16.2, lists 21.0 + 22.0);
//   a single round: lists while they halve a tile or better (81 tiles, B = 2300, D = 2048, C = 2117: 40.4 + 45.0 and 35.7 + 44.0; 94,
//     B = 300, D = 2048, C = 12 000: 39.6 + 43.1 and 35.3 + 37.9; 144, B = 777, D = 1088, C = 9001: 26.4 + 30.0 and 26.3 + 29.6; 196,
//     B = 1024, D = 2048, C = 12 500: 43.2 + 48.2 and 47.5 + 52.6);
//   more: not as several lists to a compute unit of less than a tile and a half each, which hardly run on from one tile into the next, and
//     end and start again instead (forward, tiles and lists, units of a list: B = 1408, D = 64, C = 13 471, 5: 15.8 and 19.4; B = 5409, D = 128, C =
//     2909, 4: 17.5 and 21.0; B = 1408, D = 256, C = 24 271, 6: 33.1 + 45.3 and 35.8 + 46.7; B = 14 734, D = 192, C = 3268, 8: 34.5 + 53.8 and 38.1 +
//     50.4; B = 38 406, D = 64, C = 1611, 10: 39.5 + 62.1 and 43.9 + 63.6; 12.8, B = 25 686, C = 1993: 35.8 and 36.7, 14.6, B = 18 464, C = 3220: 37.5 and 36.0);
//     of these, short contractions, whose tiles are mostly epilogue (B = 3000, D = 128, C = 20 000: 40.3 + 58.9 and 34.7 + 48.9), and longer ones if
//     the rest is half a tile or less (B = 700, D = 1024, C = 50 000: 80.5 + 93.6 and 75.1 + 85.4; B = 1024, D = 2048, C = 37 500:
//     140 + 152 and 131 + 140; B = 8192, D = 1024, C = 50 000: 691 + 794 and 662 + 744; against a rest of five units, B = 256, D = 2048,
//     C = 100 000: 120 + 121, dX 94.5 and 117 + 121, 99.0), except that long tiles over many rounds, where a workgroup that is
//     done early takes the next tile, lose nothing (B = 4096, D = 2048, C = 37 500: 460 + 507 and 469 + 509; C = 12 500: 158.9 + 174.6
//     and 159.2 + 177.4);
//   behind one or two full rounds a tail that runs as thin tiles ends sooner than the lists' rests: one round from 3 k-steps on (288 tiles, B = 2057, D =
//     832, C = 8132: 35.7 + 43.9 and 39.1 + 45.1; 264, B = 500, D = 2048: 68.1 + 74.7 and 73.1 + 79.4), two from 17 (531, B = 2057, D = 2048: 110 + 123
//     and 115 + 131; but 528, 13 k-steps, B = 700: 58.0 + 69.6 and 56.5 + 67.3), or from 9 if it is longer than 32 (560, B = 4000, D = 832:
//     58.2 + 70.6 and 63.0 + 76.0; 4 k-steps, B = 1000: 32.5 + 45.0 and 31.8 + 42.2).
static bool logits_list(const RangePlan& p, int nBT, int nCT, int k_steps) {
    const int64_t tiles = (int64_t)nBT * nCT;
    const int rest = p.per + (p.more > 0);
    if (tiles <= 64) return false;
    if (tiles <= 256) return p.full == 0 && rest <= MAX_UNITS / 2;
    if (p.ranges * nBT > LIST_WGS && MAX_UNITS * p.full + p.per < 3 * MAX_UNITS / 2) return false;
    const int64_t tail = tiles % LIST_WGS;
    if (tail > 0 && tail <= LOGITS_MAX_THIN_TAIL &&
        (tiles < 2 * LIST_WGS ? k_steps > 2 : tiles < 3 * LIST_WGS && k_steps > (tail > LOGITS_MAX_THIN_TAIL / 2 ? 8 : 16))) return false;
    return k_steps <= 8 || (rest <= MAX_UNITS / 2 && (k_steps <= 16 || tiles <= 3 * LIST_WGS));
}
static int list_grid(const RangePlan& p, int nBT) { return xcd_grid(p.ranges * nBT); }

// The kernels that compute the logits of a call, and the forward call's (the arg-max's) partial results: a pair of numbers for each
// of `parts` groups of classes and `pitch` rows.
enum LogitsWay { WAY_SMALL, WAY_BLOCKS, WAY_LISTS, WAY_TILES };
struct LogitsPlan {
    LogitsWay way;
    int64_t parts, pitch;
    RangePlan ranges;                    // of the lists
    size_t bytes() const { return (size_t)(2 * parts * pitch) * sizeof(float); }
};
// The wide tiles: what any call can do, and what it does with a workspace that its own kernels find too small.
static LogitsPlan plan_wide(int32_t B, int32_t C) {
    LogitsPlan p = {};
    p.way = WAY_TILES;
    p.parts = round_up(C, TILE_M) / TILE_M;
    p.pitch = round_up(B, TILE_N);
    return p;
}
static LogitsPlan plan_logits(int32_t B, int32_t D, int32_t C, SmallUse use) {
    LogitsPlan p = plan_wide(B, C);
    if (small_batch(B, D, C, use)) {
        const SmallPlan s(B, C);
        p.way = WAY_SMALL;
        p.parts = s.ranges;
        p.pitch = s.rows;
    } else if (logits_blocks(B, D, C, use)) {
        p.way = WAY_BLOCKS;
        p.parts = round_up(C, BLOCK) / BLOCK;
        p.pitch = round_up(B, BLOCK);
    } else if (use == SMALL_STEP) {
        const int nBT = (int)(p.pitch / TILE_N);
        p.ranges = plan_ranges(D, C, nBT);
        if (logits_list(p.ranges, nBT, (int)p.parts, D / TILE_K)) {
            p.way = WAY_LISTS;
            p.parts = p.ranges.ranges;
        }
    }
    return p;
}
// The forward call: as the step, but short contractions of a single round of wide tiles, or one with a tail of thin ones, are done
// sooner by the tiles; dz, whose epilogue is longer, is not (forward, us, tiles and lists, D = 64: 114 tiles, B = 94, C = 29 001: 11.2 and
// 12.0, dz 1.3 less; 297, B = 2303, C = 8376: 15.6 and 16.6; 312, B = 3002, C = 6596: 15.7 and 16.5; but 432, B = 4363, C = 6004: 19.3 and 18.5; two
// k-steps from some hundred tiles on: 110, B = 5631, C = 1128: 13.3 and 13.9; 126, B = 3522, C = 2073: 13.2 and 13.6; 300, B = 1410, C = 12 668: 16.9 and
// 17.7, the backward call 56.8 and 55.4; 272, B = 4084, C = 4127: 17.4 and 19.1, 56.8 and 52.4; but 87, B = 617, C = 7172: 12.5 and 12.3; 429 20.4 and
// 19.9; three k-steps: 106, B = 467, C = 13 349: 13.6 and 13.4).  Both add the products of a logit in one order.
static LogitsPlan plan_forward(int32_t B, int32_t D, int32_t C, const LogitsPlan& step) {
    const int64_t tiles = round_up(B, TILE_N) / TILE_N * (round_up(C, TILE_M) / TILE_M);
    const bool tiles_sooner = tiles <= LIST_WGS + LOGITS_MAX_THIN_TAIL && (D <= TILE_K || (D <= 2 * TILE_K && tiles > 100));
    return step.way == WAY_LISTS && tiles_sooner ? plan_wide(B, C) : step;
}

// Direction in which the logits of class tile ct and batch tile bt (256 x 256) walk the features, a function of the shard's
// step and the tile's coordinates alone, so that every kernel (and the thin and the full version of a tile) adds the products
// of a logit in the same order:
//   where the step runs in 64 x 64 tiles (or as a small batch, which has an order of its own): ascending;
//   as lists: a workgroup's whole tiles alternate, `ranges` class tiles apart, and the rest is ascending;
//   as wide tiles: a compute unit's next tile lies about 32 tile ids further on, in the next group of class tiles (up to four
//     batch tiles) or the next batch block of the same class tiles (more); alternating the direction between such groups lets it
//     find the end of the panels that the two tiles share, which it has just read, still in the L2 (launches of one round have
//     nothing to gain and keep one direction).
enum LogitsOrder { ORDER_ASCENDING, ORDER_LISTS, ORDER_FEW_BATCH_TILES, ORDER_MANY_BATCH_TILES };
static LogitsOrder logits_order(const LogitsPlan& step) {
    const int64_t nBT = step.pitch / TILE_N;
    if (step.way == WAY_LISTS) return ORDER_LISTS;
    if (step.way != WAY_TILES || nBT * step.parts <= 256) return ORDER_ASCENDING;
    return nBT <= 4 ? ORDER_FEW_BATCH_TILES : ORDER_MANY_BATCH_TILES;
}
__host__ __device__ inline bool logits_descending(LogitsOrder order, const RangePlan& ranges, int nBT, int ct, int bt) {
    if (order == ORDER_LISTS) return ct < ranges.full * ranges.ranges && (quotient((uint32_t)ct, ranges.inv_ranges) & 1) != 0;
    if (order == ORDER_FEW_BATCH_TILES) return (((ct * nBT) >> 5) & 1) != 0;
    return order == ORDER_MANY_BATCH_TILES && (((ct >> 3) ^ (bt >> 2)) & 1) != 0;
}

// The workspace that the forward call and the arg-max want, and the one that either does with.
static size_t least_fwd_bytes(int32_t B, int32_t C) { return plan_wide(B, C).bytes(); }
static size_t fwd_bytes(int32_t B, int32_t D, int32_t C) {
    return std::max({least_fwd_bytes(B, C), plan_forward(B, D, C, plan_logits(B, D, C, SMALL_STEP)).bytes(), plan_logits(B, D, C, SMALL_TOP1).bytes()});
}

}  // namespace ws
