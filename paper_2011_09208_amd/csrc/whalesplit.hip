// libwhalesplit: kernels and C-ABI entry points (see include/whalesplit.h for the contract).
//
// Kernels, in the order one training step of a shard runs them:
//   fwd_logits_stats   z^T tile = W_s . X^T on the matrix cores; per-row max / sum-exp / label
//                      logit reduced in the epilogue; one (max, sum) partial per 256-class tile
//   merge_class_tiles  merges those partials into row_max / row_sumexp of the shard
//   combine_partials   merges the shards' statistics into logsumexp and loss
//   bwd_recompute_dz   same GEMM again, epilogue dz = g (exp(z - lse) - onehot) stored as bf16
//                      [row][class]; column sums of the tile (db partials); its surplus workgroups
//                      write X^T for the dW contraction
//   predict_probs      softmax probabilities of the shard's classes, exp(z - lse), bf16
//   top1_logits        the shard's arg-max class and its logit per row (+ merge_top1, also used across shards)
//   *_small            the logits kernels for up to 32 rows (gemm_small.h; small_batch on the host)
//   *_block            the logits, dX and dW of small layers in 64 x 64 tiles (gemm_block.h; logits_blocks, dx_splits, dw_blocks)
//   bwd_dx             dX_partial = dz . W_s, split along the class contraction; partial sums
//   bwd_dw             dW_s = dz^T . X; its surplus workgroups sum the split-K partials of dX
//                      (optionally accumulating into the caller's dX) and the db partials
//   fwd_logits_list, bwd_dz_list   the same logits and dz, tiles of any height in even lists, one per compute unit
//                      (gemm_tiles.h; logits_list on the host)
// fwd_logits_stats and bwd_recompute_dz run the tiles of a ragged last round (256 compute units) as
// four thin 256 x 64 tiles each (logits_thin, fwd_stats_thin, dz_thin; plan_tiles on the host); bwd_dw
// does the same where the contraction is long (dw_thin), and takes small outputs in 64 x 64 tiles (bwd_dw_block, dw_blocks).  A plain call with several feature tiles and more than one round
// of tiles runs dW as a stream of tiles per compute unit (bwd_dw_stream, gemm_stream.h; dw_streams on the host).
// Tile orders and cache reuse: each XCD walks a contiguous range of tiles whose neighbours share operand
// panels (logits_tile_coords, bwd_dx, dw_tile); every other round of tiles walks the contraction backwards
// (logits_descending, dw_tile) and bwd_recompute_dz starts with the tiles that fwd_logits_stats ended on.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <atomic>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "../../include/whalesplit.h"
#include "gemm_block.h"
#include "gemm_core.h"
#include "gemm_small.h"
#include "gemm_stream.h"
#include "gemm_tiles.h"
#include "plan.h"

namespace ws {

constexpr float NEG_INF = -INFINITY;
constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float lane_xor(float v, int mask) { return __shfl_xor(v, mask, 64); }

// Merge of two (max, sum-exp) pairs; either may be the empty pair (-inf, 0).
__device__ __forceinline__ void merge_ms(float& m, float& s, float m2, float s2) {
    const float M = fmaxf(m, m2);
    const float f1 = (m == NEG_INF) ? 0.0f : __expf(m - M);
    const float f2 = (m2 == NEG_INF) ? 0.0f : __expf(m2 - M);
    s = s * f1 + s2 * f2;
    m = M;
}

// exp(z - m) = exp2(z * log2 e + exp_shift(m)), m the largest logit of a group (-inf: of an empty one, exp2 gives zeros).  The
// shift is rounded, which the group's sum carries as a factor of up to exp2 of half a unit in its last place: near 1 for any
// real logits, but from -2^30 on (classes masked by -1e10, -1e30, the lowest float) it would overflow, and an infinite sum times
// the weight of zero that the group has beside real logits is no number.  There the bound leaves the sum at zero.
constexpr float EXP_SHIFT_MAX = 0x1p30f * LOG2E;
__device__ __forceinline__ float exp_shift(float m) { return fminf(-m * LOG2E, EXP_SHIFT_MAX); }

// Class id (relative to the wave's first class) held in accumulator register v of M-tile mt by the
// lanes of 16-lane group g.
__device__ __forceinline__ int acc_row(int mt, int v, int g) { return 16 * mt + 4 * g + v; }

// z = acc + bias, with classes beyond the shard set to -inf.  `c_rel0` = the wave's first class
// relative to the workgroup's tile, `c_left` = number of valid classes from the wave's first class.
__device__ __forceinline__ void add_bias_and_mask(acc_t& acc, const float* sbias, bool has_bias, int c_rel0,
                                                  int c_left, int g) {
    if (has_bias) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f32x4 b4 = *reinterpret_cast<const f32x4*>(sbias + c_rel0 + 16 * mt + 4 * g);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += b4;
        }
    }
    if (c_left < WAVE_M) {   // wave-uniform: only the ragged last class tile pays for masking
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (acc_row(mt, v, g) >= c_left) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[mt][nt][v] = NEG_INF;
                }
    }
}

struct FcArgs {
    const uint16_t* X; int64_t ldx;
    const uint16_t* W; int64_t ldw;
    const float* bias;
    const int32_t* labels;
    int B, D, C, class_offset;
    int Bpad;        // B rounded up to 256
    int nBT, nCT;    // tiles along the batch and class dimensions
    LogitsOrder order;
    RangePlan ranges;
    TilePlan plan;   // which of the nBT * nCT tiles run as full tiles and which as four thin tiles each
    int last_tile_first;   // walk the full tiles from the last to the first
};

// The tile a workgroup of a logits kernel works on: full (piece < 0) or thin piece 0 .. 3 of it.
struct TileRef {
    int ct, bt, piece;
    bool valid;
};

// Tile t of a logits launch -> (class tile, batch tile).  Up to four batch tiles: batch tiles fastest, so the 32
// consecutive tiles that an XCD runs at a time share a W panel four ways and cover 32 / nBT class tiles.  More
// batch tiles: blocks of 8 class tiles x 4 batch tiles (12 operand panels for 32 tiles instead of 33), the
// batch blocks of one block of class tiles one after the other, so that consecutive rounds share its W panels.
__device__ __forceinline__ void logits_tile_coords(const FcArgs& a, int t, int& ct, int& bt) {
    if (a.nBT <= 4) {
        ct = t / a.nBT;
        bt = t % a.nBT;
        return;
    }
    const int per_block = 8 * a.nBT;
    const int cb = t / per_block, r = t - cb * per_block;
    const int rest = a.nCT - 8 * cb, h = rest < 8 ? rest : 8;     // class tiles in this block
    const int full_bb = a.nBT >> 2, in_full = h * 4 * full_bb;
    if (r < in_full) {
        const int bb = r / (h * 4), q = r - bb * (h * 4);
        ct = 8 * cb + (q >> 2);
        bt = 4 * bb + (q & 3);
    } else {
        const int w = a.nBT & 3, q = r - in_full;
        ct = 8 * cb + q / w;
        bt = 4 * full_bb + q % w;
    }
}

__device__ __forceinline__ TileRef logits_tile_ref(const FcArgs& a) {
    TileRef r;
    r.piece = -1;
    int tile;
    if ((int)blockIdx.x >= a.plan.thin_first) {
        const int q = (int)blockIdx.x - a.plan.thin_first;
        tile = q < a.plan.n_thin ? a.plan.n_full + (q >> 2) : -1;
        r.piece = q & 3;
    } else {
        tile = xcd_logical_tile(a.plan.n_full);
        if (a.last_tile_first && tile >= 0) tile = a.plan.n_full - 1 - tile;
    }
    r.valid = tile >= 0;
    r.ct = r.bt = 0;
    if (r.valid) logits_tile_coords(a, tile, r.ct, r.bt);
    return r;
}

// Runs the logits GEMM of one 256-class x 256-row tile and leaves z (bias added, padding = -inf)
// in acc.  M = classes (A = W_s, KC), N = batch rows (B operand = X, KC), K = D.
__device__ __forceinline__ void logits_tile(acc_t& acc, const FcArgs& a, int ct, int bt, char* lds,
                                            float* sbias) {
    zero_acc(acc);
    const Operand A = make_operand(a.W, a.ldw, a.C, a.D);
    const Operand Bo = make_operand(a.X, a.ldx, a.B, a.D);
    gemm_mainloop<KC>(acc, A, Bo, ct * TILE_M, bt * TILE_N, 0, a.D / TILE_K, lds, logits_descending(a.order, a.ranges, a.nBT, ct, bt));
    const int tid = threadIdx.x;
    const bool has_bias = a.bias != nullptr;
    if (has_bias) {
        if (tid < TILE_M) {
            const int c = ct * TILE_M + tid;
            sbias[tid] = c < a.C ? a.bias[c] : 0.0f;
        }
        __syncthreads();
    }
    const int wm = (tid >> 6) >> 2;
    add_bias_and_mask(acc, sbias, has_bias, wm * WAVE_M, a.C - (ct * TILE_M + wm * WAVE_M), (tid & 63) >> 4);
}

// Class id (relative to the wave's first class) of accumulator register v of M-tile mt in a thin tile
// is the same expression, with two M-tiles per wave instead of eight.
//
// z of thin tile `piece` (rows 64 * piece .. + 63 of batch tile bt), bias added, padding = -inf.
__device__ __forceinline__ void logits_thin(thin_acc_t& acc, const FcArgs& a, int ct, int bt, int piece, char* lds,
                                            float* sbias) {
#pragma unroll
    for (int i = 0; i < THIN_MT; ++i)
#pragma unroll
        for (int j = 0; j < THIN_NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const Operand A = make_operand(a.W, a.ldw, a.C, a.D);
    const Operand Bo = make_operand(a.X, a.ldx, a.B, a.D);
    thin_mainloop(acc, A, Bo, ct * TILE_M, bt * TILE_N + piece * THIN_N, 0, a.D / TILE_K, lds, logits_descending(a.order, a.ranges, a.nBT, ct, bt));
    const int tid = threadIdx.x, wave = tid >> 6, g = (tid & 63) >> 4;
    if (a.bias != nullptr) {
        if (tid < TILE_M) {
            const int c = ct * TILE_M + tid;
            sbias[tid] = c < a.C ? a.bias[c] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt) {
            const f32x4 b4 = *reinterpret_cast<const f32x4*>(sbias + wave * THIN_WAVE_M + 16 * mt + 4 * g);
#pragma unroll
            for (int nt = 0; nt < THIN_NT; ++nt) acc[mt][nt] += b4;
        }
    }
    const int c_left = a.C - (ct * TILE_M + wave * THIN_WAVE_M);
    if (c_left < THIN_WAVE_M) {
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (acc_row(mt, v, g) >= c_left) {
#pragma unroll
                    for (int nt = 0; nt < THIN_NT; ++nt) acc[mt][nt][v] = NEG_INF;
                }
    }
}

// Forward statistics of a thin tile: every wave reduces its 32 classes per row, the eight waves'
// pairs are merged through LDS in wave order.
__device__ __forceinline__ void fwd_stats_thin(const FcArgs& a, const TileRef& r, char* lds, f32x2* __restrict__ parts,
                                               float* __restrict__ label_logit) {
    float* sbias = reinterpret_cast<float*>(lds);
    float* red_m = sbias + 256;            // [8][64]
    float* red_s = red_m + 512;
    thin_acc_t acc;
    logits_thin(acc, a, r.ct, r.bt, r.piece, lds, sbias);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, jl = lane & 15;
    const int cw0 = r.ct * TILE_M + wave * THIN_WAVE_M;
    const int row0 = r.bt * TILE_N + r.piece * THIN_N;
#pragma unroll
    for (int nt = 0; nt < THIN_NT; ++nt) {
        const int row = row0 + 16 * nt + jl;
        float mx = NEG_INF;
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) mx = fmaxf(mx, acc[mt][nt][v]);
        const float shift = exp_shift(mx);
        float s = 0.0f;
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) s += __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift));
        merge_ms(mx, s, lane_xor(mx, 16), lane_xor(s, 16));
        merge_ms(mx, s, lane_xor(mx, 32), lane_xor(s, 32));
        if (g == 0) {
            red_m[wave * THIN_N + 16 * nt + jl] = mx;
            red_s[wave * THIN_N + 16 * nt + jl] = s;
        }
        const bool row_ok = row < a.B;
        const int local = row_ok ? a.labels[row] - a.class_offset : -1;
        const bool in_shard = local >= 0 && local < a.C;
        const int rel = local - cw0;
        const bool mine = in_shard && rel >= 0 && rel < THIN_WAVE_M && ((rel & 15) >> 2) == g;
        if (__any(mine)) {
            float t = 0.0f;
#pragma unroll
            for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (acc_row(mt, v, g) == rel) t = acc[mt][nt][v];
            if (mine) label_logit[row] = t;
        }
        if (r.ct == 0 && wave == 0 && g == 0 && row_ok && !in_shard) label_logit[row] = 0.0f;
    }
    __syncthreads();
    if (tid < THIN_N) {
        float m = red_m[tid], s = red_s[tid];
#pragma unroll
        for (int w = 1; w < 8; ++w) merge_ms(m, s, red_m[w * THIN_N + tid], red_s[w * THIN_N + tid]);
        parts[(int64_t)r.ct * a.Bpad + row0 + tid] = f32x2{m, s};
    }
}

// ---- logits as lists of tiles (gemm_tiles.h) ---------------------------------------------------------
// A workgroup's list: its class tiles x 256 rows, walked from the first to the last (`backwards`: from the last to the first).  Workgroups are numbered batch tiles fastest in blocks of four of them, all ranges of a block one after
// the other, so that the 32 of an XCD have up to four X panels and the fewest of W that leaves.
struct LogitsList {
    int range, n0, rounds;               // n0: first row
    int ranges, full, rest, rest_units;  // whole tiles, then rest_units units from class `rest` on
    bool backwards;
    __device__ __forceinline__ LogitsList(const FcArgs& a, bool back) : backwards(back) {
        ranges = a.ranges.ranges;
        const int it = xcd_logical_tile(ranges * a.nBT), block = (int)quotient((uint32_t)it, a.ranges.inv_block);
        const int r = it - block * 4 * ranges, left = a.nBT - 4 * block;
        range = left >= 4 ? r >> 2 : (int)quotient((uint32_t)r, a.ranges.inv_rest);
        n0 = TILE_N * (4 * block + r - range * (left >= 4 ? 4 : left));
        full = a.ranges.full;
        rest = TILE_M * full * ranges + UNIT * (range * a.ranges.per + (range < a.ranges.more ? range : a.ranges.more));
        rest_units = a.ranges.per + (range < a.ranges.more);
        rounds = it < 0 ? 0 : full + (rest_units > 0);
    }
    __device__ __forceinline__ ListTile tile(int round) const {
        const int q = backwards ? rounds - 1 - round : round;
        return ListTile{q < full ? TILE_M * (q * ranges + range) : rest, n0, q < full ? MAX_UNITS : rest_units, q < full && (q & 1) != 0};
    }
};

// LDS of a wave for what its epilogues need: the bias of its up to 128 classes, the labels of its 64 rows and one fp32 value of each.
// All of it is loaded straight into LDS: a load into registers would make the compiler wait for every load in flight.
constexpr int LIST_LABELS = 512, LIST_ROWS = 768, LIST_WAVE_BYTES = 1024;
constexpr int LIST_EXTRA_OFFSET = LDS_BYTES + 8 * LIST_WAVE_BYTES;
__device__ __forceinline__ Operand make_vector_operand(const void* base, int n) {      // of n 32-bit elements
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    return Operand{u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, 4u * (uint32_t)n, 0x00020000u}, 0u};
}

// The kernel's arguments, read afresh: what an epilogue takes from here is not held in scalar registers (there are not enough of
// them) over the main loop.
#define WS_CONSTANT const __attribute__((address_space(4)))
template <class Args>
__device__ __forceinline__ WS_CONSTANT Args* fresh_args() {
    WS_CONSTANT Args* p = (WS_CONSTANT Args*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
// The lane's number, read afresh likewise.
__device__ __forceinline__ int fresh_lane() {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

// N stores that nothing is in range of: the waits of a list's first tile count the stores of a tile before.  The empty assembly keeps
// them apart, alike as they are: the compiler made one of them, and the first waits let the tile's own loads pass for stores.
template <int N>
__device__ __forceinline__ void stores_without_effect(void* base) {
    __amdgpu_buffer_rsrc_t none = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0, 0x00020000);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        __builtin_amdgcn_raw_buffer_store_b32(0u, none, 0, 0, 0);
        asm volatile("" ::: "memory");
    }
}

// What the epilogues of the list kernels share: the wave's classes and rows, and their logits.  Positions: unit_row plus 64 in
// half 1, whatever the units of half 0.  Args begins with an FcArgs a.
template <class Args>
struct LogitsEpilogue {
    const LogitsList& list;
    char* lds;
    int c0;                  // the wave's first class (shard-local)
    __device__ __forceinline__ LogitsEpilogue(const LogitsList& l, char* lds_base) : list(l), lds(lds_base) {}
    __device__ __forceinline__ int wave() const { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
    __device__ __forceinline__ int row0() const { return list.n0 + WAVE_N * (wave() & 3); }      // the wave's first row
    __device__ __forceinline__ void begin_tile(int round) {
        const ListTile t = list.tile(round);
        const int wm = wave() >> 2, units = wave_row_units(t.units, wm);
        c0 = t.m0 + (wm == 0 ? 0 : UNIT * wave_row_units(t.units, 0));
        WS_CONSTANT Args* p = fresh_args<Args>();
        if (p->a.bias != nullptr) {                      // classes beyond the shard read as zeros
            wait_counts<NO_VM_WAIT, 0>();                // the bias of the tile before has been read
            const Operand bias = make_vector_operand(p->a.bias, p->a.C);
            const uint32_t lane4 = 4u * (uint32_t)fresh_lane();
            touch_line(bias, lane4, 4u * (uint32_t)c0, lds_offset(lds) + scratch());
            touch_line(bias, lane4, 4u * (uint32_t)(c0 + UNIT * half_units(units, 0)), lds_offset(lds) + scratch() + 256);
        }
    }
    __device__ __forceinline__ int scratch() const { return LDS_BYTES + LIST_WAVE_BYTES * wave(); }
    // Labels of the wave's rows, and from[row] if given (anything beyond the batch).
    __device__ __forceinline__ void load_rows(const float* from) {
        WS_CONSTANT Args* p = fresh_args<Args>();
        const uint32_t lane4 = 4u * (uint32_t)fresh_lane();
        touch_line(make_vector_operand(p->a.labels, p->a.B), lane4, 4u * (uint32_t)row0(), lds_offset(lds) + scratch() + LIST_LABELS);
        if (from != nullptr) touch_line(make_vector_operand(from, p->a.B), lane4, 4u * (uint32_t)row0(), lds_offset(lds) + scratch() + LIST_ROWS);
    }
    // z = acc + bias, classes beyond the shard -inf
    __device__ __forceinline__ void logits(acc_t& acc, const int (&units)[2], int g) const {
        WS_CONSTANT Args* p = fresh_args<Args>();
        wait_counts<8, NO_LG_WAIT>();                    // at least so many loads have followed those of the bias and the rows
        if (p->a.bias != nullptr) {
            const float* b = reinterpret_cast<const float*>(lds + scratch());
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if ((u & 1) < units[u >> 1]) {
#pragma unroll
                    for (int mt = 2 * u; mt < 2 * u + 2; ++mt) {
                        const f32x4 b4 = *reinterpret_cast<const f32x4*>(b + 64 * (mt >> 2) + unit_row(mt, g));
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += b4;
                    }
                }
        }
        const int C = p->a.C;
        if (c0 + UNIT * (units[0] + units[1]) > C) {     // the last tile of the last range
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (c0 + (mt >= MT / 2 ? UNIT * units[0] : 0) + unit_row(mt, g) + v >= C) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) acc[mt][nt][v] = NEG_INF;
                    }
        }
    }
    // Shard-local label of row nt of the lane, -1 if it is not in the shard or the row not in the batch.
    __device__ __forceinline__ int label(int nt, int jl, WS_CONSTANT Args* p) const {
        const int l = *reinterpret_cast<const int*>(lds + scratch() + LIST_LABELS + 4 * (16 * nt + jl)) - p->a.class_offset;
        return row0() + 16 * nt + jl < p->a.B && l >= 0 && l < p->a.C ? l : -1;
    }
    // The accumulator register 4 * mt + v of this lane that holds the logit of a row's label, -1 if none does.
    __device__ __forceinline__ int label_register(int label, const int (&units)[2], int g) const {
        int rel = label - c0;
        if (label < 0 || rel < 0 || rel >= UNIT * (units[0] + units[1]) || ((rel >> 3) & 3) != g) return -1;
        if (rel >= UNIT * units[0]) rel += 64 - UNIT * units[0];
        return 8 * (rel >> 5) + (rel & 7);               // unit_row: two M tiles to a unit of 32
    }
};

struct FwdArgs {
    FcArgs a;
    f32x2* parts;
    float* label_logit;
};

// Row statistics: a lane keeps (max, sum-exp) of its four rows over its classes of the whole list; the four lanes of a row and the
// two wave rows meet once, at its end.
struct FwdEpilogue : LogitsEpilogue<FwdArgs> {
    float mx[NT], sum[NT];
    __device__ __forceinline__ FwdEpilogue(const LogitsList& l, char* lds_base) : LogitsEpilogue(l, lds_base) {}
    __device__ __forceinline__ void begin(int round) {
        begin_tile(round);
        if (round != 0) return;
        load_rows(nullptr);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            mx[nt] = NEG_INF;
            sum[nt] = 0.0f;
        }
    }
    __device__ __forceinline__ void end(acc_t& acc, int round, const int (&units)[2]) {
        const int lane = fresh_lane(), g = lane >> 4, jl = lane & 15;
        logits(acc, units, g);
        float top[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) top[nt] = mx[nt];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((u & 1) < units[u >> 1]) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) top[nt] = fmaxf(fmaxf(top[nt], acc[2 * u][nt][v]), acc[2 * u + 1][nt][v]);
            }
        float shift[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            shift[nt] = exp_shift(top[nt]);
            sum[nt] *= mx[nt] == NEG_INF ? 0.0f : __expf(mx[nt] - top[nt]);
            mx[nt] = top[nt];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((u & 1) < units[u >> 1]) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    float s = 0.0f;
#pragma unroll
                    for (int mt = 2 * u; mt < 2 * u + 2; ++mt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) s += __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift[nt]));
                    sum[nt] += s;
                }
            }
        // Exactly one lane of the whole grid holds z[row][label - offset] when the label lies in the shard; rows whose label
        // lies outside get 0 from the first range.
        WS_CONSTANT FwdArgs* p = fresh_args<FwdArgs>();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int at = label_register(label(nt, jl, p), units, g);
            if (__any(at >= 0)) {
                float t = 0.0f;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (4 * mt + v == at) t = acc[mt][nt][v];
                if (at >= 0) p->label_logit[row0() + 16 * nt + jl] = t;
            }
        }
        if (round == list.rounds - 1) end_list(g, jl);
    }
    __device__ __forceinline__ void end_list(int g, int jl) {
        const int wm = wave() >> 2, wn = wave() & 3;
        float* red = reinterpret_cast<float*>(lds + LIST_EXTRA_OFFSET);      // [max, sum][256 rows] of wave row 1
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int row = WAVE_N * wn + 16 * nt + jl;
            merge_ms(mx[nt], sum[nt], lane_xor(mx[nt], 16), lane_xor(sum[nt], 16));
            merge_ms(mx[nt], sum[nt], lane_xor(mx[nt], 32), lane_xor(sum[nt], 32));
            if (wm == 1 && g == 0) {
                red[row] = mx[nt];
                red[256 + row] = sum[nt];
            }
        }
        wait_counts<NO_VM_WAIT, 0>();
        raw_barrier();
        WS_CONSTANT FwdArgs* p = fresh_args<FwdArgs>();
        if (wm == 0 && g == 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int row = WAVE_N * wn + 16 * nt + jl;
                merge_ms(mx[nt], sum[nt], red[row], red[256 + row]);
                p->parts[(int64_t)list.range * p->a.Bpad + list.n0 + row] = f32x2{mx[nt], sum[nt]};
                if (list.range == 0 && row0() + 16 * nt + jl < p->a.B && label(nt, jl, p) < 0) p->label_logit[row0() + 16 * nt + jl] = 0.0f;
            }
        }
    }
};

__global__ __launch_bounds__(NTHREADS) void fwd_logits_list(FwdArgs f) {
    __shared__ __attribute__((aligned(16))) char lds[LIST_EXTRA_OFFSET + 2048];
    const FcArgs& a = f.a;
    const LogitsList list(a, false);
    if (list.rounds == 0) return;
    FwdEpilogue epi(list, lds);
    gemm_tiles<KC, 0>(make_operand(a.W, a.ldw, a.C, a.D), make_operand(a.X, a.ldx, a.B, a.D), a.D / TILE_K, list, epi, lds);
}

__global__ __launch_bounds__(NTHREADS) void fwd_logits_stats(FcArgs a, f32x2* __restrict__ parts,
                                                              float* __restrict__ label_logit) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    float* sbias = reinterpret_cast<float*>(lds);          // reused after the main loop
    float* red_m = reinterpret_cast<float*>(lds) + 256;    // [2][256]
    float* red_s = red_m + 512;
    const TileRef ref = logits_tile_ref(a);
    if (!ref.valid) return;
    if (ref.piece >= 0) {
        fwd_stats_thin(a, ref, lds, parts, label_logit);
        return;
    }
    const int ct = ref.ct, bt = ref.bt;

    acc_t acc;
    logits_tile(acc, a, ct, bt, lds, sbias);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, jl = lane & 15;
    const int cw0 = ct * TILE_M + wm * WAVE_M;           // first class of this wave (shard-local)

    // A lane holds, for each of its four rows (one per N tile), 32 of the wave's 128 classes; the other
    // three 16-lane groups hold the rest.
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = bt * TILE_N + wn * WAVE_N + 16 * nt + jl;
        float mx = NEG_INF;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) mx = fmaxf(mx, acc[mt][nt][v]);
        const float shift = exp_shift(mx);
        float s = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) s += __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift));
        merge_ms(mx, s, lane_xor(mx, 16), lane_xor(s, 16));
        merge_ms(mx, s, lane_xor(mx, 32), lane_xor(s, 32));
        if (g == 0) {
            red_m[wm * 256 + wn * WAVE_N + 16 * nt + jl] = mx;
            red_s[wm * 256 + wn * WAVE_N + 16 * nt + jl] = s;
        }

        // Label logit.  Exactly one lane of the whole grid holds z[row][label - offset] when the label
        // lies in the shard; rows whose label lies outside get 0 from the first class tile.
        const bool row_ok = row < a.B;
        const int local = row_ok ? a.labels[row] - a.class_offset : -1;
        const bool in_shard = local >= 0 && local < a.C;
        const int rel = local - cw0;
        const bool mine = in_shard && rel >= 0 && rel < WAVE_M && ((rel & 15) >> 2) == g;
        if (__any(mine)) {
            float t = 0.0f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (acc_row(mt, v, g) == rel) t = acc[mt][nt][v];
            if (mine) label_logit[row] = t;
        }
        if (ct == 0 && wm == 0 && g == 0 && row_ok && !in_shard) label_logit[row] = 0.0f;
    }
    __syncthreads();
    if (tid < 256) {
        float m = red_m[tid], s = red_s[tid];
        merge_ms(m, s, red_m[256 + tid], red_s[256 + tid]);
        parts[(int64_t)ct * a.Bpad + bt * TILE_N + tid] = f32x2{m, s};
    }
}

// Loads of a merge kernel's thread in flight: a chain of them, one per 64 tiles, is what bounds these kernels.
constexpr int MERGE_BATCH = 8;

// One workgroup merges the class-tile partials, pairs (max, sum-exp), of MERGE_ROWS rows: thread (r, q) folds tiles q, q + 64, ...
// of row r, a batch of them at a time, then the 64 partial pairs of a row are merged through LDS in a fixed order
// (8 groups of 8, then the 8 group results).
// Bound by issuing exponentials where few rows have many partials, one for every 64 classes of up to 64 rows: so one for each pair and
// a batch's sum so far, and eight rows to a workgroup.  With two for each pair and 16 rows 17 to 32 rows x 125 000 classes took
// 3.9 us in here beyond the cost of a launch, with one 2.5, with one and eight rows 1.1, with four rows 1.4; 64 rows 4.0, 2.5, 1.4
// and 2.1; 256 rows on more features, whose partials are one for 256 classes, the same either way.
constexpr int MERGE_ROWS = 8;
__global__ __launch_bounds__(64 * MERGE_ROWS) void merge_class_tiles(const f32x2* __restrict__ parts, int nCT, int Bpad, int B,
                                                               float* __restrict__ row_max, float* __restrict__ row_sumexp) {
    __shared__ float sm[64][MERGE_ROWS], ss[64][MERGE_ROWS];
    const int r = threadIdx.x % MERGE_ROWS, q = threadIdx.x / MERGE_ROWS;
    const int i = blockIdx.x * MERGE_ROWS + r;        // < Bpad: the partial arrays are padded to whole tiles
    float m = NEG_INF, s = 0.0f;
    for (int t0 = q; t0 < nCT; t0 += 64 * MERGE_BATCH) {
        f32x2 v[MERGE_BATCH];
#pragma unroll
        for (int k = 0; k < MERGE_BATCH; ++k)
            v[k] = t0 + 64 * k < nCT ? parts[(int64_t)(t0 + 64 * k) * Bpad + i] : f32x2{NEG_INF, 0.0f};
        float top = m;
#pragma unroll
        for (int k = 0; k < MERGE_BATCH; ++k) top = fmaxf(top, v[k][0]);
        const float from = top == NEG_INF ? 0.0f : top;          // of empty pairs only: their exponentials are zeros
        s *= __expf(m - from);
#pragma unroll
        for (int k = 0; k < MERGE_BATCH; ++k) s += v[k][1] * __expf(v[k][0] - from);
        m = top;
    }
    sm[q][r] = m;
    ss[q][r] = s;
    __syncthreads();
    if (q < 8) {
        m = sm[8 * q][r];
        s = ss[8 * q][r];
#pragma unroll
        for (int k = 1; k < 8; ++k) merge_ms(m, s, sm[8 * q + k][r], ss[8 * q + k][r]);
    }
    __syncthreads();
    if (q < 8) {
        sm[q][r] = m;
        ss[q][r] = s;
    }
    __syncthreads();
    if (q == 0 && i < B) {
#pragma unroll
        for (int k = 1; k < 8; ++k) merge_ms(m, s, sm[k][r], ss[k][r]);
        row_max[i] = m;
        row_sumexp[i] = s;
    }
}

// Bound by the latency of its loads.  The statistics of eight shards are loaded at once; taken one after the other, with
// the largest maximum first and the sums in a second walk, 8 shards took 7.2 us at B = 1024 and 9.3 at 8192.
constexpr int COMBINE_BATCH = 8;
__device__ __forceinline__ void load_shards(float (&v)[COMBINE_BATCH], const float* __restrict__ p, int s0, int S, int64_t stride) {
#pragma unroll
    for (int k = 0; k < COMBINE_BATCH; ++k) v[k] = p[(int64_t)(s0 + k < S ? s0 + k : S - 1) * stride];
}
__device__ __forceinline__ float combine_row(const float* __restrict__ row_max, const float* __restrict__ row_sumexp,
                                             const float* __restrict__ label_logit, int S, int64_t stride, int i,
                                             float* __restrict__ logsumexp, float* __restrict__ loss_rows) {
    float vm[COMBINE_BATCH], vs[COMBINE_BATCH], vt[COMBINE_BATCH];
    load_shards(vm, row_max + i, 0, S, stride);
    load_shards(vs, row_sumexp + i, 0, S, stride);
    load_shards(vt, label_logit + i, 0, S, stride);
    float m = NEG_INF;
#pragma unroll
    for (int k = 0; k < COMBINE_BATCH; ++k) m = fmaxf(m, vm[k]);            // the last shard again beyond S
    for (int s0 = COMBINE_BATCH; s0 < S; s0 += COMBINE_BATCH) {
        float more[COMBINE_BATCH];
        load_shards(more, row_max + i, s0, S, stride);
#pragma unroll
        for (int k = 0; k < COMBINE_BATCH; ++k) m = fmaxf(m, more[k]);
    }
    float tot = 0.0f, t = 0.0f;
    for (int s0 = 0;;) {
#pragma unroll
        for (int k = 0; k < COMBINE_BATCH; ++k)
            if (s0 + k < S) {
                if (vm[k] != NEG_INF) tot += vs[k] * __expf(vm[k] - m);
                t += vt[k];
            }
        s0 += COMBINE_BATCH;
        if (s0 >= S) break;
        load_shards(vm, row_max + i, s0, S, stride);
        load_shards(vs, row_sumexp + i, s0, S, stride);
        load_shards(vt, label_logit + i, s0, S, stride);
    }
    const float lse = m + __logf(tot);
    logsumexp[i] = lse;
    loss_rows[i] = lse - t;
    return lse - t;
}
__global__ __launch_bounds__(64) void combine_partials_kernel(const float* __restrict__ row_max,
                                                              const float* __restrict__ row_sumexp,
                                                              const float* __restrict__ label_logit, int S, int B,
                                                              int64_t stride, float* __restrict__ logsumexp,
                                                              float* __restrict__ loss_rows) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B) combine_row(row_max, row_sumexp, label_logit, S, stride, i, logsumexp, loss_rows);
}

// Mean of the threads' sums of loss_rows in a fixed order (one workgroup; thread t has added rows t, t + 1024, ..).
__device__ __forceinline__ void mean_of_sums(float acc, int B, float* __restrict__ loss_mean) {
    __shared__ float red[1024];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss_mean = red[0] / (float)B;
}
__global__ __launch_bounds__(1024) void mean_loss_kernel(const float* __restrict__ loss_rows, int B,
                                                          float* __restrict__ loss_mean) {
    float acc = 0.0f;
    for (int i = threadIdx.x; i < B; i += 1024) acc += loss_rows[i];
    mean_of_sums(acc, B, loss_mean);
}
// Both in one workgroup (COMBINE_MEAN_ROWS on the host).
__global__ __launch_bounds__(1024) void combine_mean_kernel(const float* __restrict__ row_max,
                                                            const float* __restrict__ row_sumexp,
                                                            const float* __restrict__ label_logit, int S, int B,
                                                            int64_t stride, float* __restrict__ logsumexp,
                                                            float* __restrict__ loss_rows, float* __restrict__ loss_mean) {
    float acc = 0.0f;
#pragma unroll 2
    for (int i = threadIdx.x; i < B; i += 1024)
        acc += combine_row(row_max, row_sumexp, label_logit, S, stride, i, logsumexp, loss_rows);
    mean_of_sums(acc, B, loss_mean);
}

// XT[d][b] = X[b][d], zero for b >= B (the dW contraction reads whole 64-row k-steps), in 64 x 64 tiles through LDS.  Run by
// the workgroups of bwd_recompute_dz beyond its GEMM tiles: they are handed out last, onto compute units the final,
// partial round of GEMM tiles leaves idle.  Bound by the latency of its loads: a thread has 16 bytes of the next tile on their
// way while this one passes through LDS.  (The launch, us, with two bytes per lane of one tile at a time, and so: B = 4000, D =
// 2048, C = 600 76.5 and 29.1; B = 1024, D = 2048, C = 12 500 51.9 and 48.2; B = 8192, D = 1024, C = 50 000 797 and 786.)
struct XtArgs {
    uint16_t* XT; int64_t ldxt;          // [D][Bpad]
    int first_block, n_blocks;           // workgroups [first_block, first_block + n_blocks) transpose
};
constexpr int XT_PITCH = 72;             // elements of a row of the transposed tile in LDS

// `lds`: two tiles of 64 x XT_PITCH.  Workgroups of NTHREADS, a 16-byte chunk of the tile each.
__device__ __forceinline__ void transpose_x_tiles(const FcArgs& a, const XtArgs& x, int worker, char* lds) {
    const int nb = (a.B + 63) / 64, n_tiles = nb * (a.D / 64);
    const int row = threadIdx.x >> 3, chunk = threadIdx.x & 7;
    u32x4 v;
    auto load = [&](int t) {
        const int b = (t % nb) * 64 + row, d0 = (t / nb) * 64;
        v = u32x4{0, 0, 0, 0};
        if (t < n_tiles && b < a.B) v = *reinterpret_cast<const u32x4*>(a.X + (int64_t)b * a.ldx + d0 + 8 * chunk);
    };
    load(worker);
    int buffer = 0;
    for (int t = worker; t < n_tiles; t += x.n_blocks) {
        const int b0 = (t % nb) * 64, d0 = (t / nb) * 64;
        uint16_t* tile = reinterpret_cast<uint16_t*>(lds) + buffer * (64 * XT_PITCH);
        buffer ^= 1;                                     // read two tiles ago, a barrier ago
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[(8 * chunk + e) * XT_PITCH + row] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        load(t + x.n_blocks);
        wait_counts<NO_VM_WAIT, 0>();
        raw_barrier();
        *reinterpret_cast<u32x4*>(x.XT + (int64_t)(d0 + row) * x.ldxt + b0 + 8 * chunk) =
            *reinterpret_cast<const u32x4*>(tile + row * XT_PITCH + 8 * chunk);
    }
}

// dz of a thin tile: the same steps as in bwd_recompute_dz below on a 256-class x 64-row tile.  Its
// column sums are one db partial, in the slot the matching wave column of a full tile would fill.
__device__ __forceinline__ void dz_thin(const FcArgs& a, const TileRef& r, char* lds,
                                        const float* __restrict__ logsumexp, float grad_scale,
                                        uint16_t* __restrict__ dZ, int64_t ldz, float* __restrict__ db_part) {
    float* sbias = reinterpret_cast<float*>(lds);
    thin_acc_t acc;
    logits_thin(acc, a, r.ct, r.bt, r.piece, lds, sbias);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, jl = lane & 15;
    const int cw0 = r.ct * TILE_M + wave * THIN_WAVE_M;
    const int row0 = r.bt * TILE_N + r.piece * THIN_N;
#pragma unroll
    for (int nt = 0; nt < THIN_NT; ++nt) {
        const int row = row0 + 16 * nt + jl;
        const bool row_ok = row < a.B;
        const float lse = row_ok ? logsumexp[row] : 0.0f;
        const float gs = row_ok ? grad_scale : 0.0f;
        const float shift = __log2f(fabsf(gs)) - lse * LOG2E;
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[mt][nt][v] = __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift));
        if (grad_scale < 0.0f) {
#pragma unroll
            for (int mt = 0; mt < THIN_MT; ++mt) acc[mt][nt] = -acc[mt][nt];
        }
        const int local = row_ok ? a.labels[row] - a.class_offset : -1;
        const bool in_shard = local >= 0 && local < a.C;
        const int rel = local - cw0;
        const bool mine = in_shard && rel >= 0 && rel < THIN_WAVE_M && ((rel & 15) >> 2) == g;
        if (__any(mine)) {
#pragma unroll
            for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (mine && acc_row(mt, v, g) == rel) acc[mt][nt][v] -= gs;
        }
    }
    if (db_part != nullptr) {
        // a lane adds its four N-tiles; the 16 lanes with the same classes reduce-scatter the 8 sums in
        // three exchange steps and add the last pair, so lanes 2 i and 2 i + 1 both hold sum i
        float val[4 * THIN_MT];
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                val[4 * mt + v] = (acc[mt][0][v] + acc[mt][1][v]) + (acc[mt][2][v] + acc[mt][3][v]);
#pragma unroll
        for (int step = 0; step < 3; ++step) {
            const int h = (2 * THIN_MT) >> step, mask = 8 >> step;
            const bool up = (jl & mask) != 0;
#pragma unroll
            for (int i = 0; i < h; ++i) {
                const float keep = up ? val[i + h] : val[i];
                const float send = up ? val[i] : val[i + h];
                val[i] = keep + lane_xor(send, mask);
            }
        }
        val[0] += lane_xor(val[0], 1);
        if ((jl & 1) == 0) {
            const int i = jl >> 1;                      // accumulator row index 4 * mt + v
            db_part[(int64_t)(4 * r.bt + r.piece) * ldz + cw0 + 16 * (i >> 2) + 4 * g + (i & 3)] = val[0];
        }
    }
    __syncthreads();                       // the bias staging area is about to be overwritten
#pragma unroll
    for (int nt = 0; nt < THIN_NT; ++nt) {
        const int n = 16 * nt + jl;
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt) {
            u32x2 pk;
            pk[0] = pack_bf16(acc[mt][nt][0], acc[mt][nt][1]);
            pk[1] = pack_bf16(acc[mt][nt][2], acc[mt][nt][3]);
            *reinterpret_cast<u32x2*>(lds + out_tile_offset(n, wave * THIN_WAVE_M + 16 * mt + 4 * g)) = pk;
        }
    }
    __syncthreads();
    lds_tile_store_rows(lds, dZ + (int64_t)row0 * ldz + r.ct * TILE_M, ldz, THIN_N, TILE_M);
}

__global__ __launch_bounds__(NTHREADS) void bwd_recompute_dz(FcArgs a, const float* __restrict__ logsumexp,
                                                              float grad_scale, uint16_t* __restrict__ dZ,
                                                              int64_t ldz, float* __restrict__ db_part,
                                                              XtArgs xt) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    float* sbias = reinterpret_cast<float*>(lds);
    if ((int)blockIdx.x >= xt.first_block) {
        transpose_x_tiles(a, xt, (int)blockIdx.x - xt.first_block, lds);
        return;
    }
    const TileRef ref = logits_tile_ref(a);
    if (!ref.valid) return;
    if (ref.piece >= 0) {
        dz_thin(a, ref, lds, logsumexp, grad_scale, dZ, ldz, db_part);
        return;
    }
    const int ct = ref.ct, bt = ref.bt;

    acc_t acc;
    logits_tile(acc, a, ct, bt, lds, sbias);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, jl = lane & 15;
    const int cw0 = ct * TILE_M + wm * WAVE_M;

#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = bt * TILE_N + wn * WAVE_N + 16 * nt + jl;     // < Bpad: dZ has that many rows
        const bool row_ok = row < a.B;
        const float lse = row_ok ? logsumexp[row] : 0.0f;
        const float gs = row_ok ? grad_scale : 0.0f;                   // padded rows store exact zeros
        // |g| * exp(z - lse) = exp2(z * log2 e + (log2 |g| - lse * log2 e)): one FMA and one exp2 per
        // element; g = 0 gives a shift of -inf and exact zeros, as does z = -inf on padded classes.
        const float shift = __log2f(fabsf(gs)) - lse * LOG2E;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[mt][nt][v] = __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift));
        if (grad_scale < 0.0f) {                                        // uniform; the usual scales are positive
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = -acc[mt][nt];
        }

        const int local = row_ok ? a.labels[row] - a.class_offset : -1;
        const bool in_shard = local >= 0 && local < a.C;
        const int rel = local - cw0;
        const bool mine = in_shard && rel >= 0 && rel < WAVE_M && ((rel & 15) >> 2) == g;
        if (__any(mine)) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (mine && acc_row(mt, v, g) == rel) acc[mt][nt][v] -= gs;
        }
    }

    // db: the tile's column sums over its batch rows, taken from the fp32 values.  A lane first adds
    // its four N-tiles, then the 16 lanes that hold the same classes reduce-scatter their 32 sums in
    // four exchange steps (16, 8, 4, 2 values sent), which leaves lane jl the sums of accumulator
    // rows 2 jl and 2 jl + 1 (row index = 4 * M-tile + register).  One partial per wave column:
    // db_part[4 * bt + wn][class].
    if (db_part != nullptr) {
        float val[4 * MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                val[4 * mt + v] = (acc[mt][0][v] + acc[mt][1][v]) + (acc[mt][2][v] + acc[mt][3][v]);
#pragma unroll
        for (int step = 0; step < 4; ++step) {
            const int h = (2 * MT) >> step, mask = 8 >> step;
            const bool up = (jl & mask) != 0;
#pragma unroll
            for (int i = 0; i < h; ++i) {
                const float keep = up ? val[i + h] : val[i];
                const float send = up ? val[i] : val[i + h];
                val[i] = keep + lane_xor(send, mask);
            }
        }
        const int cls = cw0 + 16 * (jl >> 1) + 4 * g + 2 * (jl & 1);
        f32x2 two = {val[0], val[1]};
        *reinterpret_cast<f32x2*>(db_part + (int64_t)(4 * bt + wn) * ldz + cls) = two;
    }

    // dz [row][class] feeds both the dX contraction (over classes, read along its rows) and the dW
    // contraction (over rows, read across them).  The tile is staged in LDS so that it leaves in
    // whole 512-byte rows.
    __syncthreads();                       // the bias staging area is about to be overwritten
    acc_to_lds_bf16<KC>(acc, lds);
    __syncthreads();
    lds_tile_store_rows(lds, dZ + (int64_t)bt * TILE_N * ldz + ct * TILE_M, ldz, TILE_N, TILE_M);
}

// One step of a reduce-scatter over lanes MASK apart: 2 H sums become H.
template <int H, int MASK, int N>
__device__ __forceinline__ void exchange_half(float (&val)[N], int jl) {
    const bool up = (jl & MASK) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const float keep = up ? val[i + H] : val[i];
        const float send = up ? val[i] : val[i + H];
        val[i] = keep + lane_xor(send, MASK);
    }
}

// dz of the list kernels.  A wave's 64 rows x 64 classes of a half leave through its own 2 KiB of LDS, 16 rows at a time, so that
// eight consecutive lanes store one whole 128-byte line (16-byte chunks are XOR-ed with row & 7); nobody waits for the
// stores.  16 of them per tile and wave, whatever its units: those without classes have no records.
struct DzArgs {
    FcArgs a;
    const float* logsumexp;
    float grad_scale;
    uint16_t* dZ; int64_t ldz;
    float* db_part;
    XtArgs xt;
};
struct DzEpilogue : LogitsEpilogue<DzArgs> {
    static constexpr int SCRATCH_BYTES = 2048;
    static constexpr int STORES = 16;
    __device__ __forceinline__ DzEpilogue(const LogitsList& l, char* lds_base) : LogitsEpilogue(l, lds_base) {}
    __device__ __forceinline__ void begin(int round) {
        begin_tile(round);
        if (round != 0) return;
        load_rows(fresh_args<DzArgs>()->logsumexp);
        stores_without_effect<STORES>(fresh_args<DzArgs>()->dZ);
    }
    __device__ __forceinline__ void end(acc_t& acc, int, const int (&units)[2]) {
        const int lane = fresh_lane(), g = lane >> 4, jl = lane & 15;
        logits(acc, units, g);
        WS_CONSTANT DzArgs* p = fresh_args<DzArgs>();
        const float grad_scale = p->grad_scale;
        float shift[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            // |g| * exp(z - lse) = exp2(z * log2 e + (log2 |g| - lse * log2 e)): one FMA and one exp2 per element; g = 0 (rows
            // beyond the batch) gives a shift of -inf and exact zeros, as does z = -inf on padded classes.
            const bool row_ok = row0() + 16 * nt + jl < p->a.B;
            const float lse = *reinterpret_cast<const float*>(lds + scratch() + LIST_ROWS + 4 * (16 * nt + jl));
            shift[nt] = __log2f(row_ok ? fabsf(grad_scale) : 0.0f) - (row_ok ? lse : 0.0f) * LOG2E;
        }
        const bool negative = grad_scale < 0.0f;                            // uniform; the usual scales are positive
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((u & 1) < units[u >> 1]) {
#pragma unroll
                for (int mt = 2 * u; mt < 2 * u + 2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[mt][nt][v] = __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift[nt]));
                        if (negative) acc[mt][nt] = -acc[mt][nt];
                    }
            }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int at = label_register(label(nt, jl, p), units, g);
            if (__any(at >= 0)) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[mt][nt][v] -= 4 * mt + v == at ? grad_scale : 0.0f;      // (as a branch the compiler makes 12 of it)
            }
        }
        // db: the tile's column sums over its batch rows, taken from the fp32 values.  A lane first adds its four N-tiles, then
        // the 16 lanes that hold the same classes reduce-scatter their 32 sums in four exchange steps (16, 8, 4, 2 values
        // sent), which leaves lane jl the sums of accumulator rows 2 jl and 2 jl + 1 (row index = 4 * M-tile + register).
        // One partial per wave column: db_part[row / 64][class].
        p = fresh_args<DzArgs>();
        if (p->db_part != nullptr) {
            float val[4 * MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    val[4 * mt + v] = ((mt >> 1) & 1) < units[mt >> 2] ? (acc[mt][0][v] + acc[mt][1][v]) + (acc[mt][2][v] + acc[mt][3][v]) : 0.0f;
            exchange_half<2 * MT, 8>(val, jl);
            exchange_half<MT, 4>(val, jl);
            exchange_half<MT / 2, 2>(val, jl);
            exchange_half<MT / 4, 1>(val, jl);
            const int mt = jl >> 1;
            if (((mt >> 1) & 1) < (mt >= MT / 2 ? units[1] : units[0])) {
                const int cls = c0 + (mt >= MT / 2 ? UNIT * units[0] : 0) + unit_row(mt, g) + 2 * (jl & 1);
                f32x2 two = {val[0], val[1]};
                *reinterpret_cast<f32x2*>(p->db_part + (int64_t)(row0() >> 6) * p->ldz + cls) = two;
            }
        }
        p = fresh_args<DzArgs>();
        uint16_t* dZ = p->dZ;
        const uint32_t ldz = (uint32_t)p->ldz;
        const int n = lane >> 3, chunk = lane & 7, scratch = LIST_EXTRA_OFFSET + SCRATCH_BYTES * wave();
        const int wr = scratch + jl * 128 + ((g ^ (jl & 7)) << 4), rd = scratch + n * 128 + ((chunk ^ n) << 4);
        const uint32_t records = (uint32_t)p->a.Bpad * ldz * 2u, lane_off = ((uint32_t)n * ldz + 8u * (uint32_t)chunk) * 2u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t col = (uint32_t)(c0 + (h == 0 ? 0 : UNIT * units[0])) * 2u;
            __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(dZ, 0, units[h] > 0 ? (int)records : 0, 0x00020000);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f32x4 lo = acc[4 * h + 2 * u][nt], hi = acc[4 * h + 2 * u + 1][nt];
                    *reinterpret_cast<u32x4*>(lds + (wr ^ (64 * u))) =
                        u32x4{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(lds + rd + 1024 * k);
                    const uint32_t soff = (uint32_t)(row0() + 16 * nt + 8 * k) * ldz * 2u + col;
                    if (units[h] != 1 || chunk < 4) __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_off, (int)soff, 2);   // non-temporal
                }
            }
        }
    }
};

__global__ __launch_bounds__(NTHREADS) void bwd_dz_list(DzArgs z) {
    __shared__ __attribute__((aligned(16))) char lds[LIST_EXTRA_OFFSET + 8 * DzEpilogue::SCRATCH_BYTES];
    const FcArgs& a = z.a;
    if ((int)blockIdx.x >= z.xt.first_block) {
        transpose_x_tiles(a, z.xt, (int)blockIdx.x - z.xt.first_block, lds);
        return;
    }
    const LogitsList list(a, true);
    if (list.rounds == 0) return;
    DzEpilogue epi(list, lds);
    gemm_tiles<KC, DzEpilogue::STORES>(make_operand(a.W, a.ldw, a.C, a.D), make_operand(a.X, a.ldx, a.B, a.D), a.D / TILE_K, list, epi, lds);
}

// Predictions of the shard: P[i][c] = exp(z[i][c] - lse[i]) as bf16, the same GEMM and staging as
// bwd_recompute_dz without the one-hot term, written straight into the caller's [B][ldp] matrix
// (ragged edges cut at B and C).
__global__ __launch_bounds__(NTHREADS) void predict_probs(FcArgs a, const float* __restrict__ logsumexp,
                                                           uint16_t* __restrict__ P, int64_t ldp) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    float* sbias = reinterpret_cast<float*>(lds);
    const int tile = xcd_logical_tile(a.nBT * a.nCT);
    if (tile < 0) return;
    const int ct = tile / a.nBT, bt = tile % a.nBT;

    acc_t acc;
    logits_tile(acc, a, ct, bt, lds, sbias);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wn = wave & 3, jl = lane & 15;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = bt * TILE_N + wn * WAVE_N + 16 * nt + jl;
        const float shift = row < a.B ? -logsumexp[row] * LOG2E : 0.0f;      // rows beyond B are not stored
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[mt][nt][v] = __builtin_amdgcn_exp2f(fmaf(acc[mt][nt][v], LOG2E, shift));
    }
    __syncthreads();                       // the bias staging area is about to be overwritten
    acc_to_lds_bf16<KC>(acc, lds);
    __syncthreads();
    const int b_left = a.B - bt * TILE_N, c_left = a.C - ct * TILE_M;
    lds_tile_store_rows(lds, P + (int64_t)bt * TILE_N * ldp + ct * TILE_M, ldp, b_left < TILE_N ? b_left : TILE_N,
                        c_left < TILE_M ? c_left : TILE_M);
}

// ---- arg-max predictions --------------------------------------------------------------------------
// The better of two (logit, class) candidates: the larger logit, the lower class id among equals.
__device__ __forceinline__ void better_of(float& v, int& c, float v2, int c2) {
    if (v2 > v || (v2 == v && c2 < c)) {
        v = v2;
        c = c2;
    }
}

// Top-1 of every row over one 256-class tile: the logits GEMM of fwd_logits_stats with an arg-max
// epilogue.  Partial (logit, shard-local class) pairs go to part_val / part_cls [class tile][row].
__global__ __launch_bounds__(NTHREADS) void top1_logits(FcArgs a, float* __restrict__ part_val,
                                                         int* __restrict__ part_cls) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    float* sbias = reinterpret_cast<float*>(lds);
    float* red_v = sbias + 256;                              // [2][256]
    int* red_c = reinterpret_cast<int*>(red_v + 512);
    const int tile = xcd_logical_tile(a.nBT * a.nCT);
    if (tile < 0) return;
    const int ct = tile / a.nBT, bt = tile % a.nBT;
    acc_t acc;
    logits_tile(acc, a, ct, bt, lds, sbias);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, jl = lane & 15;
    const int cw0 = ct * TILE_M + wm * WAVE_M;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float best = NEG_INF;
        int cls = INT_MAX;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (acc[mt][nt][v] > best) {                 // classes are visited in increasing order
                    best = acc[mt][nt][v];
                    cls = cw0 + acc_row(mt, v, g);
                }
        better_of(best, cls, lane_xor(best, 16), __shfl_xor(cls, 16, 64));
        better_of(best, cls, lane_xor(best, 32), __shfl_xor(cls, 32, 64));
        if (g == 0) {
            red_v[wm * 256 + wn * WAVE_N + 16 * nt + jl] = best;
            red_c[wm * 256 + wn * WAVE_N + 16 * nt + jl] = cls;
        }
    }
    __syncthreads();
    if (tid < 256) {
        float v = red_v[tid];
        int c = red_c[tid];
        better_of(v, c, red_v[256 + tid], red_c[256 + tid]);
        const int64_t o = (int64_t)ct * a.Bpad + bt * TILE_N + tid;
        part_val[o] = v;
        part_cls[o] = c;
    }
}

// Merges n candidates per row, `stride` apart; `base` is added to the winning class.  One workgroup takes 16 rows:
// thread (r, q) folds candidates q, q + 64, ... of row r, then the 64 winners of a row are merged through LDS (the better
// of two is an order, so the grouping does not matter).  With one thread per row the loads of a row followed each
// other: 391 candidates took 129 us, now 5 us.
__global__ __launch_bounds__(1024) void merge_top1(const float* __restrict__ val, const int* __restrict__ cls, int n,
                                                   int64_t stride, int B, int base, float* __restrict__ out_val,
                                                   int* __restrict__ out_cls) {
    __shared__ float sv[64][16];
    __shared__ int sc[64][16];
    const int r = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int i = blockIdx.x * 16 + r;
    float v = NEG_INF;
    int c = INT_MAX;
    if (i < B)
        for (int t0 = q; t0 < n; t0 += 64 * MERGE_BATCH) {
            float tv[MERGE_BATCH];
            int tc[MERGE_BATCH];
#pragma unroll
            for (int k = 0; k < MERGE_BATCH; ++k)
                if (t0 + 64 * k < n) {
                    tv[k] = val[(t0 + 64 * k) * stride + i];
                    tc[k] = cls[(t0 + 64 * k) * stride + i];
                }
#pragma unroll
            for (int k = 0; k < MERGE_BATCH; ++k)
                if (t0 + 64 * k < n) better_of(v, c, tv[k], tc[k]);
        }
    sv[q][r] = v;
    sc[q][r] = c;
    __syncthreads();
    for (int w = 32; w > 0; w >>= 1) {
        if (q < w) {
            better_of(v, c, sv[q + w][r], sc[q + w][r]);
            sv[q][r] = v;
            sc[q][r] = c;
        }
        __syncthreads();
    }
    if (q == 0 && i < B) {
        out_val[i] = v;
        out_cls[i] = c == INT_MAX ? c : c + base;
    }
}

// The same for a few candidates, one thread per row with its loads side by side: the tree of the kernel above costs more
// than it saves.  B = 1024, us, here and above: 1 candidate 1.9 and 2.8, 8: 2.2 and 2.7, 12: 2.7 and 2.8, 16: 2.9 and 2.8, 64: 7.4
// and 3.2 (B = 8192: 12: 2.8 and 3.3, 64: 7.4 and 4.1).
constexpr int MERGE_FEW = 12;
__global__ __launch_bounds__(64) void merge_top1_few(const float* __restrict__ val, const int* __restrict__ cls, int n,
                                                     int64_t stride, int B, int base, float* __restrict__ out_val,
                                                     int* __restrict__ out_cls) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= B) return;
    float v = NEG_INF;
    int c = INT_MAX;
    for (int t0 = 0; t0 < n; t0 += MERGE_BATCH) {
        float tv[MERGE_BATCH];
        int tc[MERGE_BATCH];
#pragma unroll
        for (int k = 0; k < MERGE_BATCH; ++k)
            if (t0 + k < n) {
                tv[k] = val[(t0 + k) * stride + i];
                tc[k] = cls[(t0 + k) * stride + i];
            }
#pragma unroll
        for (int k = 0; k < MERGE_BATCH; ++k)
            if (t0 + k < n) better_of(v, c, tv[k], tc[k]);
    }
    out_val[i] = v;
    out_cls[i] = c == INT_MAX ? c : c + base;
}

// ---- small batches --------------------------------------------------------------------------------
// The logits kernels for up to 32 rows (gemm_small.h): workgroup w takes the classes [w * range, (w + 1) * range) and
// reports one partial result per row.
// Bound by reading W.  W of 100 000 x 2048, B = 1, arg-max: 87 us on the wide tiles, 71 here (5.8 TB/s); W of 12 500 x 2048,
// B = 32: statistics 31.5 and 14.8 us, probabilities 37.4 and 15.2 (224 of 256 units have work, turns of 32 and 24 classes).
template <int NB, class Body>
__device__ __forceinline__ void small_range(const FcArgs& a, int range, int wg, int classes, float* lds, Body body) {
    const int c_begin = wg * range, c_end = c_begin + range < classes ? c_begin + range : classes;
    small_logits<NB>(a.X, a.ldx, a.B, a.W, a.ldw, a.C, a.D, a.bias, c_begin, c_end, lds, [&](int c, float (&z)[SmallShape<NB>::CPT]) {
#pragma unroll
        for (int e = 0; e < SmallShape<NB>::CPT; ++e)
            if (c + e >= c_end) z[e] = NEG_INF;                        // the next workgroup's
        body(c, c_end - c, z);
    });
}

template <int NB>
__global__ __launch_bounds__(SMALL_THREADS) void fwd_stats_small(FcArgs a, int range, f32x2* __restrict__ parts,
                                                                           float* __restrict__ label_logit) {
    typedef SmallShape<NB> S;
    __shared__ __attribute__((aligned(16))) float lds[S::LDS_FLOATS];
    const int row = (int)threadIdx.x / S::TPR, j = (int)threadIdx.x % S::TPR;
    const bool row_ok = row < a.B;
    int local = row_ok ? a.labels[row] - a.class_offset : -1;
    const bool in_shard = local >= 0 && local < a.C;
    if (!in_shard) local = -1;
    float mx = NEG_INF, sum = 0.0f, label = 0.0f;
    bool found = false;
    small_range<NB>(a, range, blockIdx.x, a.C, lds, [&](int c, int left, const float (&z)[S::CPT]) {
        float m = NEG_INF, s = 0.0f;
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) m = fmaxf(m, z[e]);
        const float shift = exp_shift(m);
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) s += __builtin_amdgcn_exp2f(fmaf(z[e], LOG2E, shift));
        merge_ms(mx, sum, m, s);
#pragma unroll
        for (int e = 0; e < S::CPT; ++e)
            if (local == c + e && e < left) {
                label = z[e];
                found = true;
            }
    });
#pragma unroll
    for (int w = S::TPR / 2; w > 0; w >>= 1) merge_ms(mx, sum, lane_xor(mx, w), lane_xor(sum, w));
    if (j == 0) parts[(int)blockIdx.x * S::ROWS + row] = f32x2{mx, sum};
    if (found || (blockIdx.x == 0 && j == 0 && row_ok && !in_shard)) label_logit[row] = label;
}

// The N classes of a thread as bf16, in one store where the matrix is that wide (`left` classes are).
template <int N>
__device__ __forceinline__ void small_store(uint16_t* out, const float (&v)[N], int left) {
    if constexpr (N > 1) {
        uint32_t pk[N / 2];
#pragma unroll
        for (int e = 0; e < N / 2; ++e) pk[e] = pack_bf16(v[2 * e], v[2 * e + 1]);
        if (left >= N) {
            static_assert(N == 2, "");
            *reinterpret_cast<uint32_t*>(out) = pk[0];
            return;
        }
    }
#pragma unroll
    for (int e = 0; e < N; ++e)
        if (e < left) out[e] = (uint16_t)pack_bf16(v[e], 0.0f);
}

// dz of the batch's rows (the contractions that read it bound their operand at the batch), up to whole k-steps of
// classes (zeros beyond the shard: bwd_dx reads those); one db partial.
template <int NB>
__global__ __launch_bounds__(SMALL_THREADS) void dz_small(FcArgs a, int range, const float* __restrict__ logsumexp,
                                                                    float grad_scale, uint16_t* __restrict__ dZ, int64_t ldz,
                                                                    float* __restrict__ db_part, XtArgs xt) {
    typedef SmallShape<NB> S;
    __shared__ __attribute__((aligned(16))) float lds[S::LDS_FLOATS + S::SLOT_FLOATS];
    if ((int)blockIdx.x >= xt.first_block) {
        transpose_x_tiles(a, xt, (int)blockIdx.x - xt.first_block, reinterpret_cast<char*>(lds));
        return;
    }
    const int row = (int)threadIdx.x / S::TPR, j = (int)threadIdx.x % S::TPR;
    const bool row_ok = row < a.B;
    const float gs = row_ok ? grad_scale : 0.0f;
    const float shift = __log2f(fabsf(gs)) - (row_ok ? logsumexp[row] : 0.0f) * LOG2E;
    const int local = row_ok ? a.labels[row] - a.class_offset : -1;
    const int classes = (a.C + TILE_K - 1) / TILE_K * TILE_K;
    float* tile_f32 = lds + S::LDS_FLOATS;
    small_range<NB>(a, range, blockIdx.x, classes, lds, [&](int c, int left, float (&z)[S::CPT]) {
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) {
            z[e] = __builtin_amdgcn_exp2f(fmaf(z[e], LOG2E, shift));
            if (grad_scale < 0.0f) z[e] = -z[e];
            if (local == c + e && c + e < a.C) z[e] -= gs;
        }
        if (row_ok) small_store<S::CPT>(dZ + (int64_t)row * ldz + c, z, left);
        if (db_part != nullptr) {
#pragma unroll
            for (int e = 0; e < S::CPT; ++e) tile_f32[row * SMALL_PITCH + S::CPT * j + e] = z[e];
            wait_counts<NO_VM_WAIT, 0>();
            raw_barrier();                             // and the barrier of the next 32 classes comes before the next write
            const int first = c - S::CPT * j;          // of the 32
            if ((int)threadIdx.x < SMALL_C && (int)threadIdx.x < left + S::CPT * j) {
                float s = 0.0f;
#pragma unroll 8
                for (int r = 0; r < S::ROWS; ++r) s += tile_f32[r * SMALL_PITCH + threadIdx.x];
                db_part[first + (int)threadIdx.x] = s;
            }
        }
    });
}

template <int NB>
__global__ __launch_bounds__(SMALL_THREADS) void predict_small(FcArgs a, int range, const float* __restrict__ logsumexp,
                                                                         uint16_t* __restrict__ P, int64_t ldp) {
    typedef SmallShape<NB> S;
    __shared__ __attribute__((aligned(16))) float lds[S::LDS_FLOATS];
    const int row = (int)threadIdx.x / S::TPR;
    const bool row_ok = row < a.B;
    const float shift = row_ok ? -logsumexp[row] * LOG2E : 0.0f;
    small_range<NB>(a, range, blockIdx.x, a.C, lds, [&](int c, int left, float (&z)[S::CPT]) {
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) z[e] = __builtin_amdgcn_exp2f(fmaf(z[e], LOG2E, shift));
        if (row_ok) small_store<S::CPT>(P + (int64_t)row * ldp + c, z, left);
    });
}

template <int NB>
__global__ __launch_bounds__(SMALL_THREADS) void top1_small(FcArgs a, int range, float* __restrict__ part_val,
                                                                      int* __restrict__ part_cls) {
    typedef SmallShape<NB> S;
    __shared__ __attribute__((aligned(16))) float lds[S::LDS_FLOATS];
    const int row = (int)threadIdx.x / S::TPR, j = (int)threadIdx.x % S::TPR;
    float best = NEG_INF;
    int cls = INT_MAX;
    small_range<NB>(a, range, blockIdx.x, a.C, lds, [&](int c, int, const float (&z)[S::CPT]) {
#pragma unroll
        for (int e = 0; e < S::CPT; ++e)
            if (z[e] > best) {                                   // a thread's classes come in increasing order
                best = z[e];
                cls = c + e;
            }
    });
#pragma unroll
    for (int w = S::TPR / 2; w > 0; w >>= 1) better_of(best, cls, lane_xor(best, w), __shfl_xor(cls, w, 64));
    if (j == 0) {
        part_val[(int)blockIdx.x * S::ROWS + row] = best;
        part_cls[(int)blockIdx.x * S::ROWS + row] = cls;
    }
}

// ---- small layers ---------------------------------------------------------------------------------
// The logits kernels in tiles of 64 classes x 64 rows (gemm_block.h).  Workgroups are numbered row blocks fastest.
struct LogitsBlock {
    int cb, rb, c0, row;                 // class and row block; the lane's first class (4 * g of M tile 0), its row
    int wave, g, i;
    __device__ __forceinline__ explicit LogitsBlock(const FcArgs& a) {
        const int nRB = (a.B + BLOCK - 1) / BLOCK, tile = xcd_logical_tile(nRB * ((a.C + BLOCK - 1) / BLOCK));
        cb = tile < 0 ? -1 : tile / nRB;
        rb = tile - cb * nRB;
        const int lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        g = lane >> 4;
        i = lane & 15;
        c0 = cb * BLOCK + 32 * (wave >> 2) + 4 * g;
        row = rb * BLOCK + 16 * (wave & 3) + i;
    }
    __device__ __forceinline__ int cls(int x, int v) const { return c0 + 16 * x + v; }
    // z: bias added, classes beyond the shard -inf
    __device__ __forceinline__ void logits(block_logits_t& z, const FcArgs& a, char* lds) const {
        float b[2][4];                                   // on their way during the main loop
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v) b[x][v] = a.bias != nullptr && cls(x, v) < a.C ? a.bias[cls(x, v)] : 0.0f;
        block_logits(z, make_operand(a.W, a.ldw, a.C, a.D), make_operand(a.X, a.ldx, a.B, a.D), cb * BLOCK, rb * BLOCK, a.D / TILE_K, lds);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v) z[x][v] = cls(x, v) < a.C ? (a.bias != nullptr ? z[x][v] + b[x][v] : z[x][v]) : NEG_INF;
    }
};

__global__ __launch_bounds__(NTHREADS, 4) void fwd_stats_block(FcArgs a, int pitch, f32x2* __restrict__ parts,
                                                               float* __restrict__ label_logit) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    const LogitsBlock t(a);
    if (t.cb < 0) return;
    const bool row_ok = t.row < a.B;
    int local = row_ok ? a.labels[t.row] - a.class_offset : -1;
    const bool in_shard = local >= 0 && local < a.C;
    block_logits_t z;
    t.logits(z, a, lds);
    float mx = NEG_INF, s = 0.0f;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) mx = fmaxf(mx, z[x][v]);
    const float shift = exp_shift(mx);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            s += __builtin_amdgcn_exp2f(fmaf(z[x][v], LOG2E, shift));
            if (in_shard && local == t.cls(x, v)) label_logit[t.row] = z[x][v];
        }
    if (t.cb == 0 && t.wave < 4 && t.g == 0 && row_ok && !in_shard) label_logit[t.row] = 0.0f;
    merge_ms(mx, s, lane_xor(mx, 16), lane_xor(s, 16));
    merge_ms(mx, s, lane_xor(mx, 32), lane_xor(s, 32));
    float* red = reinterpret_cast<float*>(lds);          // [max, sum][64 rows] of the upper 32 classes
    const int r = 16 * (t.wave & 3) + t.i;
    if (t.wave >= 4 && t.g == 0) {
        red[r] = mx;
        red[BLOCK + r] = s;
    }
    __syncthreads();
    if (t.wave < 4 && t.g == 0) {
        merge_ms(mx, s, red[r], red[BLOCK + r]);
        parts[(int64_t)t.cb * pitch + t.row] = f32x2{mx, s};
    }
}

// dz of the batch's rows, up to whole k-steps of classes (zeros beyond the shard); one db partial per row block.
__global__ __launch_bounds__(NTHREADS, 4) void dz_block(FcArgs a, const float* __restrict__ logsumexp, float grad_scale,
                                                        uint16_t* __restrict__ dZ, int64_t ldz, float* __restrict__ db_part, XtArgs xt) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    if ((int)blockIdx.x >= xt.first_block) {
        transpose_x_tiles(a, xt, (int)blockIdx.x - xt.first_block, lds);
        return;
    }
    const LogitsBlock t(a);
    if (t.cb < 0) return;
    const bool row_ok = t.row < a.B;
    const float gs = row_ok ? grad_scale : 0.0f, lse = row_ok ? logsumexp[t.row] : 0.0f;
    const int local = row_ok ? a.labels[t.row] - a.class_offset : -1;
    block_logits_t z;
    t.logits(z, a, lds);
    const float shift = __log2f(fabsf(gs)) - lse * LOG2E;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float d = __builtin_amdgcn_exp2f(fmaf(z[x][v], LOG2E, shift));
            if (grad_scale < 0.0f) d = -d;
            z[x][v] = d - (local == t.cls(x, v) && t.cls(x, v) < a.C ? gs : 0.0f);
        }
    float* red = reinterpret_cast<float*>(lds + BLOCK_TILE_OFFSET);        // [4 row quarters][64 classes]
    if (db_part != nullptr) {
        float val[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = z[e >> 2][e & 3];
        exchange_half<4, 8>(val, t.i);
        exchange_half<2, 4>(val, t.i);
        exchange_half<1, 2>(val, t.i);
        val[0] += lane_xor(val[0], 1);
        if ((t.i & 1) == 0) {                            // lane i holds register i / 2
            const int e = t.i >> 1;
            red[(t.wave & 3) * BLOCK + 32 * (t.wave >> 2) + 16 * (e >> 2) + 4 * t.g + (e & 3)] = val[0];
        }
    }
    const u32x4 out = block_logits_rows(z, lds);         // with a barrier behind the writes to red
    const int n = t.rb * BLOCK + ((int)threadIdx.x >> 3);
    if (n < a.B) *reinterpret_cast<u32x4*>(dZ + (int64_t)n * ldz + t.cb * BLOCK + 8 * ((int)threadIdx.x & 7)) = out;
    if (db_part != nullptr && (int)threadIdx.x < BLOCK) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) s += red[q * BLOCK + threadIdx.x];
        db_part[(int64_t)t.rb * ldz + t.cb * BLOCK + threadIdx.x] = s;
    }
}

__global__ __launch_bounds__(NTHREADS, 4) void predict_block(FcArgs a, const float* __restrict__ logsumexp, uint16_t* __restrict__ P,
                                                             int64_t ldp) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    const LogitsBlock t(a);
    if (t.cb < 0) return;
    const float shift = t.row < a.B ? -logsumexp[t.row] * LOG2E : 0.0f;
    block_logits_t z;
    t.logits(z, a, lds);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) z[x][v] = __builtin_amdgcn_exp2f(fmaf(z[x][v], LOG2E, shift));
    const u32x4 out = block_logits_rows(z, lds);
    const int n = t.rb * BLOCK + ((int)threadIdx.x >> 3), c = t.cb * BLOCK + 8 * ((int)threadIdx.x & 7);
    if (n >= a.B) return;
    uint16_t* o = P + (int64_t)n * ldp + c;
    if (c + 8 <= a.C) {
        *reinterpret_cast<u32x4*>(o) = out;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (c + e < a.C) o[e] = (uint16_t)(out[e >> 1] >> (16 * (e & 1)));
    }
}

__global__ __launch_bounds__(NTHREADS, 4) void top1_block(FcArgs a, int pitch, float* __restrict__ part_val, int* __restrict__ part_cls) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    const LogitsBlock t(a);
    if (t.cb < 0) return;
    block_logits_t z;
    t.logits(z, a, lds);
    float best = NEG_INF;
    int cls = INT_MAX;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (z[x][v] > best) {                        // a lane's classes come in increasing order
                best = z[x][v];
                cls = t.cls(x, v);
            }
    better_of(best, cls, lane_xor(best, 16), __shfl_xor(cls, 16, 64));
    better_of(best, cls, lane_xor(best, 32), __shfl_xor(cls, 32, 64));
    float* red_v = reinterpret_cast<float*>(lds);        // of the upper 32 classes
    int* red_c = reinterpret_cast<int*>(red_v + BLOCK);
    const int r = 16 * (t.wave & 3) + t.i;
    if (t.wave >= 4 && t.g == 0) {
        red_v[r] = best;
        red_c[r] = cls;
    }
    __syncthreads();
    if (t.wave < 4 && t.g == 0) {
        better_of(best, cls, red_v[r], red_c[r]);
        part_val[(int64_t)t.cb * pitch + t.row] = best;
        part_cls[(int64_t)t.cb * pitch + t.row] = cls;
    }
}

struct DxArgs {
    const uint16_t* dZ; int64_t ldz;     // [Bpad][Cpad]
    const uint16_t* W; int64_t ldw;      // [C][D]
    int B, D, C;
    int nDT, nBT, splits, steps_per_split, steps_total;
    float* out; int64_t ldo; int64_t split_stride;   // out[split][b][d]
};

// dX tile: M = batch rows (A = dz, k contiguous), N = features d (B operand = W_s read k-strided: the
// narrower side of a wave's sub-tile, so the slower transposing LDS reads are the fewer ones),
// K = the shard's classes, cut into `splits` ranges.
__global__ __launch_bounds__(NTHREADS) void bwd_dx(DxArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    const int tile = xcd_logical_tile(a.nDT * a.nBT * a.splits);
    if (tile < 0) return;
    // The 32 consecutive tiles that an XCD runs at a time should share their panels: up to four batch tiles, batch
    // tiles fastest (all tiles of 32 / nBT feature tiles); more, feature tiles fastest (the tiles that share a dz
    // panel, the larger operand, sit on one XCD).
    const int td = tile % (a.nBT * a.nDT), sp = tile / (a.nBT * a.nDT);
    const int bt = a.nBT <= 4 ? td % a.nBT : td / a.nDT;
    const int dt = a.nBT <= 4 ? td / a.nBT : td % a.nDT;
    const int s0 = sp * a.steps_per_split;
    int ns = a.steps_total - s0;
    ns = ns < a.steps_per_split ? ns : a.steps_per_split;

    acc_t acc;
    zero_acc(acc);
    const Operand A = make_operand(a.dZ, a.ldz, a.B, a.ldz);      // rows beyond the batch read as zeros
    const Operand Bo = make_operand(a.W, a.ldw, a.C, a.D);          // classes beyond the shard read as zeros
    gemm_mainloop<KS>(acc, A, Bo, bt * TILE_M, dt * TILE_N, s0 * TILE_K, ns, lds);

    // The accumulator layout gives a lane four consecutive rows of one column: direct stores would be 64-byte
    // pieces.  Instead each half of the tile (the 128 rows of one wave row) goes through LDS as fp32
    // [128 rows][256 columns] (16-float chunks XOR-ed with (row >> 2) & 3, which spreads the four row groups of
    // a wave's store over the banks) and leaves in whole 1 KiB rows.
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, jl = lane & 15;
    float* out = a.out + sp * a.split_stride;
    float* tile_f32 = reinterpret_cast<float*>(lds);
    const int d_left = a.D - dt * TILE_N;
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
        if (wm == h) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int col = wave_col<KS>(wn, nt) + jl;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * mt + 4 * g + v;
                        tile_f32[row * 256 + ((((col >> 4) ^ ((row >> 2) & 3)) << 4) | (col & 15))] = acc[mt][nt][v];
                    }
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int i = 0; i < 16; ++i) {
            const int q = tid + NTHREADS * i;
            const int row = q >> 6, c4 = q & 63;
            const int grow = bt * TILE_M + h * WAVE_M + row;
            if (grow < a.B && 4 * c4 < d_left) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(
                    tile_f32 + row * 256 + ((((c4 >> 2) ^ ((row >> 2) & 3)) << 4) | ((c4 & 3) << 2)));
                *reinterpret_cast<f32x4*>(out + (int64_t)grow * a.ldo + dt * TILE_N + 4 * c4) = v;
            }
        }
        __syncthreads();
    }
}

// dX in tiles of 64 rows x 64 features (gemm_block.h), for batches and features that 256 x 256 tiles would fill poorly.  A
// tile's place in the output, and the two chunks of each thread: 4 floats of rows row() and row() + 32.
struct DxBlock {
    int split, tile, b0, d0;
    __device__ __forceinline__ DxBlock(const DxArgs& a, int logical) {
        const int nDT = a.D / BLOCK, tiles = nDT * ((a.B + BLOCK - 1) / BLOCK);
        split = logical / tiles;
        tile = logical - split * tiles;
        d0 = (tile % nDT) * BLOCK;                       // feature tiles fastest
        b0 = (tile / nDT) * BLOCK;
    }
    __device__ __forceinline__ int row() const { return b0 + ((int)threadIdx.x >> 4); }
    __device__ __forceinline__ int64_t offset(int h, int64_t ld) const { return (int64_t)(row() + 32 * h) * ld + d0 + 4 * ((int)threadIdx.x & 15); }
    __device__ __forceinline__ void compute(f32x4 (&v)[2], const DxArgs& a, char* lds) const {
        const int s0 = split * a.steps_per_split, left = a.steps_total - s0;
        const Operand A = make_operand(a.dZ, a.ldz, a.B, a.ldz);      // rows beyond the batch read as zeros
        const Operand Bo = make_operand(a.W, a.ldw, a.C, a.D);          // classes beyond the shard read as zeros
        block_acc_t acc;
        block_gemm(acc, A, Bo, b0, d0, s0 * TILE_K, left < a.steps_per_split ? left : a.steps_per_split, lds);
        block_rows_f32(v, acc, lds);
    }
};
__global__ __launch_bounds__(NTHREADS, 4) void bwd_dx_block(DxArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    const int logical = xcd_logical_tile(a.D / BLOCK * ((a.B + BLOCK - 1) / BLOCK) * a.splits);
    if (logical < 0) return;
    const DxBlock t(a, logical);
    f32x4 v[2];
    t.compute(v, a, lds);
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (t.row() + 32 * h < a.B) *reinterpret_cast<f32x4*>(a.out + t.split * a.split_stride + t.offset(h, a.ldo)) = v[h];
}

// The two small reductions that finish the backward call: the split-K partials of dX are summed in a
// fixed order (one float4 per thread and turn; optionally accumulating into the caller's dX), and the
// per-row-tile column sums into db.  Run by the workgroups of bwd_dw beyond its GEMM tiles (handed out
// last, onto compute units that the final, partial round of GEMM tiles leaves idle).
struct FinishArgs {
    const float* parts; int splits; int64_t split_stride;   // nullptr: dX was written directly
    int B, D;
    float* dX; int64_t lddx; int accumulate;
    const float* db_part; int n_db_parts; int64_t db_stride; // nullptr: no db wanted
    int C; float* db;
    int sgd; float lr;                                        // sgd: db is the bias, updated in place
    int first_block, n_blocks;
};

// Bound by the latency of its loads: FINISH_BATCH of them are in flight.  (One after the other they took longer than dW itself;
// the launch, us, one after the other and so: B = 200, D = 512, C = 16 000 (125 splits) 42.6 and 18.5; B = 1024, D = 2048, C =
// 12 500 (8 splits) 63.5 and 51.0; B = 256, D = 2048, C = 100 000 (32 splits) 140.3 and 135.5.)
constexpr int FINISH_BATCH = 16;
__device__ __forceinline__ void finish_bwd(const FinishArgs& f, int worker) {
    const int64_t stride = (int64_t)f.n_blocks * NTHREADS;
    const int64_t me = (int64_t)worker * NTHREADS + threadIdx.x;
    if (f.parts != nullptr) {
        const int d4 = f.D >> 2;
        const int64_t n4 = (int64_t)f.B * d4;
        for (int64_t i = me; i < n4; i += stride) {
            const int row = (int)(i / d4), d = (int)(i % d4) * 4;
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
            const float* at = f.parts + (int64_t)row * f.D + d;
            for (int p0 = 0; p0 < f.splits; p0 += FINISH_BATCH) {
                f32x4 v[FINISH_BATCH];
#pragma unroll
                for (int k = 0; k < FINISH_BATCH; ++k)
                    if (p0 + k < f.splits) v[k] = *reinterpret_cast<const f32x4*>(at + (p0 + k) * f.split_stride);
#pragma unroll
                for (int k = 0; k < FINISH_BATCH; ++k)
                    if (p0 + k < f.splits) s += v[k];
            }
            float* o = f.dX + (int64_t)row * f.lddx + d;
            if (f.accumulate) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] += s[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = s[e];
            }
        }
    }
    if (f.db_part != nullptr) {
        for (int64_t c = me; c < f.C; c += stride) {
            float s = 0.0f;
            for (int t0 = 0; t0 < f.n_db_parts; t0 += FINISH_BATCH) {
                float v[FINISH_BATCH];
#pragma unroll
                for (int k = 0; k < FINISH_BATCH; ++k)
                    if (t0 + k < f.n_db_parts) v[k] = f.db_part[(t0 + k) * f.db_stride + c];
#pragma unroll
                for (int k = 0; k < FINISH_BATCH; ++k)
                    if (t0 + k < f.n_db_parts) s += v[k];
            }
            f.db[c] = f.sgd ? fmaf(-f.lr, s, f.db[c]) : s;
        }
    }
}

struct DwArgs {
    const uint16_t* XT; int64_t ldxt;    // [D][Bpad]
    const uint16_t* dZ; int64_t ldz;     // [Bpad][Cpad]
    int D, C, B;
    int nDT, nCT, k_steps;
    uint16_t* dW; int64_t lddw;          // sgd: the weights themselves, updated in place
    int sgd; float lr;
    TilePlan plan;                       // full tiles, and the thin ones a ragged last round is cut into
};

// dW^T tile: M = features d (A = X^T, k contiguous), N = classes (B operand = dz read k-strided, the
// narrower side of a wave's sub-tile as in bwd_dx), K = batch rows.
// TRACE: thread 0 of the workgroup also writes the shader clock at six points of its tile, and which compute
// unit it ran on, to trace[8 * tile ..] (diagnostics; the arithmetic and the stores are the same).
template <bool TRACE>
__device__ __forceinline__ void dw_tile(const DwArgs& a, char* lds, unsigned long long* trace) {
    unsigned long long stamp[6];
    if (TRACE) stamp[0] = __builtin_readcyclecounter();
    const int tile = xcd_logical_tile(a.plan.n_full);
    if (tile < 0) return;
    const int dt = tile % a.nDT, ct = tile / a.nDT;    // feature tiles fastest: neighbours share the dz panel

    acc_t acc;
    zero_acc(acc);
    const Operand A = make_operand(a.XT, a.ldxt, a.D, a.ldxt);
    const Operand Bo = make_operand(a.dZ, a.ldz, a.B, a.ldz);      // rows beyond the batch read as zeros
    if (TRACE) stamp[1] = __builtin_readcyclecounter();
    // workgroups are dealt out 256 at a time, 32 to each XCD: alternate the direction round by round, so that a
    // compute unit's next tile finds the end of the X^T panels, which it has just read, still in the L2
    gemm_mainloop<KS>(acc, A, Bo, dt * TILE_M, ct * TILE_N, 0, a.k_steps, lds, ((blockIdx.x >> 8) & 1) != 0);
    if (TRACE) stamp[2] = __builtin_readcyclecounter();

    // [class][feature] tile through LDS, then whole 512-byte rows of dW
    const int c_left = a.C - ct * TILE_N, d_left = a.D - dt * TILE_M;
    uint16_t* out = a.dW + (int64_t)ct * TILE_N * a.lddw + dt * TILE_M;
    const int n_valid = c_left < TILE_N ? c_left : TILE_N, m_valid = d_left < TILE_M ? d_left : TILE_M;
    u32x4 weights[UPDATE_CHUNKS];
    if (a.sgd) tile_update_load(weights, out, a.lddw, n_valid, m_valid);
    acc_to_lds_bf16<KS>(acc, lds);
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();                                       // the weights may still be on their way
    if (TRACE) stamp[3] = __builtin_readcyclecounter();
    if (a.sgd) lds_tile_update_rows(lds, weights, out, a.lddw, n_valid, m_valid, a.lr);
    else lds_tile_store_rows(lds, out, a.lddw, n_valid, m_valid);
    if (TRACE) {
        stamp[4] = __builtin_readcyclecounter();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this wave's stores have been acknowledged
        stamp[5] = __builtin_readcyclecounter();
        if (threadIdx.x == 0) {
            // hardware registers HW_ID (4: wave, SIMD, compute unit, shader array and engine) and XCC_ID (20)
            const unsigned long long hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);
            const unsigned long long xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20);
            unsigned long long* t = trace + 8 * (int64_t)tile;
#pragma unroll
            for (int i = 0; i < 6; ++i) t[i] = stamp[i];
            t[6] = (unsigned long long)blockIdx.x;
            t[7] = (xcc << 32) | hw;
        }
    }
}

// Thin tile of dW: all 256 features of feature tile dt x 64 classes (piece 0 .. 3 of class tile ct); the dz
// operand is k-strided.  Used for the tiles of a ragged last round when the contraction is long (the host
// decides, plan_tiles); not traced.
__device__ __forceinline__ void dw_thin(const DwArgs& a, int q, char* lds) {
    const int tile = a.plan.n_full + (q >> 2), piece = q & 3;
    const int dt = tile % a.nDT, ct = tile / a.nDT;
    const int c0 = ct * TILE_N + piece * THIN_N;
    if (c0 >= a.C) return;                              // a piece entirely beyond the shard's classes
    thin_acc_t acc;
#pragma unroll
    for (int i = 0; i < THIN_MT; ++i)
#pragma unroll
        for (int j = 0; j < THIN_NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const Operand A = make_operand(a.XT, a.ldxt, a.D, a.ldxt);
    const Operand Bo = make_operand(a.dZ, a.ldz, a.B, a.ldz);      // rows beyond the batch read as zeros
    thin_mainloop<KS>(acc, A, Bo, dt * TILE_M, c0, 0, a.k_steps, lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, jl = lane & 15;
#pragma unroll
    for (int nt = 0; nt < THIN_NT; ++nt) {
        const int n = 16 * nt + jl;
#pragma unroll
        for (int mt = 0; mt < THIN_MT; ++mt) {
            u32x2 pk;
            pk[0] = pack_bf16(acc[mt][nt][0], acc[mt][nt][1]);
            pk[1] = pack_bf16(acc[mt][nt][2], acc[mt][nt][3]);
            *reinterpret_cast<u32x2*>(lds + out_tile_offset(n, wave * THIN_WAVE_M + 16 * mt + 4 * g)) = pk;
        }
    }
    __syncthreads();
    const int c_left = a.C - c0, d_left = a.D - dt * TILE_M;
    uint16_t* out = a.dW + (int64_t)c0 * a.lddw + dt * TILE_M;
    const int n_valid = c_left < THIN_N ? c_left : THIN_N, m_valid = d_left < TILE_M ? d_left : TILE_M;
    if (a.sgd) {
        u32x4 weights[UPDATE_CHUNKS];
        tile_update_load(weights, out, a.lddw, n_valid, m_valid);
        lds_tile_update_rows(lds, weights, out, a.lddw, n_valid, m_valid, a.lr);
    } else {
        lds_tile_store_rows(lds, out, a.lddw, n_valid, m_valid);
    }
}

// dW in tiles of 64 features x 64 classes, two workgroups to a compute unit (gemm_block.h): for layers whose 256 x 256
// tiles would leave most of the chip idle while each walks the contraction.
__device__ __forceinline__ void dw_block(const DwArgs& a, int tile, char* lds) {
    const int nDT = a.D / BLOCK, d0 = (tile % nDT) * BLOCK, c0 = (tile / nDT) * BLOCK;   // feature tiles fastest: neighbours share the dz panel
    const Operand A = make_operand(a.XT, a.ldxt, a.D, a.ldxt);
    const Operand Bo = make_operand(a.dZ, a.ldz, a.B, a.ldz);          // rows beyond the batch read as zeros
    // one 16-byte chunk of the output per thread: class c0 + tid / 8, features d0 + 8 * (tid % 8)
    const int row = (int)threadIdx.x >> 3, chunk = (int)threadIdx.x & 7;
    uint16_t* out = a.dW + (int64_t)(c0 + row) * a.lddw + d0 + 8 * chunk;
    const bool live = c0 + row < a.C;
    u32x4 w = {0, 0, 0, 0};
    if (a.sgd && live) w = *reinterpret_cast<const u32x4*>(out);
    block_acc_t acc;
    block_gemm(acc, A, Bo, d0, c0, 0, a.k_steps, lds);
    u32x4 g = block_rows_bf16(acc, lds);
    if (a.sgd) g = updated_weights(w, g, a.lr);
    if (live) __builtin_nontemporal_store(g, reinterpret_cast<u32x4*>(out));
}
__global__ __launch_bounds__(NTHREADS, 4) void bwd_dw_block(DwArgs a, FinishArgs fin) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    if ((int)blockIdx.x >= fin.first_block) {
        finish_bwd(fin, (int)blockIdx.x - fin.first_block);
        return;
    }
    const int tile = xcd_logical_tile(a.D / BLOCK * ((a.C + BLOCK - 1) / BLOCK));
    if (tile >= 0) dw_block(a, tile, lds);
}

// dX of whole contractions and dW in one launch, both in 64 x 64 tiles (neither reads what the other writes: no fused update).
// (With splits, whose last workgroup added the partial sums: correct, but what one XCD's L2 wrote has to reach the others
// first, and that took 10 to 100 us.)
struct DxTail {
    float* dX; int64_t lddx; int accumulate;
    int dw_first_block;
};
__global__ __launch_bounds__(NTHREADS, 4) void bwd_dx_dw_block(DxArgs x, DxTail tail, DwArgs w, FinishArgs fin) {
    __shared__ __attribute__((aligned(16))) char lds[BLOCK_LDS_BYTES];
    const int bid = blockIdx.x;
    if (bid >= fin.first_block) {
        finish_bwd(fin, bid - fin.first_block);
        return;
    }
    if (bid >= tail.dw_first_block) {
        const int tile = xcd_logical_tile(w.D / BLOCK * ((w.C + BLOCK - 1) / BLOCK), bid - tail.dw_first_block);
        if (tile >= 0) dw_block(w, tile, lds);
        return;
    }
    const int logical = xcd_logical_tile(x.D / BLOCK * ((x.B + BLOCK - 1) / BLOCK));
    if (logical < 0) return;
    const DxBlock t(x, logical);
    f32x4 v[2];
    t.compute(v, x, lds);
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (t.row() + 32 * h < x.B) {
            f32x4* o = reinterpret_cast<f32x4*>(tail.dX + t.offset(h, tail.lddx));
            *o = tail.accumulate ? *o + v[h] : v[h];
        }
}

__global__ __launch_bounds__(NTHREADS) void bwd_dw(DwArgs a, FinishArgs fin) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    if ((int)blockIdx.x >= fin.first_block) {
        finish_bwd(fin, (int)blockIdx.x - fin.first_block);
        return;
    }
    if ((int)blockIdx.x >= a.plan.thin_first) {
        dw_thin(a, (int)blockIdx.x - a.plan.thin_first, lds);
        return;
    }
    dw_tile<false>(a, lds, nullptr);
}

// The same tiles as a stream (gemm_stream.h): nothing waits for the 128 KiB that leave a compute unit per tile, and no
// tile for its first loads.  B = 1024, D = 2048, C = 100 000: 380 -> 345 us; B = 256: 181 -> 141 us; B = 1024, C = 12 500:
// 69 -> 67 us (1.5 tiles per compute unit).  Feature tiles fastest and the direction of the contraction
// alternating round by round as in dw_tile.
template <int RATE>
struct DwEpilogue : RowStore<RATE> {
    const DwArgs& a;
    const StreamShare& share;
    int round = -1;
    __device__ __forceinline__ DwEpilogue(const DwArgs& args, const StreamShare& s, char* lds) : a(args), share(s) {
        this->init(a.lddw, lds);
    }
    __device__ __forceinline__ void begin_next() { ++round; }
    template <int Q>
    __device__ __forceinline__ void finish(const acc_t& acc) {
        if (Q == 0) {
            const int tile = share.tile(round), dt = tile % a.nDT, ct = tile / a.nDT;
            const int64_t off = (int64_t)ct * TILE_N * a.lddw + dt * TILE_M;
            const int64_t bytes = (((int64_t)a.C - 1) * a.lddw + a.D - off) * 2;
            this->at.base = a.dW + off;
            this->at.records = bytes < 0xfffffff0ll ? (uint32_t)bytes : 0xfffffff0u;
            this->at.m_valid = a.D - dt * TILE_M;
        }
        this->template put<Q>(acc);
    }
};

template <int RATE, bool PREFETCH>
__global__ __launch_bounds__(NTHREADS) void bwd_dw_stream(DwArgs a, FinishArgs fin) {
    __shared__ __attribute__((aligned(16))) char lds[STREAM_LDS_BYTES];
    if ((int)blockIdx.x >= fin.first_block) {
        finish_bwd(fin, (int)blockIdx.x - fin.first_block);
        return;
    }
    if ((int)blockIdx.x >= a.plan.thin_first) {
        dw_thin(a, (int)blockIdx.x - a.plan.thin_first, lds);
        return;
    }
    const StreamShare share(a.plan.n_full, blockIdx.x);
    if (share.count == 0) return;
    DwEpilogue<RATE> epi(a, share, lds);
    const Operand A = make_operand(a.XT, a.ldxt, a.D, a.ldxt);
    const Operand Bo = make_operand(a.dZ, a.ldz, a.B, a.ldz);      // rows beyond the batch read as zeros
    const auto tile_at = [&](int round) {
        const int tile = share.tile(round);
        return StreamTile{(tile % a.nDT) * TILE_M, (tile / a.nDT) * TILE_N, (round & 1) != 0};
    };
    gemm_stream<RATE, PREFETCH>(A, Bo, a.k_steps, share.count, tile_at, PrefetchShare(share.first % a.nDT, a.nDT), epi, lds);
}

__global__ __launch_bounds__(NTHREADS) void bwd_dw_traced(DwArgs a, FinishArgs fin, unsigned long long* trace) {
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    if ((int)blockIdx.x >= fin.first_block) {
        finish_bwd(fin, (int)blockIdx.x - fin.first_block);
        return;
    }
    if ((int)blockIdx.x >= a.plan.thin_first) {
        dw_thin(a, (int)blockIdx.x - a.plan.thin_first, lds);
        return;
    }
    dw_tile<true>(a, lds, trace);
}

// ---- host side -----------------------------------------------------------------------------------

static inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// The mean is taken by the combine launch itself while one workgroup is as quick as two launches; us, two launches and one, 1 to 8 shards
// (and a launch less on the host, 3.7): B = 32 3.5 and 2.5; B = 1024 4.1 and 3.1; B = 1536 4.1 and 3.6; B = 1792 4.2 and 3.9; B = 1857, where the
// rows of the second turn end within a wave, 4.2 and 4.7; B = 1920 4.2 and 4.1; B = 4096 4.8 and 6.3; 16 shards, B = 2048 5.1 and 7.6.
constexpr int COMBINE_MEAN_ROWS = 1792;
#define WS_LAUNCH_SMALL(kid, name, plan, grid, stream, ...)                                                   \
    do {                                                                                                      \
        if ((plan).rows == 16) WS_LAUNCH(kid, name<1>, dim3(grid), dim3(SMALL_THREADS), stream, __VA_ARGS__); \
        else WS_LAUNCH(kid, name<2>, dim3(grid), dim3(SMALL_THREADS), stream, __VA_ARGS__);                  \
    } while (0)
// Predictions and arg-max add the products of a logit in the order of the step, whatever kernels the step runs.
static void set_step_order(FcArgs& a) {
    const LogitsPlan step = plan_logits(a.B, a.D, a.C, SMALL_STEP);
    a.order = logits_order(step);
    a.ranges = step.ranges;
}

static int check_fc_common(const void* X, int64_t ldx, const void* W, int64_t ldw, const float* bias,
                           const int32_t* labels, int32_t B, int32_t D, int32_t C, int32_t class_offset) {
    if (!X || !W || !labels) return WS_ERR_NULL;
    if (!shape_ok(B, D, C)) return WS_ERR_SHAPE;
    if (ldx < D || ldw < D) return WS_ERR_SHAPE;
    if (!fits_32bit_offsets(B, ldx) || !fits_32bit_offsets(C, ldw)) return WS_ERR_SHAPE;
    if (class_offset < 0 || (int64_t)class_offset + C > INT32_MAX) return WS_ERR_RANGE;
    if (!aligned(X, 16) || !aligned(W, 16) || ldx % 8 || ldw % 8) return WS_ERR_ALIGN;
    if (!aligned(labels, 4) || (bias && !aligned(bias, 4))) return WS_ERR_ALIGN;
    return WS_OK;
}


// ---- built-in scratch of the entry point that allocates nothing ---------------------------------------
// A fixed array in the code object stands in for the forward call's workspace.  Every GPU the library
// runs on holds its own copy at its own address; in host code the array's name is only a handle, so the
// device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[WS_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static std::atomic<void*> g_scratch_ptr[MAX_DEVICES];

// Device address of `scratch` on the current device (looked up at the first call on that device).
static int static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return WS_ERR_HIP;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return WS_ERR_HIP;
        }
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return WS_OK;
}

// ---- optional per-kernel timing --------------------------------------------------------------------
// When enabled, every kernel launch is bracketed by a pair of events recorded on the launch stream.
// The pairs come from a pool created by ws_profile_enable; when the pool is used up, launches go
// untimed.  Not thread safe; meant for benchmarks.
enum KernelId { KID_FWD = 0, KID_MERGE, KID_COMBINE, KID_MEAN, KID_DZ, KID_DX, KID_DW, KID_PREDICT, KID_TOP1, KID_TOP1_MERGE, KID_DX_DW, KID_COUNT };
static const char* const kKernelNames[KID_COUNT] = {"fwd_logits_stats", "merge_class_tiles", "combine_partials",
                                                    "mean_loss", "bwd_recompute_dz", "bwd_dx", "bwd_dw",
                                                    "predict_probs", "top1_logits", "merge_top1", "bwd_dx_dw"};
struct ProfState {
    bool on = false;
    bool paused = false;
    int capacity = 0, used = 0;
    hipEvent_t* start = nullptr;
    hipEvent_t* stop = nullptr;
    int* kid = nullptr;
};
static ProfState g_prof;

// ws_profile_trace_dw: where the dW kernel of the following backward calls writes its per-tile clock stamps.
static unsigned long long* g_dw_trace = nullptr;
static int64_t g_dw_trace_tiles = 0;

struct ScopedTimer {
    int slot = -1;
    hipStream_t s;
    ScopedTimer(int kid, hipStream_t stream) : s(stream) {
        if (g_prof.on && !g_prof.paused && g_prof.used < g_prof.capacity) {
            slot = g_prof.used++;
            g_prof.kid[slot] = kid;
            (void)hipEventRecord(g_prof.start[slot], s);
        }
    }
    ~ScopedTimer() {
        if (slot >= 0) (void)hipEventRecord(g_prof.stop[slot], s);
    }
};
#define WS_LAUNCH(kid, kernel, grid, block, stream, ...)                         \
    do {                                                                         \
        ScopedTimer timer_(kid, stream);                                         \
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);         \
    } while (0)

static int launch_status() { return hipGetLastError() == hipSuccess ? WS_OK : WS_ERR_HIP; }

}  // namespace ws

using namespace ws;

extern "C" {

const char* ws_status_string(int status) {
    switch (status) {
        case WS_OK: return "WS_OK";
        case WS_ERR_NULL: return "WS_ERR_NULL";
        case WS_ERR_SHAPE: return "WS_ERR_SHAPE";
        case WS_ERR_ALIGN: return "WS_ERR_ALIGN";
        case WS_ERR_RANGE: return "WS_ERR_RANGE";
        case WS_ERR_WORKSPACE: return "WS_ERR_WORKSPACE";
        case WS_ERR_HIP: return "WS_ERR_HIP";
        case WS_ERR_LIMIT: return "WS_ERR_LIMIT";
        default: return "WS_ERR_UNKNOWN";
    }
}

int ws_version(void) { return 1220; }

size_t ws_fwd_workspace_bytes(int32_t B, int32_t D, int32_t C_shard) {
    return shape_ok(B, D, C_shard) ? fwd_bytes(B, D, C_shard) : 0;
}

size_t ws_bwd_workspace_bytes(int32_t B, int32_t D, int32_t C_shard) {
    if (!shape_ok(B, D, C_shard)) return 0;
    const BwdPlan p = plan_bwd(B, D, C_shard);
    return p.bytes();
}

// Argument checks of the forward call that do not concern the workspace.
static int check_fwd(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                     const int32_t* labels, int32_t B, int32_t D, int32_t C_shard, int32_t class_offset,
                     float* row_max, float* row_sumexp, float* label_logit) {
    if (!row_max || !row_sumexp || !label_logit) return WS_ERR_NULL;
    int st = check_fc_common(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset);
    if (st != WS_OK) return st;
    if (!aligned(row_max, 4) || !aligned(row_sumexp, 4) || !aligned(label_logit, 4)) return WS_ERR_ALIGN;
    return WS_OK;
}

// Launches of the forward call; `workspace` holds least_fwd_bytes at least, 16-byte aligned.
static int launch_fwd(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                      const int32_t* labels, int32_t B, int32_t D, int32_t C_shard, int32_t class_offset,
                      float* row_max, float* row_sumexp, float* label_logit, void* workspace, size_t workspace_bytes,
                      void* stream) {
    FcArgs a;
    a.last_tile_first = 0;
    a.X = static_cast<const uint16_t*>(X); a.ldx = ldx;
    a.W = static_cast<const uint16_t*>(W_shard); a.ldw = ldw;
    a.bias = b_shard; a.labels = labels;
    a.B = B; a.D = D; a.C = C_shard; a.class_offset = class_offset;
    a.Bpad = (int)round_up(B, 256);
    a.nBT = a.Bpad / 256;
    a.nCT = (int)(round_up(C_shard, 256) / 256);
    const LogitsPlan step = plan_logits(B, D, C_shard, SMALL_STEP);
    a.order = logits_order(step);
    a.ranges = step.ranges;
    LogitsPlan p = plan_forward(B, D, C_shard, step);
    if (workspace_bytes < p.bytes()) p = plan_wide(B, C_shard);
    f32x2* parts = static_cast<f32x2*>(workspace);
    const int n_parts = (int)p.parts, pitch = (int)p.pitch;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (p.way == WAY_SMALL) {
        const SmallPlan sp(B, C_shard);
        WS_LAUNCH_SMALL(KID_FWD, fwd_stats_small, sp, sp.ranges, s, a, sp.range, parts, label_logit);
    } else if (p.way == WAY_BLOCKS) {
        WS_LAUNCH(KID_FWD, fwd_stats_block, dim3(xcd_grid(n_parts * (pitch / BLOCK))), dim3(NTHREADS), s, a, pitch, parts, label_logit);
    } else if (p.way == WAY_LISTS) {
        WS_LAUNCH(KID_FWD, fwd_logits_list, dim3(list_grid(a.ranges, a.nBT)), dim3(NTHREADS), s,
                  (FwdArgs{a, parts, label_logit}));
    } else {
        a.plan = plan_tiles(a.nBT * a.nCT, LOGITS_MAX_THIN_TAIL);
        WS_LAUNCH(KID_FWD, fwd_logits_stats, dim3(a.plan.thin_first + a.plan.n_thin), dim3(NTHREADS), s, a, parts,
                  label_logit);
    }
    WS_LAUNCH(KID_MERGE, merge_class_tiles, dim3((B + MERGE_ROWS - 1) / MERGE_ROWS), dim3(64 * MERGE_ROWS), s, parts, n_parts, pitch, B,
              row_max, row_sumexp);
    return launch_status();
}

int ws_split_fc_fwd(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                    const int32_t* labels, int32_t B, int32_t D, int32_t C_shard, int32_t class_offset,
                    float* row_max, float* row_sumexp, float* label_logit, void* workspace,
                    size_t workspace_bytes, void* stream) {
    int st = check_fwd(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset, row_max, row_sumexp,
                       label_logit);
    if (st != WS_OK) return st;
    if (!workspace || workspace_bytes < least_fwd_bytes(B, C_shard)) return WS_ERR_WORKSPACE;
    if (!aligned(workspace, 16)) return WS_ERR_ALIGN;
    return launch_fwd(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset, row_max, row_sumexp,
                      label_logit, workspace, workspace_bytes, stream);
}

int ws_split_fc_fwd_static(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                           const int32_t* labels, int32_t B, int32_t D, int32_t C_shard, int32_t class_offset,
                           float* row_max, float* row_sumexp, float* label_logit, void* stream) {
    int st = check_fwd(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset, row_max, row_sumexp,
                       label_logit);
    if (st != WS_OK) return st;
    if (least_fwd_bytes(B, C_shard) > (size_t)WS_STATIC_SCRATCH_BYTES) return WS_ERR_LIMIT;
    void* ws_ptr = nullptr;
    st = static_scratch(&ws_ptr);
    if (st != WS_OK) return st;
    // every partial the merge reads is written by the logits kernel of the same call: nothing to clear
    return launch_fwd(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset, row_max, row_sumexp,
                      label_logit, ws_ptr, (size_t)WS_STATIC_SCRATCH_BYTES, stream);
}

int ws_combine_partials(const float* row_max, const float* row_sumexp, const float* label_logit, int32_t S,
                        int32_t B, int64_t shard_stride, float* logsumexp, float* loss_rows, float* loss_mean,
                        void* stream) {
    if (!row_max || !row_sumexp || !label_logit || !logsumexp || !loss_rows) return WS_ERR_NULL;
    if (B <= 0 || shard_stride < B) return WS_ERR_SHAPE;
    if (S < 1 || S > 65536) return WS_ERR_RANGE;
    if (!aligned(row_max, 4) || !aligned(row_sumexp, 4) || !aligned(label_logit, 4) || !aligned(logsumexp, 4) ||
        !aligned(loss_rows, 4) || (loss_mean && !aligned(loss_mean, 4)))
        return WS_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (loss_mean && B <= COMBINE_MEAN_ROWS && S <= COMBINE_BATCH) {
        WS_LAUNCH(KID_COMBINE, combine_mean_kernel, dim3(1), dim3(1024), s, row_max, row_sumexp, label_logit, S, B, shard_stride,
                  logsumexp, loss_rows, loss_mean);
        return launch_status();
    }
    WS_LAUNCH(KID_COMBINE, combine_partials_kernel, dim3((B + 63) / 64), dim3(64), s, row_max, row_sumexp,
                       label_logit, S, B, shard_stride, logsumexp, loss_rows);
    if (loss_mean) WS_LAUNCH(KID_MEAN, mean_loss_kernel, dim3(1), dim3(1024), s, loss_rows, B, loss_mean);
    return launch_status();
}

// The backward call.  sgd = 0: dW_shard / db_shard receive the gradients.  sgd = 1: dW_shard is the weight
// matrix itself (== W_shard) and db_shard the bias itself (== b_shard or NULL); both are updated in place
// by the last kernel, after every kernel that reads them.
static int run_bwd(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                   const float* logsumexp, const int32_t* labels, int32_t B, int32_t D, int32_t C_shard,
                   int32_t class_offset, float grad_scale, float* dX_partial, int64_t lddx,
                   int32_t accumulate_dx, void* dW_shard, int64_t lddw, float* db_shard, void* workspace,
                   size_t workspace_bytes, void* stream, int sgd, float lr) {
    if (!logsumexp || !dX_partial || !dW_shard) return WS_ERR_NULL;
    int st = check_fc_common(X, ldx, W_shard, ldw, b_shard, labels, B, D, C_shard, class_offset);
    if (st != WS_OK) return st;
    if (lddx < D || lddw < D) return WS_ERR_SHAPE;
    if (!aligned(dX_partial, 16) || !aligned(dW_shard, 16) || lddx % 4 || lddw % 8) return WS_ERR_ALIGN;
    if (!aligned(logsumexp, 4) || (db_shard && !aligned(db_shard, 4))) return WS_ERR_ALIGN;
    const BwdPlan p = plan_bwd(B, D, C_shard);
    if (!fits_32bit_offsets(p.Bpad, p.Cpad) || !fits_32bit_offsets(D, p.Bpad))
        return WS_ERR_SHAPE;
    if (!workspace || workspace_bytes < p.bytes()) return WS_ERR_WORKSPACE;
    if (!aligned(workspace, 16)) return WS_ERR_ALIGN;
    if (g_dw_trace != nullptr && (int64_t)p.nDT * p.nCT > g_dw_trace_tiles) return WS_ERR_WORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(stream);
    uint16_t* dZ = static_cast<uint16_t*>(workspace);
    uint16_t* XT = dZ + (size_t)p.Bpad * p.Cpad;
    float* db_part = reinterpret_cast<float*>(static_cast<char*>(workspace) + p.dz_bytes + p.xt_bytes);
    float* parts = db_part + (size_t)4 * p.nBT * p.Cpad;

    FcArgs a;
    a.last_tile_first = 1;   // the forward call has just read the last class tiles of W: they may still be in the Infinity Cache
    a.X = static_cast<const uint16_t*>(X); a.ldx = ldx;
    a.W = static_cast<const uint16_t*>(W_shard); a.ldw = ldw;
    a.bias = b_shard; a.labels = labels;
    a.B = B; a.D = D; a.C = C_shard; a.class_offset = class_offset;
    a.Bpad = (int)p.Bpad; a.nBT = p.nBT; a.nCT = p.nCT;
    const bool one_launch = p.one_launch() && !sgd && g_dw_trace == nullptr;
    XtArgs xt;
    xt.XT = XT; xt.ldxt = p.Bpad;
    xt.n_blocks = (int)std::min<int64_t>(((B + 63) / 64) * (int64_t)(D / 64), SIDE_BLOCKS);
    const LogitsPlan lp = plan_logits(B, D, C_shard, SMALL_STEP);
    a.order = logits_order(lp);
    a.ranges = lp.ranges;
    if (lp.way == WAY_SMALL) {
        const SmallPlan sp(B, (int32_t)round_up(C_shard, TILE_K));
        xt.first_block = sp.ranges;
        WS_LAUNCH_SMALL(KID_DZ, dz_small, sp, xt.first_block + xt.n_blocks, s, a, sp.range, logsumexp, grad_scale, dZ, p.Cpad,
                        db_shard ? db_part : nullptr, xt);
    } else if (lp.way == WAY_BLOCKS) {
        xt.first_block = xcd_grid((int)(lp.parts * (lp.pitch / BLOCK)));
        WS_LAUNCH(KID_DZ, dz_block, dim3(xt.first_block + xt.n_blocks), dim3(NTHREADS), s, a, logsumexp, grad_scale, dZ, p.Cpad,
                  db_shard ? db_part : nullptr, xt);
    } else if (lp.way == WAY_LISTS) {
        xt.first_block = list_grid(a.ranges, a.nBT);
        WS_LAUNCH(KID_DZ, bwd_dz_list, dim3(xt.first_block + xt.n_blocks), dim3(NTHREADS), s,
                  (DzArgs{a, logsumexp, grad_scale, dZ, p.Cpad, db_shard ? db_part : nullptr, xt}));
    } else {
        a.plan = plan_tiles(p.nBT * p.nCT, LOGITS_MAX_THIN_TAIL);
        xt.first_block = a.plan.thin_first + a.plan.n_thin;
        WS_LAUNCH(KID_DZ, bwd_recompute_dz, dim3(xt.first_block + xt.n_blocks), dim3(NTHREADS), s, a, logsumexp,
                  grad_scale, dZ, p.Cpad, db_shard ? db_part : nullptr, xt);
    }

    DxArgs x;
    x.dZ = dZ; x.ldz = p.Cpad; x.W = a.W; x.ldw = ldw;
    x.B = B; x.D = D; x.C = C_shard;
    x.nDT = p.nDT; x.nBT = p.nBT; x.splits = p.splits; x.steps_per_split = p.steps_per_split;
    x.steps_total = p.steps_total;
    const bool direct = p.splits == 1 && !accumulate_dx;
    x.out = direct ? dX_partial : parts;
    x.ldo = direct ? lddx : D;
    x.split_stride = (int64_t)B * D;
    if (one_launch) {
        // with dW, below
    } else if (p.dx_small) {
        WS_LAUNCH(KID_DX, bwd_dx_block, dim3(xcd_grid((D / BLOCK) * ((B + BLOCK - 1) / BLOCK) * p.splits)), dim3(NTHREADS), s, x);
    } else {
        WS_LAUNCH(KID_DX, bwd_dx, dim3(xcd_grid(p.nDT * p.nBT * p.splits)), dim3(NTHREADS), s, x);
    }
    DwArgs w;
    w.XT = XT; w.ldxt = p.Bpad; w.dZ = dZ; w.ldz = p.Cpad;
    w.D = D; w.C = C_shard; w.B = B;
    w.nDT = p.nDT; w.nCT = p.nCT; w.k_steps = (B + TILE_K - 1) / TILE_K;
    w.dW = static_cast<uint16_t*>(dW_shard); w.lddw = lddw;
    w.sgd = sgd; w.lr = lr;
    w.plan = plan_tiles(p.nDT * p.nCT, dw_max_thin_tail(p.nDT * p.nCT, w.k_steps));
    FinishArgs f;
    f.parts = direct ? nullptr : parts; f.splits = p.splits; f.split_stride = (int64_t)B * D;
    f.B = B; f.D = D; f.dX = dX_partial; f.lddx = lddx; f.accumulate = accumulate_dx;
    f.db_part = db_shard ? db_part : nullptr; f.n_db_parts = lp.way == WAY_SMALL ? 1 : lp.way == WAY_BLOCKS ? (B + BLOCK - 1) / BLOCK : 4 * p.nBT; f.db_stride = p.Cpad;
    f.C = C_shard; f.db = db_shard;
    f.sgd = sgd; f.lr = lr;
    f.first_block = w.plan.thin_first + w.plan.n_thin;
    f.n_blocks = (f.parts || f.db_part) ? SIDE_BLOCKS : 0;
    if (one_launch) {
        const DxTail t = {dX_partial, lddx, accumulate_dx, xcd_grid((D / BLOCK) * ((B + BLOCK - 1) / BLOCK))};
        f.parts = nullptr;
        f.first_block = t.dw_first_block + xcd_grid((D / BLOCK) * ((C_shard + BLOCK - 1) / BLOCK));
        f.n_blocks = f.db_part ? std::min((C_shard + NTHREADS - 1) / NTHREADS, SIDE_BLOCKS) : 0;
        WS_LAUNCH(KID_DX_DW, bwd_dx_dw_block, dim3(f.first_block + f.n_blocks), dim3(NTHREADS), s, x, t, w, f);
    } else if (g_dw_trace == nullptr && p.dw_small) {
        f.first_block = xcd_grid((D / BLOCK) * ((C_shard + BLOCK - 1) / BLOCK));
        WS_LAUNCH(KID_DW, bwd_dw_block, dim3(f.first_block + f.n_blocks), dim3(NTHREADS), s, w, f);
    } else if (g_dw_trace != nullptr) {
        WS_LAUNCH(KID_DW, bwd_dw_traced, dim3(f.first_block + f.n_blocks), dim3(NTHREADS), s, w, f, g_dw_trace);
    } else if (!sgd && dw_streams(p.nDT, w.plan.n_full, w.k_steps, lddw)) {
        w.plan.thin_first = STREAM_WGS;
        f.first_block = w.plan.thin_first + w.plan.n_thin;
        const bool far = dw_prefetches(p.nDT, 2 * (p.Bpad * p.Cpad + (int64_t)C_shard * D), w.k_steps);
        const int rate = stream_rate(w.k_steps);
        auto kernel = far ? (rate == 1 ? bwd_dw_stream<1, true> : rate == 2 ? bwd_dw_stream<2, true> : bwd_dw_stream<4, true>)
                          : (rate == 1 ? bwd_dw_stream<1, false> : rate == 2 ? bwd_dw_stream<2, false> : bwd_dw_stream<4, false>);
        WS_LAUNCH(KID_DW, kernel, dim3(f.first_block + f.n_blocks), dim3(NTHREADS), s, w, f);
    } else {
        WS_LAUNCH(KID_DW, bwd_dw, dim3(f.first_block + f.n_blocks), dim3(NTHREADS), s, w, f);
    }
    return launch_status();
}

int ws_split_fc_bwd(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                    const float* logsumexp, const int32_t* labels, int32_t B, int32_t D, int32_t C_shard,
                    int32_t class_offset, float grad_scale, float* dX_partial, int64_t lddx,
                    int32_t accumulate_dx, void* dW_shard, int64_t lddw, float* db_shard, void* workspace,
                    size_t workspace_bytes, void* stream) {
    return run_bwd(X, ldx, W_shard, ldw, b_shard, logsumexp, labels, B, D, C_shard, class_offset, grad_scale,
                   dX_partial, lddx, accumulate_dx, dW_shard, lddw, db_shard, workspace, workspace_bytes, stream, 0,
                   0.0f);
}

int ws_split_fc_bwd_sgd(const void* X, int64_t ldx, void* W_shard, int64_t ldw, float* b_shard,
                        const float* logsumexp, const int32_t* labels, int32_t B, int32_t D, int32_t C_shard,
                        int32_t class_offset, float grad_scale, float lr, float* dX_partial, int64_t lddx,
                        int32_t accumulate_dx, void* workspace, size_t workspace_bytes, void* stream) {
    if (!(lr == lr) || lr - lr != 0.0f) return WS_ERR_RANGE;          // NaN or infinite learning rate
    return run_bwd(X, ldx, W_shard, ldw, b_shard, logsumexp, labels, B, D, C_shard, class_offset, grad_scale,
                   dX_partial, lddx, accumulate_dx, W_shard, ldw, b_shard, workspace, workspace_bytes, stream, 1, lr);
}

static void launch_merge_top1(const float* val, const int* cls, int n, int64_t stride, int B, int base, float* out_val,
                              int* out_cls, hipStream_t s) {
    if (n <= MERGE_FEW)
        WS_LAUNCH(KID_TOP1_MERGE, merge_top1_few, dim3((B + 63) / 64), dim3(64), s, val, cls, n, stride, B, base, out_val, out_cls);
    else
        WS_LAUNCH(KID_TOP1_MERGE, merge_top1, dim3((B + 15) / 16), dim3(1024), s, val, cls, n, stride, B, base, out_val, out_cls);
}

int ws_split_fc_predict(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard,
                        const float* logsumexp, int32_t B, int32_t D, int32_t C_shard, void* P, int64_t ldp,
                        void* stream) {
    if (!X || !W_shard || !logsumexp || !P) return WS_ERR_NULL;
    if (!shape_ok(B, D, C_shard)) return WS_ERR_SHAPE;
    if (ldx < D || ldw < D || ldp < C_shard) return WS_ERR_SHAPE;
    if (!fits_32bit_offsets(B, ldx) || !fits_32bit_offsets(C_shard, ldw)) return WS_ERR_SHAPE;
    if (!aligned(X, 16) || !aligned(W_shard, 16) || !aligned(P, 16) || ldx % 8 || ldw % 8 || ldp % 8) return WS_ERR_ALIGN;
    if (!aligned(logsumexp, 4) || (b_shard && !aligned(b_shard, 4))) return WS_ERR_ALIGN;
    FcArgs a;
    a.last_tile_first = 0;
    a.X = static_cast<const uint16_t*>(X); a.ldx = ldx;
    a.W = static_cast<const uint16_t*>(W_shard); a.ldw = ldw;
    a.bias = b_shard; a.labels = nullptr;
    a.B = B; a.D = D; a.C = C_shard; a.class_offset = 0;
    a.Bpad = (int)round_up(B, 256);
    a.nBT = a.Bpad / 256;
    a.nCT = (int)(round_up(C_shard, 256) / 256);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const LogitsPlan p = plan_logits(B, D, C_shard, SMALL_PROBS);
    set_step_order(a);
    if (p.way == WAY_SMALL) {
        const SmallPlan sp(B, C_shard);
        WS_LAUNCH_SMALL(KID_PREDICT, predict_small, sp, sp.ranges, s, a, sp.range, logsumexp, static_cast<uint16_t*>(P), ldp);
    } else if (p.way == WAY_BLOCKS) {
        WS_LAUNCH(KID_PREDICT, predict_block, dim3(xcd_grid((int)(p.parts * (p.pitch / BLOCK)))), dim3(NTHREADS), s, a, logsumexp,
                  static_cast<uint16_t*>(P), ldp);
    } else {
        WS_LAUNCH(KID_PREDICT, predict_probs, dim3(xcd_grid(a.nBT * a.nCT)), dim3(NTHREADS), s, a, logsumexp,
                  static_cast<uint16_t*>(P), ldp);
    }
    return launch_status();
}

int ws_split_fc_top1(const void* X, int64_t ldx, const void* W_shard, int64_t ldw, const float* b_shard, int32_t B,
                     int32_t D, int32_t C_shard, int32_t class_offset, float* top_logit, int32_t* top_class,
                     void* workspace, size_t workspace_bytes, void* stream) {
    if (!X || !W_shard || !top_logit || !top_class) return WS_ERR_NULL;
    if (!shape_ok(B, D, C_shard)) return WS_ERR_SHAPE;
    if (ldx < D || ldw < D) return WS_ERR_SHAPE;
    if (!fits_32bit_offsets(B, ldx) || !fits_32bit_offsets(C_shard, ldw)) return WS_ERR_SHAPE;
    if (class_offset < 0 || (int64_t)class_offset + C_shard > INT32_MAX) return WS_ERR_RANGE;
    if (!aligned(X, 16) || !aligned(W_shard, 16) || ldx % 8 || ldw % 8) return WS_ERR_ALIGN;
    if (!aligned(top_logit, 4) || !aligned(top_class, 4) || (b_shard && !aligned(b_shard, 4))) return WS_ERR_ALIGN;
    if (!workspace || workspace_bytes < least_fwd_bytes(B, C_shard)) return WS_ERR_WORKSPACE;
    if (!aligned(workspace, 16)) return WS_ERR_ALIGN;
    FcArgs a;
    a.last_tile_first = 0;
    a.X = static_cast<const uint16_t*>(X); a.ldx = ldx;
    a.W = static_cast<const uint16_t*>(W_shard); a.ldw = ldw;
    a.bias = b_shard; a.labels = nullptr;
    a.B = B; a.D = D; a.C = C_shard; a.class_offset = class_offset;
    a.Bpad = (int)round_up(B, 256);
    a.nBT = a.Bpad / 256;
    a.nCT = (int)(round_up(C_shard, 256) / 256);
    LogitsPlan p = plan_logits(B, D, C_shard, SMALL_TOP1);
    if (workspace_bytes < p.bytes()) p = plan_wide(B, C_shard);
    float* part_val = static_cast<float*>(workspace);
    int* part_cls = reinterpret_cast<int*>(part_val + p.parts * p.pitch);
    const int parts = (int)p.parts, pitch = (int)p.pitch;
    hipStream_t s = static_cast<hipStream_t>(stream);
    set_step_order(a);
    if (p.way == WAY_SMALL) {
        const SmallPlan sp(B, C_shard);
        WS_LAUNCH_SMALL(KID_TOP1, top1_small, sp, sp.ranges, s, a, sp.range, part_val, part_cls);
    } else if (p.way == WAY_BLOCKS) {
        WS_LAUNCH(KID_TOP1, top1_block, dim3(xcd_grid(parts * (pitch / BLOCK))), dim3(NTHREADS), s, a, pitch, part_val, part_cls);
    } else {
        WS_LAUNCH(KID_TOP1, top1_logits, dim3(xcd_grid(a.nBT * a.nCT)), dim3(NTHREADS), s, a, part_val, part_cls);
    }
    launch_merge_top1(part_val, part_cls, parts, pitch, B, class_offset, top_logit, top_class, s);
    return launch_status();
}

int ws_combine_top1(const float* top_logit, const int32_t* top_class, int32_t S, int32_t B, int64_t shard_stride,
                    float* best_logit, int32_t* best_class, void* stream) {
    if (!top_logit || !top_class || !best_logit || !best_class) return WS_ERR_NULL;
    if (B <= 0 || shard_stride < B) return WS_ERR_SHAPE;
    if (S < 1 || S > 65536) return WS_ERR_RANGE;
    if (!aligned(top_logit, 4) || !aligned(top_class, 4) || !aligned(best_logit, 4) || !aligned(best_class, 4))
        return WS_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    launch_merge_top1(top_logit, top_class, S, shard_stride, B, 0, best_logit, best_class, s);
    return launch_status();
}

static void profile_free_pool() {
    for (int i = 0; i < g_prof.capacity; ++i) {
        (void)hipEventDestroy(g_prof.start[i]);
        (void)hipEventDestroy(g_prof.stop[i]);
    }
    delete[] g_prof.start; delete[] g_prof.stop; delete[] g_prof.kid;
    g_prof = ProfState();
}

int ws_profile_enable(int32_t max_launches) {
    if (g_prof.start) profile_free_pool();
    if (max_launches <= 0) return WS_OK;
    g_prof.start = new hipEvent_t[max_launches];
    g_prof.stop = new hipEvent_t[max_launches];
    g_prof.kid = new int[max_launches];
    for (int i = 0; i < max_launches; ++i) {
        if (hipEventCreate(&g_prof.start[i]) != hipSuccess) {
            profile_free_pool();                      // the pairs created so far; timing stays off
            return WS_ERR_HIP;
        }
        if (hipEventCreate(&g_prof.stop[i]) != hipSuccess) {
            (void)hipEventDestroy(g_prof.start[i]);
            profile_free_pool();
            return WS_ERR_HIP;
        }
        g_prof.capacity = i + 1;
    }
    g_prof.on = true;
    return WS_OK;
}

int ws_profile_reset(void) {
    g_prof.used = 0;
    return WS_OK;
}

int ws_profile_pause(int32_t paused) {
    g_prof.paused = paused != 0;
    return WS_OK;
}

int ws_profile_trace_dw(void* device_trace, int64_t tiles) {
    if (device_trace == nullptr) {
        g_dw_trace = nullptr;
        g_dw_trace_tiles = 0;
        return WS_OK;
    }
    if (tiles <= 0) return WS_ERR_SHAPE;
    if (!aligned(device_trace, 8)) return WS_ERR_ALIGN;
    g_dw_trace = static_cast<unsigned long long*>(device_trace);
    g_dw_trace_tiles = tiles;
    return WS_OK;
}

int32_t ws_profile_kernel_count(void) { return KID_COUNT; }

const char* ws_profile_kernel_name(int32_t kernel) {
    return (kernel >= 0 && kernel < KID_COUNT) ? kKernelNames[kernel] : "";
}

int ws_profile_read(int32_t kernel, double* total_ms, int64_t* launches) {
    if (!total_ms || !launches) return WS_ERR_NULL;
    if (kernel < 0 || kernel >= KID_COUNT) return WS_ERR_RANGE;
    double tot = 0.0;
    int64_t n = 0;
    for (int i = 0; i < g_prof.used; ++i) {
        if (g_prof.kid[i] != kernel) continue;
        if (hipEventSynchronize(g_prof.stop[i]) != hipSuccess) return WS_ERR_HIP;
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, g_prof.start[i], g_prof.stop[i]) != hipSuccess) return WS_ERR_HIP;
        tot += ms;
        ++n;
    }
    *total_ms = tot;
    *launches = n;
    return WS_OK;
}

}  // extern "C"
