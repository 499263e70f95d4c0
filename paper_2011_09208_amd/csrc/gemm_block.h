// GEMM of small output tiles: 64 (M) x 64 (N), A k-contiguous, B k-strided.
//
// A 256 x 256 tile (gemm_core.h) takes a compute unit 2048 matrix cycles per k-step; an output of a few dozen of them leaves
// the rest of the chip idle for the length of the contraction.  A 64 x 64 tile moves four times the operand bytes per
// flop and is bound by the 64 B/clk of the path into LDS (16 KiB per k-step: 256 cycles against 128 of the matrix
// cores), but there are sixteen times as many.  Eight waves: 2 x 2 quarters of the tile (32 x 32) x the two halves of a k-step, whose
// sums meet in LDS at the end.  Five 16 KiB stages, loaded four k-steps ahead, one barrier per k-step; 80 KiB, so that a second
// workgroup on the compute unit computes while this one waits.
#pragma once
#include "gemm_core.h"

namespace ws {

constexpr int BLOCK = 64;
constexpr int BLOCK_OPERAND_BYTES = BLOCK * TILE_K * 2;          // 8 KiB
constexpr int BLOCK_STAGE_BYTES = 2 * BLOCK_OPERAND_BYTES;
constexpr int BLOCK_STAGES = 5;
constexpr int BLOCK_LDS_BYTES = BLOCK_STAGES * BLOCK_STAGE_BYTES;

typedef f32x4 block_acc_t[2][2];

// Sums over k in [k_begin, k_begin + 64 * k_steps) of A(m, k) * B(k, n): waves 0 .. 3 end with quarter (pm, pn) = (wave % 2, wave
// / 2) of the tile, acc[x][y] M tile x and N tile y of it.  All 512 threads call it together.
__device__ __forceinline__ void block_gemm(block_acc_t& acc, const Operand& A, const Operand& Bop, int m0, int n0, int k_begin,
                                           int k_steps, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int pm = wave & 1, pn = (wave >> 1) & 1, half = wave >> 2;
    const int last = k_steps - 1;
    // wave w loads rows 8 w .. + 7 of A and k-rows 8 w .. + 7 of B: one load of 1 KiB each, swizzled as in thin_mainloop
    const int row = 8 * wave + (lane >> 3);
    const uint32_t a_lane = ((uint32_t)(m0 + row) * A.ld + (uint32_t)(8 * ((lane & 7) ^ ((row >> 1) & 7)))) * 2u;
    const uint32_t b_lane = ((uint32_t)row * Bop.ld + (uint32_t)(n0 + 8 * ((lane & 7) ^ thin_ks_swizzle(row)))) * 2u;
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;
    auto load = [&](int step, int stage) {
        const uint32_t k = (uint32_t)(k_begin + step * TILE_K);
        load_to_lds(A, a_lane, 2u * k, lds_wave + (uint32_t)stage);
        load_to_lds(Bop, b_lane, 2u * k * Bop.ld, lds_wave + (uint32_t)stage + BLOCK_OPERAND_BYTES);
    };
    const int a_frag = (32 * pm + i) * 128 + (((4 * half + g) ^ (i >> 1)) << 4);
    int b_frag[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int krow = 8 * g + (i >> 2), col = 32 * pn + 16 * t + 4 * (i & 3);
        b_frag[t] = BLOCK_OPERAND_BYTES + (32 * half + krow) * 128 + (((col >> 3) ^ thin_ks_swizzle(krow)) << 4) + ((col & 7) << 1);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < BLOCK_STAGES - 1 && j <= last; ++j) load(j, j * BLOCK_STAGE_BYTES);
    int cur = 0, nxt = (BLOCK_STAGES - 1) * BLOCK_STAGE_BYTES;        // stages of k-steps j and j + 4
    for (int j = 0; j <= last; ++j) {
        // k-steps j + 1 .. j + 3 may still be on their way
        if (j + 3 <= last) wait_counts<6, NO_LG_WAIT>();
        else if (j + 2 <= last) wait_counts<4, NO_LG_WAIT>();
        else if (j + 1 <= last) wait_counts<2, NO_LG_WAIT>();
        else wait_counts<0, NO_LG_WAIT>();
        raw_barrier();                                   // every wave has read k-step j - 1, whose stage is refilled
        if (j + BLOCK_STAGES - 1 <= last) load(j + BLOCK_STAGES - 1, nxt);
        bf16x8 af[2], bf[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            af[t] = *reinterpret_cast<const bf16x8*>(lds + (a_frag + cur) + t * 2048);
            typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
            const char* p = lds + (b_frag[t] + cur);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * 128));
            bf[t] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[x], bf[y], acc[x][y], 0, 0, 0);
        cur += BLOCK_STAGE_BYTES;
        if (cur == BLOCK_LDS_BYTES) cur = 0;
        nxt += BLOCK_STAGE_BYTES;
        if (nxt == BLOCK_LDS_BYTES) nxt = 0;
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    f32x4* other = reinterpret_cast<f32x4*>(lds) + (wave & 3) * 256 + lane;        // [quarter][x, y][lane]
    if (half == 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) other[64 * q] = acc[q >> 1][q & 1];
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    if (half == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q >> 1][q & 1] += other[64 * q];
    }
}
constexpr int BLOCK_TILE_OFFSET = 4 * 4096;             // LDS behind the sums of the second half

// The tile as bf16 [n][m]: 16-byte chunk tid % 8 (elements 8 * (tid % 8) ..) of row tid / 8.  It passes through LDS, 128 bytes per
// n, 8-byte slots XOR-ed with n & 15.
__device__ __forceinline__ u32x4 block_rows_bf16(const block_acc_t& acc, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
    char* tile = lds + BLOCK_TILE_OFFSET;
    if (wave < 4) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const f32x4 v = acc[x][y];
                const int n = 32 * (wave >> 1) + 16 * y + i, slot = (32 * (wave & 1) + 16 * x + 4 * g) >> 2;
                *reinterpret_cast<u32x2*>(tile + n * 128 + ((slot ^ (n & 15)) << 3)) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    const int n = tid >> 3, c = tid & 7;                 // chunk c is slots 2 c and 2 c + 1, side by side, swapped when n is odd
    u32x4 v = *reinterpret_cast<const u32x4*>(tile + n * 128 + ((c ^ ((n & 15) >> 1)) << 4));
    return n & 1 ? __builtin_shufflevector(v, v, 2, 3, 0, 1) : v;
}

// The tile as fp32 [m][n]: out[half] is elements 4 * (tid % 16) .. + 3 of row 32 * half + tid / 16.  256 bytes per m in LDS, 16-float
// chunks XOR-ed with (m >> 2) & 3, which spreads the four row groups of a wave's store over the banks.
__device__ __forceinline__ void block_rows_f32(f32x4 (&out)[2], const block_acc_t& acc, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
    float* tile = reinterpret_cast<float*>(lds + BLOCK_TILE_OFFSET);
    if (wave < 4) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v)              // row m = .. + 4 g + v: (m >> 2) & 3 = g
                    tile[(32 * (wave & 1) + 16 * x + 4 * g + v) * 64 + 16 * ((2 * (wave >> 1) + y) ^ g) + i] = acc[x][y][v];
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int m = 32 * h + (tid >> 4), c = tid & 15;
        out[h] = *reinterpret_cast<const f32x4*>(tile + m * 64 + 16 * ((c >> 2) ^ ((m >> 2) & 3)) + 4 * (c & 3));
    }
}

// ---- logits ---------------------------------------------------------------------------------------------
// 64 classes (M, rows of A) x 64 batch rows (N, rows of B), both k-contiguous.  Eight waves: 2 (M) x 4 (N), each 32 classes x 16
// rows and the whole contraction, so that a logit's products are added in the order of the wide tiles.
typedef f32x4 block_logits_t[2];

// acc[x][v] is class 32 * wm + 16 * x + 4 * g + v of row 16 * wn + i of the tile (wave 4 * wm + wn, lane 16 * g + i).  All 512
// threads call it together; ends with a workgroup barrier.
__device__ __forceinline__ void block_logits(block_logits_t& acc, const Operand& A, const Operand& Bop, int m0, int n0, int k_steps,
                                             char* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3, i = lane & 15, g = lane >> 4;
    const int last = k_steps - 1;
    // wave w loads rows 8 w .. + 7 of either operand: one load of 1 KiB each
    const int row = 8 * wave + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    const uint32_t a_lane = ((uint32_t)(m0 + row) * A.ld + (uint32_t)(8 * chunk)) * 2u;
    const uint32_t b_lane = ((uint32_t)(n0 + row) * Bop.ld + (uint32_t)(8 * chunk)) * 2u;
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;
    auto load = [&](int step, int stage) {
        load_to_lds(A, a_lane, (uint32_t)step * 128u, lds_wave + (uint32_t)stage);
        load_to_lds(Bop, b_lane, (uint32_t)step * 128u, lds_wave + (uint32_t)stage + BLOCK_OPERAND_BYTES);
    };
    int a_frag[2], b_frag[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int at = i * 128 + (((4 * s + g) ^ (i >> 1)) << 4);
        a_frag[s] = 32 * wm * 128 + at;
        b_frag[s] = BLOCK_OPERAND_BYTES + 16 * wn * 128 + at;
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < BLOCK_STAGES - 1 && j <= last; ++j) load(j, j * BLOCK_STAGE_BYTES);
    int cur = 0, nxt = (BLOCK_STAGES - 1) * BLOCK_STAGE_BYTES;        // stages of k-steps j and j + 4
    for (int j = 0; j <= last; ++j) {
        // k-steps j + 1 .. j + 3 may still be on their way
        if (j + 3 <= last) wait_counts<6, NO_LG_WAIT>();
        else if (j + 2 <= last) wait_counts<4, NO_LG_WAIT>();
        else if (j + 1 <= last) wait_counts<2, NO_LG_WAIT>();
        else wait_counts<0, NO_LG_WAIT>();
        raw_barrier();                                   // every wave has read k-step j - 1, whose stage is refilled
        if (j + BLOCK_STAGES - 1 <= last) load(j + BLOCK_STAGES - 1, nxt);
        bf16x8 af[2][2], bf[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf[s] = *reinterpret_cast<const bf16x8*>(lds + (b_frag[s] + cur));
#pragma unroll
            for (int x = 0; x < 2; ++x) af[x][s] = *reinterpret_cast<const bf16x8*>(lds + (a_frag[s] + cur) + x * 2048);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[x][s], bf[s], acc[x], 0, 0, 0);
        cur += BLOCK_STAGE_BYTES;
        if (cur == BLOCK_LDS_BYTES) cur = 0;
        nxt += BLOCK_STAGE_BYTES;
        if (nxt == BLOCK_LDS_BYTES) nxt = 0;
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
}

// The tile as bf16 [row][class]: 16-byte chunk tid % 8 of row tid / 8.  Through LDS as in block_rows_bf16.
__device__ __forceinline__ u32x4 block_logits_rows(const block_logits_t& acc, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int n = 16 * (wave & 3) + i, slot = (32 * (wave >> 2) + 16 * x + 4 * g) >> 2;
        *reinterpret_cast<u32x2*>(lds + n * 128 + ((slot ^ (n & 15)) << 3)) = u32x2{pack_bf16(acc[x][0], acc[x][1]), pack_bf16(acc[x][2], acc[x][3])};
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    const int n = tid >> 3, c = tid & 7;
    u32x4 v = *reinterpret_cast<const u32x4*>(lds + n * 128 + ((c ^ ((n & 15) >> 1)) << 4));
    return n & 1 ? __builtin_shufflevector(v, v, 2, 3, 0, 1) : v;
}

}  // namespace ws
