// GEMM of small output tiles: 64 (M) x 64 (N), A k-contiguous, B k-strided, bf16 out.
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

// Returns 16-byte chunk tid % 8 (elements m0 + 8 * (tid % 8) ..) of row n0 + tid / 8 of the tile as bf16 out[n][m]: sums over
// k < 64 * k_steps of A(m, k) * B(k, n).  All 512 threads call it together.
__device__ __forceinline__ u32x4 block_gemm(const Operand& A, const Operand& Bop, int m0, int n0, int k_steps, char* lds) {
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
        load_to_lds(A, a_lane, (uint32_t)step * 128u, lds_wave + (uint32_t)stage);
        load_to_lds(Bop, b_lane, (uint32_t)step * 128u * Bop.ld, lds_wave + (uint32_t)stage + BLOCK_OPERAND_BYTES);
    };
    const int a_frag = (32 * pm + i) * 128 + (((4 * half + g) ^ (i >> 1)) << 4);
    int b_frag[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int krow = 8 * g + (i >> 2), col = 32 * pn + 16 * t + 4 * (i & 3);
        b_frag[t] = BLOCK_OPERAND_BYTES + (32 * half + krow) * 128 + (((col >> 3) ^ thin_ks_swizzle(krow)) << 4) + ((col & 7) << 1);
    }
    f32x4 acc[2][2];
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
    // the second half's sums as [quarter][x, y][lane], then the tile as [n][m], 128 bytes per n, 8-byte slots XOR-ed with n & 15
    f32x4* other = reinterpret_cast<f32x4*>(lds) + (wave & 3) * 256 + lane;
    if (half == 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) other[64 * q] = acc[q >> 1][q & 1];
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    char* tile = lds + 4 * 4096;
    if (half == 0) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const f32x4 v = acc[x][y] + other[64 * (2 * x + y)];
                const int n = 32 * pn + 16 * y + i, slot = (32 * pm + 16 * x + 4 * g) >> 2;
                *reinterpret_cast<u32x2*>(tile + n * 128 + ((slot ^ (n & 15)) << 3)) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    const int n = tid >> 3, c = tid & 7;                 // chunk c is slots 2 c and 2 c + 1, side by side, swapped when n is odd
    u32x4 v = *reinterpret_cast<const u32x4*>(tile + n * 128 + ((c ^ ((n & 15) >> 1)) << 4));
    return n & 1 ? __builtin_shufflevector(v, v, 2, 3, 0, 1) : v;
}

}  // namespace ws
