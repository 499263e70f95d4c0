// Logits of small batches (up to 32 rows, up to 2048 features), bound by reading W once.
//
// A 256-row tile (gemm_core.h) computes 256 rows whatever the batch, and 256 classes per workgroup leave most of the
// chip idle on a narrow shard.  Here the classes are dealt out evenly, one range per compute unit, walked 32 classes at
// a time.  The waves of a workgroup share out the contraction (wave w the k-steps w, w + WAVES, ..) and keep their part of
// X in registers for the whole range, so that the loop reads nothing but W: 128 KiB per 32 classes at 2048 features, all
// of it in flight while the waves' partial sums of the 32 classes before meet in LDS.  One barrier per 32 classes.
// (With X read again for every 32 or 64 classes, W of 100 000 x 2048: 76 us for 16 rows, 113 for 32.)
#pragma once
#include "gemm_core.h"

namespace ws {

constexpr int SMALL_MAX_ROWS = 32;
constexpr int SMALL_MAX_STEPS = 32;          // k-steps of X that the registers of a workgroup hold
constexpr int SMALL_C = 32;                  // classes at a time
constexpr int SMALL_WAVES = 8, SMALL_THREADS = 64 * SMALL_WAVES;
constexpr int SMALL_PITCH = SMALL_C + 4;     // floats per row of a partial sum

// NB = 16-row blocks of the batch (1 or 2).  The finished logits are dealt out CPT classes of one row per thread,
// the TPR threads of a row side by side in one wave.
template <int NB> struct SmallShape {
    static constexpr int ROWS = 16 * NB;
    static constexpr int STEPS = SMALL_MAX_STEPS / SMALL_WAVES;  // k-steps per wave
    static constexpr int CPT = SMALL_C * ROWS / SMALL_THREADS;   // classes per thread: 1 or 2
    static constexpr int TPR = SMALL_C / CPT;                // threads per row: 32 or 16
    static constexpr int SLOT_FLOATS = ROWS * SMALL_PITCH;
    static constexpr int LDS_FLOATS = 2 * SMALL_WAVES * SLOT_FLOATS;
};
constexpr int SMALL_MAX_RANGES = 256;        // one per compute unit

// Calls body(c, z): z[e] = W[c + e] . X[tid / TPR] + bias[c + e] (-inf beyond C), c = c_begin + 32 n + CPT * (tid % TPR), for
// all n with c_begin + 32 n < c_end; c + e may lie beyond c_end.  All threads call it together.
template <int NB, class Body>
__device__ __forceinline__ void small_logits(const uint16_t* X, int64_t ldx, int B, const uint16_t* W, int64_t ldw, int C, int D,
                                             const float* bias, int c_begin, int c_end, float* lds, Body body) {
    typedef SmallShape<NB> S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int k_steps = D / TILE_K;
    // rows beyond the batch and classes beyond the range or the shard read as zeros (bounds check of the resource)
    const int c_read = c_end < C ? c_end : C;
    const int64_t w_bytes = c_read > c_begin ? (((int64_t)c_read - 1) * ldw + D) * 2 : 0;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(W), 0, (int)(uint32_t)w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(X), 0, (int)(uint32_t)((((int64_t)B - 1) * ldx + D) * 2), 0x00020000);
    // all in the per-lane offset, one register
    const uint32_t a_lane = ((uint32_t)i * (uint32_t)ldw + 8u * g) * 2u + 128u * (uint32_t)wave;
    const uint32_t b_lane = ((uint32_t)i * (uint32_t)ldx + 8u * g) * 2u + 128u * (uint32_t)wave;
    const int c_mine = S::CPT * (tid % S::TPR);

    u32x4 a[S::STEPS][2][2], x[S::STEPS][NB][2];
    float bias_next[S::CPT];
    auto load = [&](int c0) {
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) {                   // before the loads of W: they return in order
            const int c = c0 + c_mine + e;
            bias_next[e] = bias != nullptr && c < C ? bias[c] : 0.0f;
        }
        const uint32_t row = a_lane + (uint32_t)c0 * (uint32_t)ldw * 2u;
#pragma unroll
        for (int n = 0; n < S::STEPS; ++n)
            if (wave + n * SMALL_WAVES < k_steps) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        a[n][t][s] = __builtin_amdgcn_raw_buffer_load_b128(
                            ra, (int)(row + 32u * t * (uint32_t)ldw + (uint32_t)(128 * n * SMALL_WAVES + 64 * s)), 0, 0);
            }
    };
    load(c_begin);
#pragma unroll
    for (int n = 0; n < S::STEPS; ++n)
        if (wave + n * SMALL_WAVES < k_steps) {
#pragma unroll
            for (int r = 0; r < NB; ++r)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    x[n][r][s] = __builtin_amdgcn_raw_buffer_load_b128(
                        rb, (int)(b_lane + 32u * r * (uint32_t)ldx + (uint32_t)(128 * n * SMALL_WAVES + 64 * s)), 0, 0);
        }
    float* slots = lds;                                      // this tile's partial sums; the next one uses the other half
    float* other = lds + SMALL_WAVES * S::SLOT_FLOATS;
    for (int c0 = c_begin; c0 < c_end; c0 += SMALL_C) {
        f32x4 acc[2][NB];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < NB; ++r) acc[t][r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < S::STEPS; ++n)
            if (wave + n * SMALL_WAVES < k_steps) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < NB; ++r)
                            acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[n][t][s]),
                                                                                __builtin_bit_cast(bf16x8, x[n][r][s]), acc[t][r], 0, 0, 0);
            }
        float bias_now[S::CPT];
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) bias_now[e] = bias_next[e];
        __builtin_amdgcn_sched_barrier(0);
        if (c0 + SMALL_C < c_end) load(c0 + SMALL_C);
        __builtin_amdgcn_sched_barrier(0);
        // partial sums as [row][class]: a lane holds four adjacent classes of a row
        float* p = slots + wave * S::SLOT_FLOATS + i * SMALL_PITCH + 4 * g;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < NB; ++r) *reinterpret_cast<f32x4*>(p + 16 * r * SMALL_PITCH + 16 * t) = acc[t][r];
        wait_counts<NO_VM_WAIT, 0>();
        raw_barrier();                                       // the loads stay in flight
        // A wave writes these slots again two tiles on, behind the next tile's barrier, which every wave passes
        // after it has read them.
        const float* mine = slots + (tid / S::TPR) * SMALL_PITCH + c_mine;
        float z[S::CPT];
#pragma unroll
        for (int e = 0; e < S::CPT; ++e) {
            z[e] = mine[e];
#pragma unroll
            for (int w = 1; w < SMALL_WAVES; ++w) z[e] += mine[w * S::SLOT_FLOATS + e];
            z[e] = c0 + c_mine + e < C ? z[e] + bias_now[e] : -INFINITY;
        }
        body(c0 + c_mine, z);
        float* swap = slots;
        slots = other;
        other = swap;
    }
}

}  // namespace ws
