// Shared bf16 MFMA GEMM main loop for gfx950 (MI355X), used by all four contractions
// of the split fully-connected head.
//
// One workgroup of 512 threads (8 wave64s, two per SIMD) owns a 256 x 256 output tile
// and walks the contraction in steps of 64.  The waves form a 2 (M) x 4 (N) grid; each
// owns a 128 x 64 sub-tile held as 8 x 4 accumulators of v_mfma_f32_16x16x32_bf16 (measured
// about 7 % faster than the 32x32x16 form under the chip's power limit: it moves half as many
// accumulator registers per flop).
//
// Tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds).  Such a load writes 64 x 16
// consecutive bytes of LDS, so a layout's swizzle is applied to the global address each lane reads.  The layout of
// an operand tile depends on how the operand lies in memory relative to the contraction index k:
//   KC ("k contiguous"): memory is [row][k]; LDS holds rows of 64 k (128 B), 16-byte chunks XOR-swizzled by
//       (row >> 1) & 7; a lane's MFMA fragment (8 consecutive k of one row) is one ds_read_b128.
//   KS ("k strided"):    memory is [k][col]; LDS holds k-rows, 16-byte chunks XOR-swizzled by a function of k
//       (ks_swizzle); the fragment is gathered with two ds_read_b64_tr_b16 transpose reads (4 consecutive k of
//       one column each).
// Lane layouts used (checked on the hardware): for v_mfma_f32_16x16x32_bf16 lane l
// supplies row l % 16, k = 8 * (l / 16) .. + 7 of either operand; accumulator register v
// of lane l is element (4 * (l / 16) + v, l % 16).  ds_read_b64_tr_b16
// works on blocks of 16 lanes: lane i of a block receives, as element e, the (i % 4)-th
// 16-bit value of the 8 bytes addressed by lane 4 * e + i / 4 of the same block.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace ws {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr int TILE_M = 256;
constexpr int TILE_N = 256;
constexpr int TILE_K = 64;
constexpr int NTHREADS = 512;
constexpr int WAVE_M = 128;     // rows of the output tile one wave owns
constexpr int WAVE_N = 64;
constexpr int MT = WAVE_M / 16; // 16 x 16 MFMA tiles per wave along M: 8
constexpr int NT = WAVE_N / 16; // and along N: 4
constexpr int HALF_TILE_BYTES = 128 * TILE_K * 2;              // half of an operand tile: 16 KiB
constexpr int OPERAND_TILE_BYTES = 2 * HALF_TILE_BYTES;        // 32 KiB
constexpr int STAGE_BYTES = 2 * OPERAND_TILE_BYTES;            // A + B
constexpr int LDS_BYTES = 2 * STAGE_BYTES;                     // double buffered: 128 KiB

enum { KC = 0, KS = 1 };

// One GEMM operand in global memory (16-bit elements), addressed through a buffer resource:
//   KC: element (row, k) at base[row * ld + k];   KS: element (k, col) at base[k * ld + col].
// A load has a scalar resource, a scalar offset (the k-step and the part of the tile) and ONE 32-bit per-lane
// offset per operand that never changes inside the main loop.
// The resource covers exactly rows x cols of the matrix: a tile may hang over its end (ragged row or
// class counts, the last k-step of a contraction) and the overhang reads as zeros, as the hardware
// bounds check returns 0 beyond the resource.  Offsets are 32-bit: (rows + 256) * ld * 2 bytes must stay
// below 4 GiB (checked on the host).
// The rule of that check, for loads and stores: an access is in range if lane offset + scalar offset lies within the
// records, as a sum that does not wrap; with a scalar offset alone beyond the records, or no records, nothing is in range.
// (Measured on 324 combinations of records, lane and scalar offsets inside one allocation, loads and stores.)  The
// tests that fail if it were not so: a batch of fewer than 32 rows in dW, whose second 32 rows of dz start beyond the
// records, in a workspace of NaNs (test_gpu_small.py); the dW stream with D = 320 and 576, where the stores of the last
// feature tile's missing quadrants have no records and would land in the next row (test_gpu_stream.py, test_gpu_guards.py).
struct Operand {
    u32x4 rsrc;
    uint32_t ld;        // row pitch in elements
};

// `rows` x `cols` elements are valid (KC: rows x k extent; KS: k extent x columns).
__device__ __forceinline__ Operand make_operand(const uint16_t* base, int64_t ld, int64_t rows, int64_t cols) {
    const int64_t bytes = ((rows - 1) * ld + cols) * 2;
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    Operand op;
    op.rsrc = u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xffffu, (uint32_t)bytes, 0x00020000u};
    op.ld = (uint32_t)ld;
    return op;
}

// ---- global -> LDS ------------------------------------------------------------------------------
// 16 bytes per lane from `voff` (per lane) + `soff` (uniform) of the operand to LDS byte lds_off + 16 * lane.
// Inline assembly, because for the builtin the compiler makes every later LDS read wait for ALL loads in flight;
// here the main loop counts them itself (wait_counts).  The load is complete in LDS when vmcnt says so.
__device__ __forceinline__ void load_to_lds(const Operand& op, uint32_t voff, uint32_t soff, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_off), "v"(voff), "s"(op.rsrc), "s"(soff) : "memory");
}

// Brings a line into the L2: 4 bytes per lane, to LDS byte lds_off + 4 * lane, where nobody reads them.  To LDS because a
// load in inline assembly may not have a register for its result: the compiler takes an output as written at once, and
// moves other values into its register while the load is still on its way.
__device__ __forceinline__ void touch_line(const Operand& op, uint32_t voff, uint32_t soff, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds_off), "v"(voff), "s"(op.rsrc), "s"(soff) : "memory");
}

// LDS byte offset of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_offset(const char* lds) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds;
}

// Waits until at most VM vector-memory operations and LG LDS operations of this wave are outstanding.
template <int VM, int LG>
__device__ __forceinline__ void wait_counts() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70 | (LG << 8));
    __builtin_amdgcn_sched_barrier(0);
}
constexpr int NO_VM_WAIT = 63, NO_LG_WAIT = 15;

// Workgroup barrier that orders nothing by itself (no implied waits): the caller has waited for what it needs.
__device__ __forceinline__ void raw_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Chunk swizzle of a KS tile.  A transposing read is served half a wave at a time; the 32 lanes of a
// half cover 4 k-rows (k & 3) in each of 2 lane blocks 8 k-rows apart ((k >> 3) & 1), two adjacent
// chunks and both 8-byte halves of a chunk each.  Those 16 (k-row, chunk) pairs must fall into 16
// different chunks modulo 16 (256 bytes span all banks, a k-row is 256 bytes): k & 3 goes to chunk bits 2-3,
// (k >> 3) & 1 to bit 1, the two adjacent chunks differ in bit 0.  Bits 2 and 5 of k are left out so that the
// reads 4 and 32 k-rows further on keep the same pattern.
__device__ __forceinline__ int ks_swizzle(int k) { return (((k >> 3) & 1) << 1) | ((k & 3) << 2); }

// ---- main loop ---------------------------------------------------------------------------------

// acc[mt][nt] += A(m0 .. m0+255, k) * B(n0 .. n0+255, k) for k in [k_begin, k_begin + 64 * k_steps).
// A is KC, m0 its first row; for a KC operand B n0 is its first row, for a KS one its first column.
// A wave's M tiles are rows WAVE_M * wm + 16 * mt of the tile, its N tiles columns wave_col<BKIND>(wn, nt).
// Ends with a workgroup barrier, so LDS may be reused by the caller right away.
//
// Ping-pong between the two waves of a SIMD.  Waves 0-3 (M half 0) and 4-7 (M half 1) sit on the four SIMDs in
// pairs.  A k-step is four phases, one per quadrant of the wave's 128 x 64 sub-tile (A half x B half, 16 MFMAs
// each, both k-substeps); a phase is a LOAD slot (LDS fragments for its MFMAs, global -> LDS loads for a later
// k-step, waits) and an MFMA slot, with a workgroup barrier after each.  The second half of the waves runs one
// slot behind, so that in every slot one wave of a SIMD feeds the matrix core while the other one reads LDS and
// issues loads: neither competes with the other for issue slots, and every wait is covered by the partner's
// 256 MFMA cycles.
//
// LDS holds two stages (k-step j in stage j & 1) of four 16 KiB half tiles (A0 A1 B0 B1; half h of A holds the 64
// rows of the h-th half of each wave row, and likewise for the columns of B).  Each phase reads one half tile
// and the phase after it refills that half tile with k-step j + 2:
//   phase   MFMAs      reads          loads (2 per wave)
//     0     A0 x B0    A0(j)          B0(j + 2)
//     1     A0 x B1    B1(j)          A0(j + 2)
//     2     A1 x B0    A1(j)          B1(j + 2)
//     3     A1 x B1    B0(j + 1)      A1(j + 2)
// A wave's reads of phase p are complete (lgkmcnt 0) before the barrier that ends its LOAD slot; the refill is
// issued after a later barrier than that of either half of the waves.  Every half tile is read seven phases after
// its loads were issued: at the end of a LOAD slot, what the next phase reads has landed when at most the
// 6 phases x 2 loads issued since are outstanding (vmcnt 12), so a load has more than 3000 cycles to arrive.
//
// Measured (4096 x 4096 x 8192, normal random operands, against the loop that went through registers and left the
// interleaving of the two waves to the hardware): KC 1335 -> 1497, KS 1285 -> 1442 TFLOP/s; all ones 1866 ->
// 2140.  Two phases of 32 MFMAs: 1467; raising the wave priority (s_setprio) in the MFMA slots: 1486.
typedef f32x4 acc_t[MT][NT];

// First column of N tile nt of wave column wn in the 256-wide tile.  The B half tiles are chosen so that their
// global loads are whole lines: a KS half tile is 128 adjacent columns.
template <int BKIND>
__device__ __forceinline__ int wave_col(int wn, int nt) {
    return BKIND == KC ? WAVE_N * wn + 16 * nt : 128 * (nt >> 1) + 32 * wn + 16 * (nt & 1);
}

// LDS -> fragments: af[tile of the half][k-substep], bf the same for half a B.  LEAN keeps one offset per operand: chunk
// numbers are XOR-ed with the swizzle, so the second k-substep (KC, chunk bit 2) and the second 16-wide tile (KS, bit 1)
// are an XOR away.  For a loop that has no register left: two variants of the tile stream spilled 1 and 6 without it; the
// others lose 1 % by its two instructions a phase.
template <int BKIND, bool LEAN = false>
struct FragReader {
    int a_frag[2], b_frag[2];
    __device__ __forceinline__ FragReader(int wm, int wn, int i, int g) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int chunk = (4 * s + g) ^ (i >> 1);
            a_frag[s] = (64 * wm + i) * 128 + 16 * chunk;
            if (BKIND == KC) {
                b_frag[s] = OPERAND_TILE_BYTES + (32 * wn + i) * 128 + 16 * chunk;
            } else {                                       // s counts the two 16-wide tiles here
                const int krow = 8 * g + (i >> 2), col = 32 * wn + 16 * s + 4 * (i & 3);
                b_frag[s] = OPERAND_TILE_BYTES + krow * 256 + (((col >> 3) ^ ks_swizzle(krow)) << 4) + ((col & 7) << 1);
            }
        }
    }
    // Both offsets of an operand; `bit` is where they differ.  The empty assembly keeps the compiler from holding the
    // second one between calls all the same.
    static __device__ __forceinline__ void offsets(int (&o)[2], const int (&f)[2], int bit) {
        o[0] = f[0];
        if (LEAN) asm volatile("" : "+v"(o[0]));
        o[1] = LEAN ? o[0] ^ bit : f[1];
    }
    template <int UNITS = MT / 4>                          // the first 2 * UNITS tiles of the half
    __device__ __forceinline__ void read_a(bf16x8 (&af)[MT / 2][2], const char* lds, int half, int stage) const {
        int o[2];
        offsets(o, a_frag, 64);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < 2 * UNITS; ++t)
                af[t][s] = *reinterpret_cast<const bf16x8*>(lds + (o[s] + stage) + half * HALF_TILE_BYTES + t * 2048);
    }
    __device__ __forceinline__ void read_b(bf16x8 (&bf)[NT / 2][2], const char* lds, int half, int stage) const {
        int o[2];
        offsets(o, b_frag, BKIND == KC ? 64 : 32);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < NT / 2; ++t) {
                if (BKIND == KC) {
                    bf[t][s] = *reinterpret_cast<const bf16x8*>(lds + (o[s] + stage) + half * HALF_TILE_BYTES + t * 2048);
                } else {
                    typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
                    const char* p = lds + (o[t] + stage) + half * HALF_TILE_BYTES + s * (32 * 256);
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * 256));
                    bf[t][s] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
    }
};

// The 16 MFMAs of quadrant Q = 2 * (A half) + (B half).  FIRST: the accumulators start from zero.
template <int Q, bool FIRST = false>
__device__ __forceinline__ void quadrant_mfmas(acc_t& acc, const bf16x8 (&af)[MT / 2][2], const bf16x8 (&bf)[NT / 2][2]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int x = 0; x < MT / 2; ++x)
#pragma unroll
            for (int y = 0; y < NT / 2; ++y) {
                f32x4& c = acc[MT / 2 * (Q >> 1) + x][NT / 2 * (Q & 1) + y];
                const f32x4 from = FIRST && s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : c;
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[x][s], bf[y][s], from, 0, 0, 0);
            }
    __builtin_amdgcn_sched_barrier(0);
}

// `descending` (uniform over the workgroup): walk the k-steps from the last to the first.  Tiles that follow each
// other on a compute unit and share an operand panel can alternate the direction, so that the second finds
// the end of the panel, which the first has just read, still in the L2.
template <int BKIND>
__device__ __forceinline__ void gemm_mainloop(acc_t& acc, const Operand& A, const Operand& Bop,
                                              int m0, int n0, int k_begin, int k_steps, char* lds,
                                              bool descending = false) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int i = lane & 15, g = lane >> 4;
    const int last = k_steps - 1;
    const int k_first = descending ? k_begin + last * TILE_K : k_begin;
    const int k_stride = descending ? -TILE_K : TILE_K;

    // Global -> LDS.  A half tile is 16 loads of 1 KiB; wave w issues loads w and w + 8.
    //   KC: a load is 8 rows of 128 bytes; LDS rows 8 w .. + 7 and 64 + 8 w .. + 7 of the half tile.
    //       A: half tile row r is tile row 128 * (r / 64) + 64 * half + r % 64;
    //       B: half tile row r is tile row  64 * (r / 32) + 32 * half + r % 32.
    //   KS: a load is 4 k-rows of 256 bytes: k-rows 4 w .. + 3 and 32 + 4 w .. + 3, columns 128 * half .. + 127.
    const int r8 = lane >> 3, kc_chunk = (lane & 7) ^ ((((8 * wave + r8) >> 1)) & 7);
    const uint32_t a_lane = ((uint32_t)(m0 + 8 * wave + r8) * A.ld + (uint32_t)(8 * kc_chunk)) * 2u;
    const uint32_t a_half = 128u * A.ld, a_second = 256u * A.ld;                  // 64 and 128 rows, in bytes
    const int k4 = 4 * wave + (lane >> 4);
    const uint32_t b_lane = BKIND == KC
        ? ((uint32_t)(n0 + 64 * (wave >> 2) + 8 * (wave & 3) + r8) * Bop.ld + (uint32_t)(8 * kc_chunk)) * 2u
        : ((uint32_t)k4 * Bop.ld + (uint32_t)(n0 + 8 * ((lane & 15) ^ ks_swizzle(k4)))) * 2u;
    const uint32_t b_half = BKIND == KC ? 64u * Bop.ld : 256u;                    // 32 rows | 128 columns
    const uint32_t b_second = BKIND == KC ? 256u * Bop.ld : 64u * Bop.ld;         // 128 rows | 32 k-rows
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;
    auto load_a = [&](int half, int step) {
        const uint32_t src = (uint32_t)(k_first + step * k_stride) * 2u + half * a_half;
        const uint32_t dst = lds_wave + (step & 1) * STAGE_BYTES + half * HALF_TILE_BYTES;
        load_to_lds(A, a_lane, src, dst);
        load_to_lds(A, a_lane, src + a_second, dst + HALF_TILE_BYTES / 2);
    };
    auto load_b = [&](int half, int step) {
        const uint32_t k = (uint32_t)(k_first + step * k_stride);
        const uint32_t src = (BKIND == KC ? k : k * Bop.ld) * 2u + half * b_half;
        const uint32_t dst = lds_wave + (step & 1) * STAGE_BYTES + OPERAND_TILE_BYTES + half * HALF_TILE_BYTES;
        load_to_lds(Bop, b_lane, src, dst);
        load_to_lds(Bop, b_lane, src + b_second, dst + HALF_TILE_BYTES / 2);
    };

    const FragReader<BKIND> frag(wm, wn, i, g);
    bf16x8 af[MT / 2][2], bf0[NT / 2][2], bf1[NT / 2][2];
    auto read_a = [&](int half, int stage) { frag.read_a(af, lds, half, stage); };
    auto read_b = [&](bf16x8 (&bf)[NT / 2][2], int half, int stage) { frag.read_b(bf, lds, half, stage); };

    // k-steps 0 and 1 in the order in which the loop would have issued their loads; then B0(0), which the loop
    // reads one phase ahead
    load_b(0, 0); load_a(0, 0); load_b(1, 0); load_a(1, 0);
    if (last > 0) {
        load_b(0, 1); load_a(0, 1); load_b(1, 1); load_a(1, 1);
        wait_counts<12, NO_LG_WAIT>();
    } else {
        wait_counts<4, NO_LG_WAIT>();
    }
    raw_barrier();
    read_b(bf0, 0, 0);
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    if (wm == 1) raw_barrier();                        // the second half of the waves falls one slot behind

    for (int j = 0; j < last - 1; ++j) {
        const int cur = (j & 1) * STAGE_BYTES, nxt = STAGE_BYTES - cur;
        read_a(0, cur);      load_b(0, j + 2); wait_counts<12, 0>(); raw_barrier();
        quadrant_mfmas<0>(acc, af, bf0); raw_barrier();
        read_b(bf1, 1, cur); load_a(0, j + 2); wait_counts<12, 0>(); raw_barrier();
        quadrant_mfmas<1>(acc, af, bf1); raw_barrier();
        read_a(1, cur);      load_b(1, j + 2); wait_counts<12, 0>(); raw_barrier();
        quadrant_mfmas<2>(acc, af, bf0); raw_barrier();
        read_b(bf0, 0, nxt); load_a(1, j + 2); wait_counts<12, 0>(); raw_barrier();
        quadrant_mfmas<3>(acc, af, bf1); raw_barrier();
    }
    if (last > 0) {          // the last but one: nothing left to load
        const int cur = ((last - 1) & 1) * STAGE_BYTES, nxt = STAGE_BYTES - cur;
        read_a(0, cur);      wait_counts<10, 0>(); raw_barrier();
        quadrant_mfmas<0>(acc, af, bf0); raw_barrier();
        read_b(bf1, 1, cur); wait_counts<8, 0>(); raw_barrier();
        quadrant_mfmas<1>(acc, af, bf1); raw_barrier();
        read_a(1, cur);      wait_counts<6, 0>(); raw_barrier();
        quadrant_mfmas<2>(acc, af, bf0); raw_barrier();
        read_b(bf0, 0, nxt); wait_counts<4, 0>(); raw_barrier();
        quadrant_mfmas<3>(acc, af, bf1); raw_barrier();
    }
    {
        const int cur = (last & 1) * STAGE_BYTES;
        read_a(0, cur);      wait_counts<2, 0>(); raw_barrier();
        quadrant_mfmas<0>(acc, af, bf0); raw_barrier();
        read_b(bf1, 1, cur); wait_counts<0, 0>(); raw_barrier();
        quadrant_mfmas<1>(acc, af, bf1); raw_barrier();
        read_a(1, cur);      wait_counts<NO_VM_WAIT, 0>(); raw_barrier();
        quadrant_mfmas<2>(acc, af, bf0); raw_barrier();
        quadrant_mfmas<3>(acc, af, bf1);
    }
    if (wm == 0) raw_barrier();
    raw_barrier();
}

__device__ __forceinline__ void zero_acc(acc_t& acc) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;
}

// ---- thin tiles ------------------------------------------------------------------------------------
// A launch whose tile count is not a multiple of the 256 compute units ends with a round in which
// most of them idle.  The tiles of that last round can instead be cut into four "thin" tiles of
// 256 x 64 (one wave column of a full tile each) and handed to four times as many workgroups.  A thin
// tile does a quarter of the MFMA work for 5/8 of the staging traffic in about half of a full tile's time.
constexpr int THIN_N = WAVE_N;                         // 64 columns
constexpr int THIN_WAVE_M = TILE_M / 8;                // a wave of a thin tile: 32 rows x 64 columns
constexpr int THIN_MT = THIN_WAVE_M / 16, THIN_NT = THIN_N / 16;
constexpr int THIN_STAGE_BYTES = OPERAND_TILE_BYTES + THIN_N * TILE_K * 2;    // 32 KiB A + 8 KiB B
constexpr int THIN_STAGES = 3;
static_assert(THIN_STAGES * THIN_STAGE_BYTES <= LDS_BYTES, "");
typedef f32x4 thin_acc_t[THIN_MT][THIN_NT];

// A thin tile's B operand may also be k-strided (memory [k][col]): LDS then holds [64 k][64 cols], 128 bytes per
// k-row, 16-byte chunks XOR-ed with thin_ks_swizzle(k).  A transposing read is served half a wave at a time:
// 8 k-rows (k & 3 and bit 3 of k), two adjacent chunks and both halves of a chunk; k & 1 picks the 128-byte
// half of the bank window, bits 1 and 3 of k go to chunk bits 1-2, the adjacent chunks differ in bit 0.
__device__ __forceinline__ int thin_ks_swizzle(int k) { return (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2); }

// acc[mt][nt] += A(m0 .. m0+255, k) * B(n0 .. n0+63, k) for k in [k_begin, k_begin + 64 * k_steps);
// wave w holds rows 32 w .. 32 w + 31.  A is KC; BKIND KS: B is k-strided, n0 its first column.  Three LDS stages
// filled straight from global memory two k-steps ahead, one barrier per k-step: behind the barrier of k-step j
// every wave has its loads of k-step j in LDS and has finished reading k-step j - 1, whose stage the loads of
// k-step j + 2 refill.  Ends with a workgroup barrier.
template <int BKIND = KC>
__device__ __forceinline__ void thin_mainloop(thin_acc_t& acc, const Operand& A, const Operand& Bop, int m0, int n0,
                                              int k_begin, int k_steps, char* lds, bool descending = false) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4, r8 = lane >> 3;
    const int last = k_steps - 1;
    const int k_first = descending ? k_begin + last * TILE_K : k_begin;
    const int k_stride = descending ? -TILE_K : TILE_K;
    // wave w loads rows 64 q + 8 w .. + 7 of A (q = 0 .. 3) and rows (KC) or k-rows (KS) 8 w .. + 7 of B
    const int row = 8 * wave + r8, kc_chunk = (lane & 7) ^ ((row >> 1) & 7);
    const uint32_t a_lane = ((uint32_t)(m0 + row) * A.ld + (uint32_t)(8 * kc_chunk)) * 2u;
    const uint32_t b_lane = BKIND == KC
        ? ((uint32_t)(n0 + row) * Bop.ld + (uint32_t)(8 * kc_chunk)) * 2u
        : ((uint32_t)row * Bop.ld + (uint32_t)(n0 + 8 * ((lane & 7) ^ thin_ks_swizzle(row)))) * 2u;
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;
    auto load = [&](int step, int stage) {
        const uint32_t k = (uint32_t)(k_first + step * k_stride);
        const uint32_t dst = lds_wave + (uint32_t)stage;
#pragma unroll
        for (int q = 0; q < 4; ++q) load_to_lds(A, a_lane, 2u * k + (uint32_t)q * 128u * A.ld, dst + q * 8192);
        load_to_lds(Bop, b_lane, (BKIND == KC ? k : k * Bop.ld) * 2u, dst + OPERAND_TILE_BYTES);
    };
    int a_frag[2], b_frag[THIN_NT];
#pragma unroll
    for (int s = 0; s < 2; ++s) a_frag[s] = (THIN_WAVE_M * wave + i) * 128 + (((4 * s + g) ^ (i >> 1)) << 4);
#pragma unroll
    for (int t = 0; t < THIN_NT; ++t) {
        if (BKIND == KC) {
            b_frag[t] = OPERAND_TILE_BYTES + i * 128 + (((4 * (t & 1) + g) ^ (i >> 1)) << 4);    // t = k-substep 0 | 1
        } else {
            const int krow = 8 * g + (i >> 2), col = 16 * t + 4 * (i & 3);
            b_frag[t] = OPERAND_TILE_BYTES + krow * 128 + (((col >> 3) ^ thin_ks_swizzle(krow)) << 4) + ((col & 7) << 1);
        }
    }
    load(0, 0);
    if (last > 0) load(1, THIN_STAGE_BYTES);
    int cur = 0, nxt = 2 * THIN_STAGE_BYTES;              // stages of k-steps j and j + 2
    for (int j = 0; j <= last; ++j) {
        if (j < last) wait_counts<5, NO_LG_WAIT>();       // k-step j + 1 may still be on its way
        else wait_counts<0, NO_LG_WAIT>();
        raw_barrier();
        if (j + 2 <= last) load(j + 2, nxt);
        bf16x8 af[THIN_MT][2], bf[THIN_NT][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int t = 0; t < THIN_MT; ++t)
                af[t][s] = *reinterpret_cast<const bf16x8*>(lds + (a_frag[s] + cur) + t * 2048);
#pragma unroll
            for (int t = 0; t < THIN_NT; ++t) {
                if (BKIND == KC) {
                    bf[t][s] = *reinterpret_cast<const bf16x8*>(lds + (b_frag[s] + cur) + t * 2048);
                } else {
                    typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
                    const char* p = lds + (b_frag[t] + cur) + s * (32 * 128);
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * 128));
                    bf[t][s] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int x = 0; x < THIN_MT; ++x)
#pragma unroll
                for (int y = 0; y < THIN_NT; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[x][s], bf[y][s], acc[x][y], 0, 0, 0);
        cur += THIN_STAGE_BYTES;
        if (cur == THIN_STAGES * THIN_STAGE_BYTES) cur = 0;
        nxt += THIN_STAGE_BYTES;
        if (nxt == THIN_STAGES * THIN_STAGE_BYTES) nxt = 0;
    }
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
}

// How a launch of n_tiles full tiles is cut: the tiles of the last, partial round become thin tiles
// when those fit one round of the compute units.
struct TilePlan {
    int n_full;      // full tiles, logical ids 0 .. n_full - 1 (workgroups 0 .. 8 * ceil(n_full / 8) - 1)
    int n_thin;      // thin tiles: 4 per remaining full tile, workgroups thin_first .. thin_first + n_thin - 1
    int thin_first;
};

// Workgroups are handed to the 8 XCDs round-robin by their linear id; each XCD has its own L2.
// Map the hardware id to a logical tile id so that each XCD walks one contiguous range of
// logical tiles (tiles that share an operand panel are numbered next to each other).
// The grid must hold 8 * ceil(n_tiles / 8) workgroups; returns -1 for the surplus ones.
__device__ __forceinline__ int xcd_logical_tile(int n_tiles, int bid = blockIdx.x) {
    const int per = (n_tiles + 7) >> 3;
    const int t = (bid & 7) * per + (bid >> 3);
    return t < n_tiles ? t : -1;
}

// Round-to-nearest-even conversion of two floats to a packed bf16 pair.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2 f = {a, b};
    bf16x2 r = __builtin_convertvector(f, bf16x2);
    return __builtin_bit_cast(uint32_t, r);
}

// ---- output tiles through LDS ------------------------------------------------------------------------
// The MFMA accumulator layout gives a lane one N index and groups of four consecutive M indices, which
// makes direct global stores 8 or 16 bytes wide and scattered over 16 rows.  Instead the 256 x 256 tile
// is rounded to bf16 and laid out in LDS as [n][m] (512 bytes per n; it fills the 128 KiB the main loop
// no longer needs), then written out row by row.  Every n-row starts at bank 0, so the eight-byte slots of
// a row are XOR-ed with n & 15.  Measured on gfx950 with the bank-conflict counter:
//   accumulator writes (ds_write_b64): served 16 consecutive lanes at a time, and the 16 slots must differ
//       modulo 16 (a 128-byte window).  The 16 lanes are 16 consecutive n and one slot s, and s ^ (n & 15)
//       takes every value modulo 16 once;
//   row reads (ds_read_b128): served in the lane sets {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} of each
//       half wave, whose 16-byte chunks must differ modulo 16 (a 256-byte window).  A lane's chunk is two
//       adjacent slots, swapped when n is odd; both lane sets cover every chunk index modulo 16 once and
//       c -> c ^ ((n & 15) >> 1) permutes them.

__device__ __forceinline__ int out_tile_swizzle(int n) { return n & 15; }

// Byte offset of element (n, m) in the swizzled tile; m must be a multiple of 4 for 8-byte accesses.
__device__ __forceinline__ int out_tile_offset(int n, int m) {
    return n * 512 + (((m >> 2) ^ out_tile_swizzle(n)) << 3) + ((m & 3) << 1);
}

template <int BKIND>
__device__ __forceinline__ void acc_to_lds_bf16(const acc_t& acc, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3, g = lane >> 4, jl = lane & 15;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = wave_col<BKIND>(wn, nt) + jl;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            u32x2 p;
            p[0] = pack_bf16(acc[mt][nt][0], acc[mt][nt][1]);
            p[1] = pack_bf16(acc[mt][nt][2], acc[mt][nt][3]);
            *reinterpret_cast<u32x2*>(lds + out_tile_offset(n, wm * WAVE_M + 16 * mt + 4 * g)) = p;
        }
    }
}

// Writes the LDS tile to out[n][m] (row pitch ld elements, `out` = address of element (0, 0) of the
// tile), rows n < n_valid and columns m < m_valid only.  A wave stores two whole 512-byte rows per
// instruction; a chunk that m_valid cuts (m_valid not a multiple of 8) goes out element by element.
__device__ __forceinline__ void lds_tile_store_rows(const char* lds, uint16_t* out, int64_t ld, int n_valid,
                                                    int m_valid) {
    const int tid = threadIdx.x;
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
        const int q = tid + NTHREADS * i;
        const int n = q >> 5, cq = q & 31;
        if (n < n_valid && cq * 8 < m_valid) {
            // the two 8-byte halves of a 16-byte chunk stay in one chunk, swapped when the swizzle is odd
            const int g = out_tile_swizzle(n);
            u32x4 v = *reinterpret_cast<const u32x4*>(lds + n * 512 + ((cq ^ (g >> 1)) << 4));
            if (g & 1) v = __builtin_shufflevector(v, v, 2, 3, 0, 1);
            uint16_t* o = out + (int64_t)n * ld + cq * 8;
            if (cq * 8 + 8 <= m_valid) {
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(o));
            } else {
                const int left = m_valid - cq * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e < left) o[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

// bf16(w - lr * g), eight weights w and gradients g (bf16), in fp32.
__device__ __forceinline__ u32x4 updated_weights(u32x4 w, u32x4 g, float lr) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float w0 = __uint_as_float(w[e] << 16), w1 = __uint_as_float(w[e] & 0xffff0000u);
        const float g0 = __uint_as_float(g[e] << 16), g1 = __uint_as_float(g[e] & 0xffff0000u);
        r[e] = pack_bf16(fmaf(-lr, g0, w0), fmaf(-lr, g1, w1));
    }
    return r;
}

// The LDS tile holds a gradient; out[n][m] <- bf16(out[n][m] - lr * tile[n][m]) for rows n < n_valid and columns
// m < m_valid (a multiple of 8), each 16-byte chunk read, updated in fp32 and written back.  All of a thread's chunks are
// read by tile_update_load, called while the accumulators are on their way to LDS: read four at a time between the
// stores, the fused update of 125 000 x 2048 weights at B = 1024 took 621 us, now 549.
constexpr int UPDATE_CHUNKS = TILE_M * TILE_N / 8 / NTHREADS;
__device__ __forceinline__ void tile_update_load(u32x4 (&w)[UPDATE_CHUNKS], const uint16_t* out, int64_t ld, int n_valid, int m_valid) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < UPDATE_CHUNKS; ++i) {
        const int q = tid + NTHREADS * i;
        const int n = q >> 5, cq = q & 31;
        w[i] = u32x4{0, 0, 0, 0};
        if (n < n_valid && cq * 8 < m_valid) w[i] = *reinterpret_cast<const u32x4*>(out + (int64_t)n * ld + cq * 8);
    }
}
__device__ __forceinline__ void lds_tile_update_rows(const char* lds, u32x4 (&w)[UPDATE_CHUNKS], uint16_t* out, int64_t ld,
                                                     int n_valid, int m_valid, float lr) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < UPDATE_CHUNKS; ++i) {
        const int q = tid + NTHREADS * i;
        const int n = q >> 5, cq = q & 31;
        if (n < n_valid && cq * 8 < m_valid) {
            const int g = out_tile_swizzle(n);
            u32x4 gr = *reinterpret_cast<const u32x4*>(lds + n * 512 + ((cq ^ (g >> 1)) << 4));
            if (g & 1) gr = __builtin_shufflevector(gr, gr, 2, 3, 0, 1);
            __builtin_nontemporal_store(updated_weights(w[i], gr, lr), reinterpret_cast<u32x4*>(out + (int64_t)n * ld + cq * 8));
        }
    }
}

}  // namespace ws
