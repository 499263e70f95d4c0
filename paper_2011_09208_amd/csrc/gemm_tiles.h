// Persistent form of the GEMM main loop (gemm_core.h) for tiles of any height: one workgroup per compute unit walks a list of
// tiles of 32 to 256 rows (M) x 256 columns (N).
//
// Why lists: a launch of whole 256 x 256 tiles takes as long as the compute unit with the most of them.  12 500 classes x 1024
// rows are 196 tiles, so 60 units idle; 37 500 classes are 588, three rounds for 2.3.  Here every unit has the same
// number of classes, cut into tiles of nearly equal height.  Why persistent: the loads run two k-steps ahead across tile
// boundaries, so that the next tile's operands arrive during the epilogue, its stores are on their way
// during the next tile, and no unit waits for a workgroup to end and another to start.
#pragma once
#include "gemm_core.h"

namespace ws {

// Rows of a tile come in units of 32, two M tiles of the matrix instruction.  A tile of u units gives ceil(u / 2) of them to wave
// row 0 and the rest to wave row 1 (the two waves of a SIMD, so every SIMD has the same work); a wave row's q units are
// ceil(q / 2) in half 0 of its sub-tile and the rest in half 1 (the halves of the main loop's phases).
constexpr int UNIT = 32;
constexpr int MAX_UNITS = TILE_M / UNIT;
__host__ __device__ constexpr int wave_row_units(int units, int wm) { return (units + 1 - wm) >> 1; }
__host__ __device__ constexpr int half_units(int row_units, int half) { return (row_units + 1 - half) >> 1; }

// The rows of a unit are dealt to the MFMA row index so that a lane's accumulators of its two M tiles are 8 consecutive rows:
// element (mt, v) of lane group g is row unit_row(mt, g) + v of its half's 64 (if the half has that many).
__device__ __forceinline__ int unit_row(int mt, int g) { return 32 * ((mt >> 1) & 1) + 8 * g + 4 * (mt & 1); }

// A tile of the list: rows m0 .. m0 + 32 * units - 1 of A, columns n0 .. n0 + 255 of B (KC: rows); the k-steps from the last to
// the first if `descending`.
struct ListTile {
    int m0, n0, units;
    bool descending;
};

constexpr int LIST_WGS = 256;            // a workgroup per compute unit

// Nothing of an operand is in range from here on, or a row's length around here (unless it has more than 3.7 GiB: then the load
// reads what nobody uses).
constexpr uint32_t NOWHERE = 0xf0000000u;

// The MFMAs of the first UNITS units of quadrant Q (quadrant_mfmas).
template <int Q, int UNITS>
__device__ __forceinline__ void quadrant_units(acc_t& acc, const bf16x8 (&af)[MT / 2][2], const bf16x8 (&bf)[NT / 2][2]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int x = 0; x < 2 * UNITS; ++x)
#pragma unroll
            for (int y = 0; y < NT / 2; ++y) {
                f32x4& c = acc[MT / 2 * (Q >> 1) + x][NT / 2 * (Q & 1) + y];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[x][s], bf[y][s], c, 0, 0, 0);
            }
    __builtin_amdgcn_sched_barrier(0);
}
// Accumulators of quadrant Q start from zero.  In registers of their own, which the empty assembly sees to: as the constant
// operand of the first MFMA they would be other registers in either branch above, and the compiler copies and spills.
template <int Q>
__device__ __forceinline__ void quadrant_zero(acc_t& acc) {
#pragma unroll
    for (int x = 0; x < MT / 2; ++x)
#pragma unroll
        for (int y = 0; y < NT / 2; ++y) {
            f32x4& c = acc[MT / 2 * (Q >> 1) + x][NT / 2 * (Q & 1) + y];
            c = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+v"(c));
        }
}

// Runs the list: list.rounds > 0 tiles list.tile(round) of k_steps k-steps each, starting at k = 0.  Epi:
//   begin(round)                    issue loads for the tile's epilogue, if any; in round 0 STORES stores without effect, too
//   end(acc, round, units[2])       the tile is complete: units[h] units of this wave's half h are in acc.  All waves are
//                                   here together (barriers are allowed); STORES vector-memory operations at least are issued
//                                   by every wave, all of them after every load of this call.
// A phase's waits are those of gemm_mainloop: the loads of the last six phases may be outstanding, and in the first six phases
// of a tile the STORES operations between the tiles, too (loads and stores count in one order).
template <int BKIND, int STORES, class List, class Epi>
__device__ __forceinline__ void gemm_tiles(const Operand& A, const Operand& Bop, int k_steps, const List& list, Epi& epi,
                                           char* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int i = lane & 15, g = lane >> 4;

    // Global -> LDS, as in gemm_mainloop with the rows of A permuted (unit_row) and the tile in the scalar offset.  Of a half tile
    // of A, wave w loads LDS rows 8 w .. + 7 of each wave row's 64: a quarter of unit w / 4.
    const int r8 = lane >> 3, kc_chunk = (lane & 7) ^ (((8 * wave + r8) >> 1) & 7);
    const int a_row = 32 * (wave >> 2) + 4 * ((wave >> 1) & 1) + 16 * (wave & 1) + (r8 & 3) + 8 * (r8 >> 2);
    const uint32_t a_lane = ((uint32_t)a_row * A.ld + (uint32_t)(8 * kc_chunk)) * 2u;
    const int k4 = 4 * wave + (lane >> 4);
    const uint32_t b_lane = BKIND == KC
        ? ((uint32_t)(64 * (wave >> 2) + 8 * (wave & 3) + r8) * Bop.ld + (uint32_t)(8 * kc_chunk)) * 2u
        : ((uint32_t)k4 * Bop.ld + (uint32_t)(8 * ((lane & 15) ^ ks_swizzle(k4)))) * 2u;
    const uint32_t b_half = BKIND == KC ? 64u * Bop.ld : 256u;                    // 32 rows | 128 columns
    const uint32_t b_second = BKIND == KC ? 256u * Bop.ld : 64u * Bop.ld;         // 128 rows | 32 k-rows
    const uint32_t b_step = BKIND == KC ? 128u : 128u * Bop.ld;
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;
    const uint32_t unit_bytes = (uint32_t)UNIT * A.ld * 2u;

    // The load cursor: a k-step of some tile, two k-steps ahead of the MFMAs.  Past the last tile it loads from nowhere,
    // so that every phase issues the same number of loads.
    uint32_t a_src[2][2], a_inc = 0, b_src, b_inc = 0;   // a_src[half][wave row]
    int load_round = 0, load_left = 0;
    auto cursor_next = [&]() __attribute__((always_inline)) {
        if (load_left > 0) {
            --load_left;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 2; ++r) a_src[h][r] += a_inc;      // nowhere stays nowhere
            b_src += b_inc;
            return;
        }
        if (load_round == list.rounds) {
            a_src[0][0] = a_src[0][1] = a_src[1][0] = a_src[1][1] = b_src = NOWHERE;
            a_inc = b_inc = 0;
            load_left = INT32_MAX;
            return;
        }
        const ListTile t = list.tile(load_round++);
        const uint32_t k = t.descending ? (uint32_t)(k_steps - 1) : 0u;
        uint32_t from = (uint32_t)t.m0 * A.ld * 2u + k * 128u;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int u = half_units(wave_row_units(t.units, r), h);
                a_src[h][r] = (wave >> 2) < u ? from : NOWHERE;
                from += (uint32_t)u * unit_bytes;
            }
        b_src = (BKIND == KC ? (uint32_t)t.n0 * Bop.ld * 2u : (uint32_t)t.n0 * 2u) + k * b_step;
        a_inc = t.descending ? 0u - 128u : 128u;
        b_inc = t.descending ? 0u - b_step : b_step;
        load_left = k_steps - 1;
    };
    auto load_a = [&](int half, int stage) {
        const uint32_t dst = lds_wave + stage + half * HALF_TILE_BYTES;
        load_to_lds(A, a_lane, a_src[half][0], dst);
        load_to_lds(A, a_lane, a_src[half][1], dst + HALF_TILE_BYTES / 2);
    };
    auto load_b = [&](int half, int stage) {
        const uint32_t src = b_src + half * b_half, dst = lds_wave + stage + OPERAND_TILE_BYTES + half * HALF_TILE_BYTES;
        load_to_lds(Bop, b_lane, src, dst);
        load_to_lds(Bop, b_lane, src + b_second, dst + HALF_TILE_BYTES / 2);
    };

    const FragReader<BKIND> frag(wm, wn, i, g);
    bf16x8 af[MT / 2][2], bf0[NT / 2][2], bf1[NT / 2][2];
    acc_t acc;

    int cur = 0;                                         // stage of the k-step being multiplied
    cursor_next();
    load_b(0, 0); load_a(0, 0); load_b(1, 0); load_a(1, 0);
    cursor_next();
    load_b(0, STAGE_BYTES); load_a(0, STAGE_BYTES); load_b(1, STAGE_BYTES); load_a(1, STAGE_BYTES);
    cursor_next();
    epi.begin(0);
    wait_counts<12 + STORES, NO_LG_WAIT>();
    raw_barrier();
    frag.read_b(bf0, lds, 0, 0);
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    if (wm == 1) raw_barrier();                          // the second half of the waves falls one slot behind

    int units[2];
    auto step = [&](auto units0, auto units1, auto first, auto stores_in_first_two) __attribute__((always_inline)) {
        constexpr int U0 = decltype(units0)::value, U1 = decltype(units1)::value;
        constexpr bool FIRST = decltype(first)::value;
        constexpr int S01 = decltype(stores_in_first_two)::value ? STORES : 0, S23 = FIRST ? STORES : 0;
        const int nxt = STAGE_BYTES - cur;
        frag.template read_a<U0>(af, lds, 0, cur);
        load_b(0, cur);
        if (FIRST) quadrant_zero<0>(acc);
        wait_counts<12 + S01, 0>();
        raw_barrier();
        quadrant_units<0, U0>(acc, af, bf0);
        raw_barrier();
        frag.read_b(bf1, lds, 1, cur);
        load_a(0, cur);
        if (FIRST) quadrant_zero<1>(acc);
        wait_counts<12 + S01, 0>();
        raw_barrier();
        quadrant_units<1, U0>(acc, af, bf1);
        raw_barrier();
        frag.template read_a<U1>(af, lds, 1, cur);
        load_b(1, cur);
        if (FIRST) quadrant_zero<2>(acc);
        wait_counts<12 + S23, 0>();
        raw_barrier();
        quadrant_units<2, U1>(acc, af, bf0);
        raw_barrier();
        frag.read_b(bf0, lds, 0, nxt);
        load_a(1, cur);
        cursor_next();
        if (FIRST) quadrant_zero<3>(acc);
        wait_counts<12 + S23, 0>();
        raw_barrier();
        quadrant_units<3, U1>(acc, af, bf1);
        raw_barrier();
        cur = nxt;
    };
    for (int r = 0; r < list.rounds; ++r) {
        const int mine = wave_row_units(list.tile(r).units, wm);
        units[0] = half_units(mine, 0);
        units[1] = half_units(mine, 1);
        auto tile = [&](auto units0, auto units1) __attribute__((always_inline)) {
            step(units0, units1, std::true_type(), std::true_type());
            if (k_steps > 1) step(units0, units1, std::false_type(), std::true_type());
            for (int j = 2; j < k_steps; ++j) step(units0, units1, std::false_type(), std::false_type());
        };
        typedef std::integral_constant<int, 0> none;
        typedef std::integral_constant<int, 1> one;
        typedef std::integral_constant<int, 2> two;
        if (mine == 4) tile(two(), two());
        else if (mine == 3) tile(two(), one());
        else if (mine == 2) tile(one(), one());
        else if (mine == 1) tile(one(), none());
        else tile(none(), none());
        if (wm == 0) raw_barrier();                      // the halves of the waves come together
        epi.end(acc, r, units);
        if (r + 1 < list.rounds) {
            epi.begin(r + 1);
            if (wm == 1) raw_barrier();
        }
    }
    wait_counts<0, 0>();                                 // the loads past the last tile write LDS
}

}  // namespace ws
