// Persistent form of the GEMM main loop (gemm_core.h) with a k-strided B operand: one workgroup per compute unit walks a
// list of output tiles as ONE stream of k-steps.  The loads run two k-steps ahead across tile boundaries, so a tile starts on operands
// that are already in LDS; the epilogue of a tile sits in the LOAD slots around the boundary, where the other wave
// of the SIMD feeds the matrix core; and the stores of a tile are spread over the k-steps of the next one.
#pragma once
#include "gemm_core.h"

namespace ws {

// Rows of the A tile are dealt to the MFMA row index so that a lane's accumulators of M tiles 2 u and 2 u + 1 are 8
// consecutive rows: element (mt, v) of lane group g is row stream_row(mt, g) + v of the wave's 128.  A lane then
// packs 16 consecutive bytes of the output.
__device__ __forceinline__ int stream_row(int mt, int g) {
    return 64 * (mt >> 2) + 32 * ((mt >> 1) & 1) + 8 * g + 4 * (mt & 1);
}

constexpr int STREAM_WGS = 256;          // one workgroup per compute unit
constexpr int STREAM_SCRATCH_BYTES = 4096;                              // LDS per wave for its epilogue
constexpr int STREAM_LDS_BYTES = LDS_BYTES + 8 * STREAM_SCRATCH_BYTES;  // all 160 KiB of the compute unit
constexpr int STREAM_MIN_K_STEPS = 4;    // shortest tile whose 16 stores fit before the next tile's (stream_stores)

// Where a tile of the stream lies in the operands.
struct StreamTile {
    int m0, n0;
    bool descending;
};

// Tiles of a launch of n_tiles for stream workgroup `wg`: XCD wg % 8 owns one contiguous range of tiles (as
// xcd_logical_tile deals them), its 32 workgroups take every 32nd of it.
struct StreamShare {
    int first, count;
    __device__ __forceinline__ StreamShare(int n_tiles, int wg) {
        const int per = (n_tiles + 7) >> 3, lo = (wg & 7) * per, idx = wg >> 3;
        const int left = (lo + per < n_tiles ? lo + per : n_tiles) - lo - idx;
        first = lo + idx;
        count = left > 0 ? (left + 31) >> 5 : 0;
    }
    __device__ __forceinline__ int tile(int round) const { return first + 32 * round; }
};

// The k-steps of a tile: the first, the second, those that still store values of the tile before (FETCH: the last
// quadrant's values are taken from LDS), those that only multiply, the last.
enum StreamStep { FIRST_STEP, SECOND_STEP, STORE_STEP, FETCH_STEP, PLAIN_STEP, LAST_STEP };

// Vector-memory stores issued in a phase.  A wave has 16 for a tile; they start in phase 2 of its last k-step and
// go on in the next tile at RATE per k-step.
//   RATE 1: 8 around the boundary, then 8: tiles of 10 k-steps or more
//   RATE 2: the same 8, then 8: 6 or more      RATE 4: 12 and 4: 4 or more
// At most four values (16 registers) wait for their turn while all accumulators are in use.
constexpr int stream_stores(int rate, int step, int phase) {
    if (step == LAST_STEP && phase >= 2) return rate == 4 || phase == 3 ? 2 : 1;
    if (step == FIRST_STEP) return rate == 4 || phase == 0 ? 2 : 1;
    if (step == PLAIN_STEP || step == LAST_STEP) return 0;
    return rate == 4 ? 1 : rate == 2 ? (phase % 2 == 0) : (phase == 0);
}
// Stores of the last six phases up to and including this one (at least so many: the steps before a plain or the last
// one are taken for plain, those before a storing one for storing, a FIRST_STEP before it stores no less).
constexpr int stream_window_stores(int rate, int step, int phase) {
    int n = 0;
    for (int back = 0; back < 6; ++back) {
        int p = phase - back, s = step;
        while (p < 0) {
            p += 4;
            s = s == SECOND_STEP ? FIRST_STEP : s == FIRST_STEP ? LAST_STEP : s == LAST_STEP ? PLAIN_STEP : s;
        }
        n += stream_stores(rate, s, p);
    }
    return n;
}
// Prefetch of B's lines into the L2, for an operand that comes from HBM while the kernel writes much: with
// writes in flight a few of a k-step's 256 lines arrive late, and all eight waves wait for the last one.  A load that
// brings a line into the L2 three k-steps before its tile's loads hides that (dW, B = 1024, D = 2048, C = 100 000: 372 ->
// 345 us; B = 256: 165 -> 141); further ahead changes nothing.  Where the lines are near anyway it costs 2 %.
// Workgroups of an XCD that run tiles with the same panel share the work: this one is `index` of `count` (1, 2, 4, 8).
constexpr int PREFETCH_STEPS = 3;
struct PrefetchShare {
    int index, count;
    // `sharers` workgroups share a panel, this is the n-th of them
    __device__ __forceinline__ PrefetchShare(int n, int sharers) {
        count = sharers >= 8 ? 8 : sharers >= 4 ? 4 : sharers >= 2 ? 2 : 1;
        index = n & (count - 1);
    }
};

constexpr int stream_rate(int k_steps) { return k_steps >= 10 ? 1 : k_steps >= 6 ? 2 : 4; }

// Runs the stream.  `tile_at(round)` gives the tile of a round (0 .. rounds - 1); every tile has k_steps k-steps
// starting at k = 0, RATE = stream_rate(k_steps).  Epi:
//   begin_next()      finish<q> from now on is called for the next tile of the list
//   finish<q>(acc)    quadrant q = 2 * (A half) + (B half) of the tile is complete: take it out of acc
//   fetch<q>()        called after finish<q> (q < 3: one phase later, just before finish<q + 1>)
//   store<n>()        issue exactly one vector-memory store, of the oldest of the at most n values that are fetched
//                     and not stored (called 16 times between fetch<0> of one tile and of the next, and more often:
//                     then, and before the first tile is finished, the store must have no effect)
// Loads and stores count in one order, so the wait of a phase allows the 12 loads of the main loop plus the stores
// (and the prefetch, in phase 3) issued in the last six phases.
template <int RATE, bool PREFETCH, class TileAt, class Epi>
__device__ __forceinline__ void gemm_stream(const Operand& A, const Operand& Bop, int k_steps, int rounds,
                                            TileAt tile_at, PrefetchShare share, Epi& epi, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int i = lane & 15, g = lane >> 4;

    // Global -> LDS, as in gemm_mainloop with the rows of A permuted (stream_row) and the tile in the scalar offset.
    const int r8 = lane >> 3, kc_chunk = (lane & 7) ^ (((8 * wave + r8) >> 1) & 7);
    const int a_row = 32 * (wave >> 2) + 4 * ((wave >> 1) & 1) + 16 * (wave & 1) + (r8 & 3) + 8 * (r8 >> 2);
    const uint32_t a_lane = ((uint32_t)a_row * A.ld + (uint32_t)(8 * kc_chunk)) * 2u;
    const uint32_t a_half = 128u * A.ld, a_second = 256u * A.ld;
    const int k4 = 4 * wave + (lane >> 4);
    const uint32_t b_lane = ((uint32_t)k4 * Bop.ld + (uint32_t)(8 * ((lane & 15) ^ ks_swizzle(k4)))) * 2u;
    const uint32_t b_second = 64u * Bop.ld, b_step = 128u * Bop.ld;
    const uint32_t lds_wave = lds_offset(lds) + 1024u * (uint32_t)wave;

    // The load cursor: a k-step of some tile, two k-steps ahead of the MFMAs.  Past the last tile it starts that tile
    // again (nobody reads what it loads), so that every phase issues the same number of loads.
    uint32_t a_src, b_src, a_inc, b_inc;
    int load_round = 0, load_left = 0;
    auto cursor_tile = [&](int round) {
        const StreamTile t = tile_at(round);
        const uint32_t k = t.descending ? (uint32_t)(k_steps - 1) : 0u;
        a_src = (uint32_t)t.m0 * A.ld * 2u + k * 128u;
        b_src = (uint32_t)t.n0 * 2u + k * b_step;
        a_inc = t.descending ? 0u - 128u : 128u;
        b_inc = t.descending ? 0u - b_step : b_step;
        load_left = k_steps;
    };
    auto cursor_next = [&]() {
        a_src += a_inc;
        b_src += b_inc;
        if (--load_left == 0) {
            if (load_round < rounds - 1) ++load_round;
            cursor_tile(load_round);
        }
    };
    auto load_a = [&](int half, int stage) {
        const uint32_t src = a_src + half * a_half, dst = lds_wave + stage + half * HALF_TILE_BYTES;
        load_to_lds(A, a_lane, src, dst);
        load_to_lds(A, a_lane, src + a_second, dst + HALF_TILE_BYTES / 2);
    };
    auto load_b = [&](int half, int stage) {
        const uint32_t src = b_src + half * 256u, dst = lds_wave + stage + OPERAND_TILE_BYTES + half * HALF_TILE_BYTES;
        load_to_lds(Bop, b_lane, src, dst);
        load_to_lds(Bop, b_lane, src + b_second, dst + HALF_TILE_BYTES / 2);
    };

    // The prefetch cursor runs PREFETCH_STEPS k-steps ahead of the loads.  Line L of the 256 lines of a tile's k-step:
    // columns 64 (L % 4) .. + 63 of k-row L / 4.  This workgroup touches one of `share.count` parts of them, wave w an
    // eighth of that, one load of 4 bytes for all (lanes share lines).
    uint32_t p_src = 0, p_inc = 0, p_lane = 0;
    int p_round = 0, p_left = 0;
    auto prefetch_tile = [&](int round) {
        const StreamTile t = tile_at(round);
        const uint32_t k = t.descending ? (uint32_t)(k_steps - 1) : 0u;
        p_src = (uint32_t)t.n0 * 2u + k * b_step;
        p_inc = t.descending ? 0u - b_step : b_step;
        p_left = k_steps;
    };
    auto prefetch_next = [&]() {
        p_src += p_inc;
        if (--p_left == 0) {
            if (p_round < rounds - 1) ++p_round;
            prefetch_tile(p_round);
        }
    };
    if (PREFETCH) {
        const int per_wave = 32 / share.count;
        const int line = (8 * share.index + wave) * per_wave + (lane & (per_wave - 1));
        p_lane = ((uint32_t)(line >> 2) * Bop.ld + (uint32_t)(64 * (line & 3))) * 2u;
        prefetch_tile(0);
        for (int j = 0; j < 2 + PREFETCH_STEPS; ++j) prefetch_next();
    }
    // The bytes go to the part of A half 1 that this wave's next load_a(1, stage) overwrites: a wave's loads return in the
    // order in which they were issued.
    auto prefetch = [&](int stage) {
        if (!PREFETCH) return;
        touch_line(Bop, p_lane, p_src, lds_wave + stage + HALF_TILE_BYTES);
        prefetch_next();
    };

    const FragReader<KS, RATE == 2> frag(wm, wn, i, g);
    bf16x8 af[MT / 2][2], bf0[NT / 2][2], bf1[NT / 2][2];
    acc_t acc;

    int cur = 0;                                         // stage of the k-step being multiplied
    cursor_tile(0);
    load_b(0, 0); load_a(0, 0); load_b(1, 0); load_a(1, 0);
    cursor_next();
    load_b(0, STAGE_BYTES); load_a(0, STAGE_BYTES); load_b(1, STAGE_BYTES); load_a(1, STAGE_BYTES);
    cursor_next();
    wait_counts<0, NO_LG_WAIT>();                        // the first phases' waits count stores that are not there yet
    raw_barrier();
    frag.read_b(bf0, lds, 0, 0);
    wait_counts<NO_VM_WAIT, 0>();
    raw_barrier();
    if (wm == 1) raw_barrier();                          // the second half of the waves falls one slot behind

    auto step = [&](auto which) {
        constexpr int V = decltype(which)::value;
        constexpr bool FIRST = V == FIRST_STEP, LAST = V == LAST_STEP;
        constexpr int P = PREFETCH;
        constexpr int WAITING = FIRST || LAST ? 9 : 4;
        const int nxt = STAGE_BYTES - cur;
        auto stores = [&](auto phase) {
#pragma unroll
            for (int n = 0; n < stream_stores(RATE, V, decltype(phase)::value); ++n) epi.template store<WAITING>();
        };
        // phase 0
        frag.read_a(af, lds, 0, cur);
        if constexpr (FIRST) epi.template fetch<2>();
        stores(std::integral_constant<int, 0>());
        if constexpr (FIRST) epi.template finish<3>(acc);
        load_b(0, cur);
        wait_counts<12 + 2 * P + stream_window_stores(RATE, V, 0), 0>();
        raw_barrier();
        quadrant_mfmas<0, FIRST>(acc, af, bf0);
        raw_barrier();
        // phase 1
        frag.read_b(bf1, lds, 1, cur);
        if constexpr (FIRST) epi.begin_next();
        stores(std::integral_constant<int, 1>());
        if constexpr (LAST) epi.template finish<0>(acc);
        if constexpr (FIRST && RATE == 4) epi.template fetch<3>();
        load_a(0, cur);
        wait_counts<12 + P + stream_window_stores(RATE, V, 1), 0>();
        raw_barrier();
        quadrant_mfmas<1, FIRST>(acc, af, bf1);
        raw_barrier();
        // phase 2
        frag.read_a(af, lds, 1, cur);
        if constexpr (LAST) epi.template fetch<0>();
        stores(std::integral_constant<int, 2>());
        if constexpr (LAST) epi.template finish<1>(acc);
        load_b(1, cur);
        wait_counts<12 + P + stream_window_stores(RATE, V, 2), 0>();
        raw_barrier();
        quadrant_mfmas<2, FIRST>(acc, af, bf0);
        raw_barrier();
        // phase 3
        frag.read_b(bf0, lds, 0, nxt);
        if constexpr (LAST) epi.template fetch<1>();
        stores(std::integral_constant<int, 3>());
        if constexpr (LAST) epi.template finish<2>(acc);
        if constexpr (V == FETCH_STEP) epi.template fetch<3>();
        prefetch(cur);
        load_a(1, cur);
        cursor_next();
        wait_counts<12 + 2 * P + stream_window_stores(RATE, V, 3), 0>();
        raw_barrier();
        quadrant_mfmas<3, FIRST>(acc, af, bf1);
        raw_barrier();
        cur = nxt;
    };
    for (int r = 0; r < rounds; ++r) {
        step(std::integral_constant<int, FIRST_STEP>());
        step(std::integral_constant<int, SECOND_STEP>());
        if constexpr (RATE == 1)
            for (int j = 0; j < 2; ++j) step(std::integral_constant<int, STORE_STEP>());
        if constexpr (RATE != 4) {
            step(std::integral_constant<int, FETCH_STEP>());
            for (int j = 0; j < 4 / RATE; ++j) step(std::integral_constant<int, STORE_STEP>());
        }
        for (int j = RATE == 1 ? 10 : RATE == 2 ? 6 : 3; j < k_steps; ++j) step(std::integral_constant<int, PLAIN_STEP>());
        step(std::integral_constant<int, LAST_STEP>());
    }
    if (wm == 0) raw_barrier();
    epi.template fetch<2>();
#pragma unroll
    for (int n = 0; n < (RATE == 4 ? 4 : 9); ++n) epi.template store<9>();
    epi.template finish<3>(acc);
    epi.template fetch<3>();
#pragma unroll
    for (int n = 0; n < (RATE == 4 ? 8 : 4); ++n) epi.template store<9>();
    wait_counts<0, 0>();                                 // the loads past the last tile write LDS
}

// Finished quadrants leave as bf16 rows out[n][m] (m = the A rows of the tile, n = its B columns).  A quadrant of a
// wave is 32 rows n of 64 columns m; it passes through the wave's own 4 KiB of LDS so that eight consecutive lanes
// store one whole 128-byte line (stored from the accumulator layout, where a line's pieces sit in lanes 16 apart,
// the dW kernel took 394 us at B = 1024, D = 2048, C = 100 000 through the cache and 552 us past it, against 383
// and 376 with whole lines and the same schedule).  16-byte chunks are XOR-ed with n & 7.  Store s (0 .. 15) of a
// tile is rows 8 i .. + 7 of quadrant q, s = 4 q + i.
struct RowStoreTile {
    uint16_t* base;                      // element (0, 0) of the tile
    uint32_t records;                    // bytes from there to the end of the matrix: rows beyond it are dropped
    int m_valid;                         // columns of the matrix from there (a multiple of 64)
};
template <int RATE>
struct RowStore {
    static constexpr int QUEUE = 9;
    u32x4 queue[QUEUE];                  // fetched values, oldest first
    RowStoreTile at;
    uint32_t lane_off, ld;
    int next = 16;                       // next store of the tile
    int wm;
    char* lds;
    int wr[2], rd;                       // LDS offsets
    __device__ __forceinline__ void init(int64_t ld_elems, char* lds_base) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int scratch = LDS_BYTES + STREAM_SCRATCH_BYTES * wave;
        lds = lds_base;
        wm = wave >> 2;
        ld = (uint32_t)ld_elems;
        at = RowStoreTile{nullptr, 0, 0};
#pragma unroll
        for (int k = 0; k < QUEUE; ++k) queue[k] = u32x4{0, 0, 0, 0};
        const int n = lane >> 3, chunk = lane & 7;       // row of the eight, 16-byte chunk of the line
        rd = scratch + n * 128 + ((chunk ^ n) << 4);
        lane_off = ((uint32_t)(wave_col<KS>(wave & 3, 0) + n) * ld + (uint32_t)(WAVE_M * wm + 8 * chunk)) * 2u;
#pragma unroll
        for (int u = 0; u < 2; ++u) wr[u] = scratch + (lane & 15) * 128 + (((4 * u + (lane >> 4)) ^ (lane & 7)) << 4);
    }
    template <int Q>
    __device__ __forceinline__ void put(const acc_t& acc) {
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const f32x4 lo = acc[4 * (Q >> 1) + 2 * u][2 * (Q & 1) + y], hi = acc[4 * (Q >> 1) + 2 * u + 1][2 * (Q & 1) + y];
                const u32x4 v = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
                // chunk 4 u + g of row 16 y + lane % 16
                *reinterpret_cast<u32x4*>(lds + wr[u] + y * 2048) = v;
            }
    }
    // Where the four values of quadrant Q go in the queue: behind those not yet stored (see stream_stores).
    template <int Q>
    __device__ __forceinline__ void fetch() {
        constexpr int AT = Q == 0 ? 0 : RATE == 4 ? (Q == 1 ? 2 : 4) : Q == 1 ? 3 : Q == 2 ? 5 : 0;
        static_assert(AT + 4 <= QUEUE, "");
#pragma unroll
        for (int i = 0; i < 4; ++i) queue[AT + i] = *reinterpret_cast<const u32x4*>(lds + rd + i * 1024);
        if (Q == 0) next = 0;
    }
    template <int WAITING>
    __device__ __forceinline__ void store() {
        const int q = next >> 2;
        const uint32_t soff = ((uint32_t)(wave_col<KS>(0, 2 * (q & 1)) + 8 * (next & 3)) * ld + (uint32_t)(64 * (q >> 1))) * 2u;
        // no records, nothing in range whatever the offsets (make_operand): a store without effect
        const bool live = next < 16 && WAVE_M * wm + 64 * (q >> 1) < at.m_valid;
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(at.base, 0, live ? (int)at.records : 0, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b128(queue[0], r, (int)lane_off, (int)soff, 2);      // non-temporal
        ++next;
#pragma unroll
        for (int k = 0; k < WAITING - 1; ++k) queue[k] = queue[k + 1];
    }
};

}  // namespace ws
