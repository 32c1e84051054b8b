// How conv_sliced_kernel (anszp_conv.hip) is launched for a call (internal to the library; plain host code, so that it
// can be checked without a GPU).
#ifndef ANSZP_CONV_PLAN_H
#define ANSZP_CONV_PLAN_H

#include <stdint.h>

#include <algorithm>

#include "anszp.h"
#include "anszp_panel.h"

constexpr uint32_t kWave = 64;
constexpr uint32_t kThreads = 768;
constexpr uint32_t kWaves = kThreads / kWave;
static_assert(kWaves == kPanelWaves, "the staging room is counted in wavefronts");
constexpr uint32_t kRows = 16;              // output channels per MFMA row tile
constexpr uint32_t kRowPad = 8;             // bytes between panel rows: rows start two LDS banks apart
constexpr uint32_t kWidenPieces = 7;        // 16-byte pieces of a byte panel one thread widens to bf16
constexpr uint32_t kMaxK = 4608;           // reduction length whose 16-row panel (72 KiB) fits LDS beside the table
constexpr uint32_t kLdsLimit = 160u * 1024u;

// How its contraction addresses the activations: 1 x 1; three taps wide, stride 1; three taps wide, any stride.
enum { kPoint = 1, kShift = 2, kRow = 3 };
constexpr uint32_t units_in_flight(uint32_t mr, uint32_t mode, uint32_t qt) { return mode == kRow ? 2u : mr * qt > 8u || mode == kShift ? 3u : 4u; }
// The most column tiles per wavefront the registers hold.
constexpr uint32_t most_tiles(uint32_t mr, uint32_t mode) { return mode == kRow ? (mr == 1u ? 4u : 3u) : mr == 4u ? 3u : 4u; }

// conv_sliced_kernel's row tiles, column tiles, slices and workgroups for a call: the fewest clocks by an estimate.  Its
// constants, all in clocks, are fitted to 843 calls with every choice forced in turn (1 x 1 and three taps wide, 16 to 2048
// channels, images of 5 to 64, batches up to 256, both layouts, 2^12 states; whole calls of 8 to 500 us): the choice is 1.6 %
// slower than the best one on average, more than 10 % for 34 of them, 23 % at worst.  Per turn of workgroups over the CUs:
// Decoding: rounds of chunks over the twelve wavefronts, 2500 and a quarter of a clock per symbol each.  Widening a panel
// of bytes: 6000.  A unit of a wavefront: whichever takes longest of its SIMD's wavefronts' instructions (9 per matrix
// instruction, 12 per step), all wavefronts' panel reads (8), all wavefronts' activation loads (22; NHWC, whose lanes touch
// four times as many lines, 32) and a load's latency over the units in flight (1600).  A round of tiles: 1500, and its
// stores (35 per tile, row tile and output byte; NHWC 105).  Slices: 48 bytes of sums a clock.
//
// Rows: a panel of 16, 32 or 64 output channels, or (plan_half_tile) of half a row tile, 8 of them, whose matrix instructions
// multiply every row twice and store one.  Long rows are worth that where there are few pixels: a panel of 16 x 4608 is sixteen
// chunks, two rounds of decoding, and of bytes, since as bf16 values it does not fit LDS beside the table; half of it is one round
// and needs no widening.  512 x 4608 weights on one 7 x 7 image 12.4 -> 8.4 us.
struct SlicedPlan {
    uint32_t mr = 0, qt = 0, k_groups = 0, round_tiles = 0, slice_units = 0, splits = 0, tiles_per_split = 0, lds_bytes = 0;
    uint32_t rows = 0;                                            // of a panel: 16 per row tile, or 8
    bool p16 = false;
    uint64_t clocks = ~0ull;
};
// `best` or the cheapest plan with panels of `rows` rows.
inline void plan_panels(const anszp_conv_args_t& a, uint32_t mode, uint32_t K, uint32_t row_stride, uint32_t n_tiles, uint32_t cus, uint32_t rows, SlicedPlan& best) {
    const uint32_t table_bytes = 16u << a.table_log, fixed = kStageBytes + table_bytes + 64u;
    const uint32_t taps = mode == kPoint ? 1u : 3u, units = (mode == kPoint ? 1u : a.kh) * ((a.cin + 31u) / 32u);
    const uint32_t mr = rows < kRows ? 1u : rows / kRows;
    if (a.cout % rows || rows % a.rows_per_chunk) return;
    const uint32_t elems = rows * row_stride;
    const bool p16 = fixed + 2u * elems <= kLdsLimit;             // the panel decoded as bf16 values; else as bytes, widened in place
    if (!p16 && (rows < kRows || fixed + elems > kLdsLimit || 2u * (elems + 64u) > kLdsLimit || elems + 64u > kWidenPieces * kThreads * 16u)) return;
    const uint32_t n_mtiles = a.cout / rows, most = most_tiles(mr, mode);
    const uint32_t chunk_rounds = (rows / a.rows_per_chunk + kWaves - 1u) / kWaves;
    const uint64_t decode = chunk_rounds * (2500u + uint64_t(a.rows_per_chunk) * K / 4u) + (p16 ? 0u : 6000u);
    // few, long-lived workgroups, as many as are resident at once (one per CU): each decodes its panel once.  Where the panels
    // do not divide the CUs: a few CUs left over, or a few workgroups that wait for a CU.
    for (uint32_t more = 0; more < 2u; ++more) {
        uint32_t splits = std::max(1u, std::min(cus / n_mtiles + more, n_tiles));
        if (more && (splits * n_mtiles <= cus || cus % n_mtiles == 0u)) break;               // (no more than before, or too many)
        const uint32_t tiles = (n_tiles + splits - 1u) / splits;
        splits = (n_tiles + tiles - 1u) / tiles;
        const uint32_t turns = (n_mtiles * splits + cus - 1u) / cus;                         // (n_mtiles * splits < cus + n_mtiles)
        if (turns * decode >= best.clocks) continue;
        for (const uint32_t ks : {1u, 2u, 3u, 4u, 6u, 12u}) {
            const uint32_t ts = kWaves / ks, rounds = (tiles + most * ts - 1u) / (most * ts);
            const uint32_t per_round = (tiles + rounds - 1u) / rounds, qt = (per_round + ts - 1u) / ts;
            const uint64_t sums = ks > 1u ? uint64_t(kWaves) * qt * mr * 1024u : 0u;
            if (ks > 1u && (rounds > 1u || units < ks || sums > kLdsLimit)) continue;
            const uint32_t busy = (per_round + qt - 1u) / qt * ks, slots = units_in_flight(mr, mode, qt);
            const uint64_t issue = uint64_t((busy + 3u) / 4u) * taps * (9u * qt * mr + 12u), reads = uint64_t(busy) * mr * taps * 8u;
            const uint64_t loads = uint64_t(busy) * (mode == kRow ? 3u * qt : mode == kShift ? qt + 1u : qt) * (a.x_layout == ANSZP_ACT_NHWC ? 32u : 22u);
            const uint64_t unit = std::max(std::max(issue, reads), std::max<uint64_t>(loads, 1600u / slots));
            const uint64_t stores = uint64_t(per_round) * mr * (a.y_dtype == ANSZP_OUT_BF16 ? 70u : 140u) * (a.y_layout == ANSZP_ACT_NHWC ? 3u : 1u);
            const uint64_t clocks = turns * (decode + rounds * ((units + ks - 1u) / ks * unit + 1500u + stores) + sums / 48u);
            if (clocks >= best.clocks) continue;
            best.clocks = clocks;
            best.mr = mr; best.rows = rows; best.p16 = p16; best.qt = qt; best.k_groups = ks; best.round_tiles = per_round;
            best.slice_units = (units + ks - 1u) / ks; best.splits = splits; best.tiles_per_split = tiles;
            best.lds_bytes = std::max(std::max(fixed + elems * (p16 ? 2u : 1u), p16 ? 0u : 2u * (elems + 64u)), uint32_t(sums));
        }
    }
}
inline SlicedPlan plan_sliced(const anszp_conv_args_t& a, uint32_t mode, uint32_t K, uint32_t row_stride, uint32_t n_tiles, uint32_t cus) {
    SlicedPlan best;
    for (const uint32_t mr : {4u, 2u, 1u}) plan_panels(a, mode, K, row_stride, n_tiles, cus, kRows * mr, best);
    return best;                                                  // (one row tile always fits: K <= 4608)
}
// The plan above, or one with panels of half a row tile where that is estimated to take fewer clocks; a fifth fewer where the
// former's panel is one of bytes, whose widening the estimate takes for longer than it is in calls this short.  Of 70 calls for
// which half a tile was the cheaper plan, drawn over the channels and images of a network, the 16 below that line went 0.83 to 1.13
// times as fast (seven of them slower), the 54 others 0.98 to 1.52 times (one slower; geometric mean 1.27).
inline SlicedPlan plan_half_tile(const anszp_conv_args_t& a, uint32_t mode, uint32_t K, uint32_t row_stride, uint32_t n_tiles, uint32_t cus) {
    SlicedPlan best = plan_sliced(a, mode, K, row_stride, n_tiles, cus), half;
    plan_panels(a, mode, K, row_stride, n_tiles, cus, kRows / 2u, half);
    return half.rows && half.clocks + (best.p16 ? 0u : half.clocks / 5u) < best.clocks ? half : best;
}

// How `images` images are convolved: the way a unit's vectors are loaded, and the plan.  The columns of an output row that are
// gone through begin first_column before it.
struct CallPlan { uint32_t mode, first_column, columns; SlicedPlan plan; };
inline CallPlan plan_call(const anszp_conv_args_t& a, uint32_t K, uint32_t row_stride, uint32_t out_h, uint32_t out_w, uint32_t images, uint32_t cus) {
    // (without padding kShift takes two pixels more per row: narrow images are better off with kRow)
    auto plan_of = [&](uint32_t mode) {
        const uint32_t first = mode == kShift && a.pad == 0u ? 1u : 0u, columns = out_w + 2u * first;
        return CallPlan{mode, first, columns, plan_half_tile(a, mode, K, row_stride, (images * out_h * columns + 15u) / 16u, cus)};
    };
    const CallPlan best = plan_of(a.kw != 3 ? kPoint : a.stride == 1 ? kShift : kRow);
    if (!best.first_column) return best;
    const CallPlan by_row = plan_of(kRow);
    return by_row.plan.clocks < best.plan.clocks ? by_row : best;
}

#endif
