// What the fused convolution's panel decoder does with addresses and positions in plain arithmetic (internal to the
// library; host code too, so that it can be checked without a GPU).
#ifndef ANSZP_PANEL_H
#define ANSZP_PANEL_H

#include <stdint.h>

#if defined(__HIPCC__)
#define ANSZP_PANEL_HD __host__ __device__ inline
#else
#define ANSZP_PANEL_HD inline
#endif

constexpr uint32_t kPanelWaves = 12;        // wavefronts that decode a panel
constexpr uint32_t kStageWords = 384;       // per wavefront: LDS room for one chunk's compressed words (2.6 bit per
                                            // weight at 4608 symbols; a larger chunk is read from global memory)
constexpr uint32_t kStageBytes = kPanelWaves * kStageWords * 4u;     // at the start of LDS; the table's entries follow
constexpr uint32_t kLeastLds = 65536u;      // every launch asks for at least this much LDS

// The staged words of a chunk lie in [0, kStageBytes), the first one at the highest address.  With `left` = 8 * address of
// the end of the wavefront's room - 32 - bits read, the next 32 bits are in the word at this address and the one behind
// it.  Valid streams stay inside the room; a corrupt one may count on below zero: the mask leaves every address it can
// reach, and the word behind it, in LDS that is there.
constexpr uint32_t kStageMask = 0x7FFCu;
ANSZP_PANEL_HD uint32_t stage_address(uint32_t left) { return (left >> 3) & kStageMask; }
static_assert(kStageBytes <= kStageMask + 4u && kStageMask + 8u <= kLeastLds, "all of the room is reached, and nothing outside LDS");

// The row of a chunk's element `pos`, pos / K, as one 24-bit multiplication: the upper 32 of the 48 bits of
// (pos << shift) * magic, magic = floor(2^(32 - shift) / K) + 1.  Both factors must be below 2^24 and the error
// pos * (magic * K - 2^(32 - shift)) <= pos * K below 2^(32 - shift): K >= 257 takes shift 0 (pos * K < 2^32), 2 <= K <= 256
// shift 8 (pos < 2^16, pos * K < 2^24), K = 1 shift 9 and 2^23 exactly (pos < 2^15).  A chunk has at most 16 rows, and a
// look-up may step past its end by eight symbols of each of 64 streams: pos < 16 K + 512, within all three.
// (With 2^24 for every K, chunks of 4 rows of 2304 or 16 of 1152 were beyond it and read their words from global memory: a
// call of 256 x 2304 weights on sixteen 7 x 7 images took 13.4 us, 11.8 staged; 256 x 1152 in chunks of 16 rows 15.4, 12.3.)
struct RowReciprocal {
    uint32_t magic, shift;
};
ANSZP_PANEL_HD RowReciprocal row_reciprocal(uint32_t K) {
    RowReciprocal r;
    r.shift = K >= 257u ? 0u : K >= 2u ? 8u : 9u;
    r.magic = K >= 2u ? uint32_t((uint64_t(1) << (32u - r.shift)) / K) + 1u : 1u << 23;
    return r;
}

#endif
