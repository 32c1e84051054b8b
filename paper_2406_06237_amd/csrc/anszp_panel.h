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

#endif
