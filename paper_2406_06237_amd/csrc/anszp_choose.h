// Which kernel decodes a call (internal to the library; host code only, so that a test can look at it without a GPU), and what of
// the kernels' geometries that depends on.
#ifndef ANSZP_CHOOSE_H
#define ANSZP_CHOOSE_H

#include <cstdint>
#include <initializer_list>

#include "anszp.h"
#include "anszp_layout.h"

constexpr uint32_t kBlockLookups = 8u;         // look-ups a lane makes per block of the look-ahead kernel

// LDS geometry of the look-ahead kernel.  The large one takes tables of up to 2^12 states (64 KiB of
// look-ahead entries) and two chunks of a layer per workgroup, one workgroup per CU; the small one (tables
// of up to 2^11 states, shorter windows) leaves room for two workgroups per CU.
struct LargeLds {
    static constexpr uint32_t kTableLog = ANSZP_MAX_TABLE_LOG, kPayloadWords = 4096u, kRingElems = 16u * 1024u;
    static constexpr uint32_t kLogSlots = 8u, kWorkgroupsPerCu = 1u, kTag = 1u;
    static constexpr uint32_t kSoloWords = 11672u;         // of a chunk that has a workgroup to itself
};
struct SmallLds {
    static constexpr uint32_t kTableLog = 11u, kPayloadWords = 2048u, kRingElems = 8u * 1024u;
    static constexpr uint32_t kLogSlots = 4u, kWorkgroupsPerCu = 2u, kTag = 2u;
    static constexpr uint32_t kSoloWords = 5912u;
};

constexpr uint32_t kWavesLds = 160u * 1024u - 64u;
constexpr uint32_t kWavesCtl = 64u;                        // behind the table: what the wavefronts of a run share
constexpr uint32_t kWavesPad = 16u;                        // words beside a chunk's: four before, zeros behind (see kSplitPad)
constexpr uint32_t kWavesBehind = kLookaheadMaxSymbols * ANSZP_MAX_STREAMS + 16u;      // bytes behind the buffer
constexpr uint32_t kWavesRoom = 2048u, kWavesLeastRoom = 512u;    // symbols in the buffer beside a mean chunk's words; beside any chunk's

// Wavefronts per workgroup and the LDS each has for a chunk's words and the buffer (waves == 0: not a launch for this
// kernel).  As many wavefronts as leave room for a quarter more words than the mean chunk has beside kWavesRoom
// symbols; chunks of up to a good deal more still fit, with a shorter buffer.
// What a chunk costs counts as its words and `fixed` (a chunk without words takes about as long as two words a stream do),
// in units of which the mean chunk has 32 (unit_scale / 2^16 units a word); staging a layer's table counts as stage_units.
struct WavesShape { uint32_t waves, own, mean, fixed, unit_scale, stage_units; };
inline WavesShape waves_shape(uint32_t table_log, uint32_t n_streams, uint64_t mean_words) {
    for (uint32_t waves : {16u, 12u, 8u}) {
        if (table_log == ANSZP_MAX_TABLE_LOG && waves == 16u) continue;
        const uint32_t own = (kWavesLds - (16u << table_log) - kWavesCtl) / waves & ~15u;
        if (4u * (mean_words * 5u / 4u + 16u + kWavesPad) + kWavesRoom + kWavesBehind > own) continue;
        const uint32_t mean = static_cast<uint32_t>(mean_words), fixed = 2u * n_streams;
        // (4 us for a table of 2^12 states; a chunk's words and `fixed` take 0.87 us for each word of a stream, `waves` of them at once)
        return WavesShape{waves, own, mean, fixed, (32u << 16) / (mean + fixed), (147u * waves * n_streams >> (ANSZP_MAX_TABLE_LOG - table_log)) / (mean + fixed)};
    }
    return WavesShape{0u, 0u, 0u, 0u, 0u, 0u};
}

constexpr uint32_t kSplitWords = 11096u;                  // longest stream decode_split takes (what the look-ahead kernel can hold)
constexpr uint32_t kSplitMinBits = 2048u;

constexpr uint32_t kFewMostPerCu = 4u;
// LDS of a workgroup of which so many are to fit a CU, which gives it out in pieces of 1,280 bytes (a third of it all, 54,613 bytes, would be
// given 55,040, and two workgroups fit: 700 chunks of 8,192 symbols, 2^10 states, 11.3 us, 8.1 with three)
constexpr uint32_t kLdsPiece = 1280u;
constexpr uint32_t few_lds(uint32_t per_cu) { return 160u * 1024u / per_cu / kLdsPiece * kLdsPiece - 64u; }
static_assert(few_lds(3u) % 16u == 0u && 3u * ((few_lds(3u) + kLdsPiece - 1u) / kLdsPiece * kLdsPiece) <= 160u * 1024u, "three fit");
constexpr uint32_t kFewLeastRoom = 2048u;                  // symbols in each of two buffers
// Words of a chunk that fit beside table and buffers in `lds` bytes (negative: not even those do).
constexpr int32_t few_words(uint32_t lds, uint32_t table_log) {
    return (int32_t(lds) - int32_t(16u << table_log) - 2 * int32_t(kFewLeastRoom + kWavesBehind) - 16) / 4 - int32_t(kWavesPad);
}

// few: workgroups of decode_few on a CU, or 0
struct LaunchChoice { bool stepwise, byte_table, shared, streaming, small, per_channel, split; uint32_t few; WavesShape waves; };

// a: checked, with chunks and tables.
inline LaunchChoice choose_kernel(const anszp_decode_args_t& a, int mode, bool planned, uint32_t cus) {
    LaunchChoice k;
    // chunks whose compressed words cannot fit the look-ahead kernel's LDS window would all take its
    // fallback: they go to the streaming kernel, whatever their number (measured on 772 to 24,704
    // chunks of 82 KB of words: 5 to 7 times faster than one step-wise wavefront per chunk)
    const uint64_t mean_words = a.payload_words / a.n_chunks;
    k.stepwise = mode == 1 || mode == 3 || mode == 4 || (mode == 0 && mean_words > LargeLds::kPayloadWords);
    k.byte_table = mode == 5;
    k.shared = mode == 3;
    k.streaming = mode == 4 || (mode == 0 && k.stepwise);
    // small tables and short chunks: the variant that fits two workgroups on a CU
    k.small = a.table_log <= SmallLds::kTableLog && 2u * mean_words <= SmallLds::kPayloadWords &&
              kBlockLookups * kLookaheadMaxSymbols * a.n_streams < SmallLds::kRingElems;     // a block must fit its ring
    k.per_channel = a.scales != nullptr && a.n_scales != 0;
    // One stream per chunk: its chain split over a workgroup where the stream is long enough for walks started anywhere
    // to meet it, i.e. as many bits as the table has states and 3,072, or twice as many and 2,048 (2^11 states: 2,048 bits
    // 28.6 us as one chain, 32.0 split; 3,072 bits 40.7 and 28.9; 2^10 states: 2,048 bits 28.2 and 18.6), and either the
    // chunks leave CUs idle otherwise or a chain is so long that four chunks at once on a CU do not make up for it (600
    // chunks of 11,000 bits 148 us as chains, of 17,000 bits 146 split).  Longer than the kernel can hold: as before (the
    // mean is exact for one chunk; several may differ, then the bound is the look-ahead kernel's).
    const uint64_t bits = 32u * mean_words, states = 1ull << a.table_log;
    k.split = mode == 0 && a.n_streams == 1 && bits >= kSplitMinBits && bits >= states && (bits >= 3072u || bits >= 2u * states) &&
              mean_words <= (a.n_chunks == 1 ? kSplitWords : LargeLds::kPayloadWords) &&
              (a.n_chunks <= cus || bits >= 16384u);
    if (k.split) k.stepwise = k.streaming = false;
    // More chunks than the look-ahead kernel decodes at once (two per workgroup): a wavefront per chunk and a table staged
    // once per workgroup and layer, where the chunks' words fit and there are chunks enough for a workgroup's share to be of
    // few layers (24 a layer where only eight wavefronts fit a CU: 130 layers of 12 chunks of 1,600 words 70 us, 84 this way).
    // Up to four chunks per CU only short ones, and with a plan, which spares the look-ahead kernel its search, fewer still.
    // 16 layers of 544 to 992 chunks, layers in a row and descriptors in any order, times as fast as the look-ahead kernel:
    //   2^12 states, without a plan                  1.4 to 3.4 (few streams or 65,536 symbols 1.0 to 1.6)     1.3 to 2.4 (1.0)
    //   2^12 states, with one, up to 480 bits a stream    1.1 to 1.8 (once 0.91)      1.04 to 1.9
    //     more bits or more than 8,192 symbols       0.72 to 1.4                      0.72 to 2
    //   small geometry, without, up to 512 bits and symbols a stream     1.2 to 2.4   1.04 to 1.6
    //     longer streams                             0.72 to 1.3                      0.9 to 1.5
    //   small geometry, with one, more than three chunks per CU of up to 240 bits and 256 symbols a stream     0.98 to 1.3   0.86 to 1
    //     others                                     0.68 to 1.25                     0.67 to 1.2
    // 1,120 chunks: 0.96 to 2 but for 1,870 bits a stream with a plan in the small geometry, 0.77.
    k.waves = WavesShape{};
    const uint64_t per_layer = a.n_chunks / a.n_tables, N = a.n_streams, symbols = a.out_elems / a.n_chunks;
    const bool short_enough = a.n_chunks > 4u * cus ? !(planned && k.small && a.n_chunks <= 6u * cus && bits > 1024u * N)
                              : k.small              ? mean_words <= 256u && (planned ? a.n_chunks > 3u * cus && bits <= 240u * N && symbols <= 256u * N
                                                                                      : bits <= 512u * N && symbols <= 512u * N)
                                                     : mean_words <= 450u && (!planned || (bits <= 480u * N && symbols <= 8192u));
    if (mode == 0 && !k.stepwise && !k.split && per_layer >= 8u && a.n_chunks > 2u * cus && short_enough) {
        k.waves = waves_shape(a.table_log, a.n_streams, mean_words);
        if (k.waves.waves == 8u && per_layer < 24u) k.waves.waves = 0u;
    }
    // Few chunks: a workgroup per chunk that stages and walks, and stores behind the walk or a window later (decode_few), as many on a
    // CU as there are chunks for it and LDS for.  It starts 1.5 to 2 us earlier than the look-ahead kernel and takes 5 ns a look-up
    // longer.  64 streams, bf16, look-ahead kernel with a plan -> here, equal chunks of 2,048 / 8,192 / 16,384 / 32,768 / 65,536 symbols:
    // (2^12 states, 2.2 bits; 24 of them) 7.2 / 10.9 / 16.2 / 26.2 / 89 -> 5.5 / 9.2 / 14.4 / 24.1 / 44; (2^12 states, mostly dominant; 249)
    // 6.8 / 8.2 / 9.4 / 11.9 / 16.8 -> 5.0 / 6.2 / 7.9 / 10.7 / 16.6, as fp32 (99) 6.8 / 8.0 / 9.4 / 12.0 / 16.8 -> 4.9 / 6.4 / 8.3 / 11.3 /
    // 17.0; (2^10 states, 1.2 bits; 499, two on a CU) 8.5 / 10.4 / 12.3 / 27 / 42 -> 5.3 / 7.2 / 9.7 / 14.8 / 24.8.  Without a plan 0.4 us
    // more are saved.  Three and four on a CU without a plan only: 700 and 1,000 of 2,048 to 16,384 1.8 to 2.7 times as fast.  The
    // line lies where a kernel that stored nothing before a chunk was walked to its end became the slower one; longer chunks
    // are for the look-ahead kernel, up to twice the mean chunk has to fit LDS whole.  Chunks much longer than their set's mean: see anszp_few.h.
    // The host knows the mean chunk only: a workgroup gets LDS for the longest the look-ahead kernel would decode, and where that
    // leaves fewer of them on a CU than there are chunks, some wait for a CU.  (440 chunks of 2,000 symbols and 20 of 65,536, 1.8 bits,
    // 2^12 states: the look-ahead kernel 41 us, with a plan 30; here 262 where two workgroups were to share a CU and the long chunks'
    // words, which did not fit, were walked in memory, 33 with one.  500 of 3,000: 19 and 14, here 7 with two, 10 with one.)
    k.few = 0u;
    const uint64_t per_cu = (a.n_chunks + cus - 1u) / cus;
    if (mode == 0 && !k.stepwise && !k.split && !k.waves.waves && per_cu <= (planned ? 2u : kFewMostPerCu) && symbols <= 512u * N &&
        symbols <= (a.out_dtype == ANSZP_OUT_F32 ? 12288u : 20480u) &&
        (16ull << a.table_log) + 8u * mean_words + 2u * symbols + kFewLeastRoom <= few_lds(uint32_t(per_cu))) {
        k.few = uint32_t(per_cu);
        while (k.few > 1u && few_words(few_lds(k.few), a.table_log) < int32_t(k.small ? SmallLds::kSoloWords : LargeLds::kSoloWords)) --k.few;
    }
    return k;
}

#endif
