// Fused decode + convolution for gfx950: a conv layer's entropy-coded weights are decoded into LDS
// and consumed there by bf16 MFMA instructions; the decoded weights never reach global memory
// (Sec. II: the weights are to be decoded on their way from memory to the compute units).
//
// The convolution is an implicit GEMM  Y[n, o] = sum_k A[o, k] * B[k, n]  with
//   o = output channel, n = (image, output row, output column), k = (kernel row, kernel column,
//   input channel), input channel innermost,
//   A[o, k] = q - z, the decoded symbol minus the layer's zero-point (Sec. II-B): an integer of at
//   most 8 bits and therefore exact in bf16; the scale multiplies the fp32 sums at the end,
//   B[k, n] = the bf16 activation under kernel tap (r, s) of output pixel n, zero outside the image.
// Activations and outputs are NHWC or in blocks of 8 channels ([batch][channels / 8][h][w][8]); in both
// the 8 consecutive k one lane feeds into an MFMA are 16 contiguous bytes of the activation tensor.  In
// the blocked layout the 16 lanes that hold the same 8 k of 16 neighbouring pixels read 256 contiguous
// bytes, where NHWC makes them read 16 pieces a whole pixel apart.
//
// One workgroup owns a panel of 16 * MR output channels (MR = 4, 2 or 1 row tiles, conv_sliced_kernel also half a one, of
// v_mfma_f32_16x16x32_bf16: as many as fit in LDS) and a range of output pixels.  Phase 1: its twelve
// wavefronts decode the chunks that hold those weight rows, one lane per stream (Sec. II-A, III-B),
// through the table's look-ahead entries (one look-up per run of up to eight symbols) into a
// [16 * MR][K] panel in LDS: symbols as bytes, or, where they fit, the bf16 values q - z.  Phase 2, by
// kind of layer: input channels that are multiples of 8 under 1 x 1 kernels without padding or kernels
// three taps wide (nearly all layers of a network) have conv_sliced_kernel, which also slices the
// reduction over the wavefronts; conv_fused_kernel has the others (see the enumeration in front of it).
// fp32 accumulators; one store of four consecutive output channels per lane, row tile and column tile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>

#include <cstdint>

#include "anszp.h"
#include "anszp_conv_plan.h"
#include "anszp_cus.h"
#include "anszp_layout.h"
#include "anszp_panel.h"

namespace {

constexpr uint32_t kPatchPieces = 4;        // kGenericPatch: 16-byte pieces of the staged rows per thread
constexpr uint32_t kMaxMine = (4u * kRows + kWaves - 1u) / kWaves;   // chunks of a panel one wavefront may have to decode

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) uint32_t words4;
typedef __attribute__((ext_vector_type(2))) uint32_t words2;
typedef words4 __attribute__((aligned(4))) words4_word_aligned;

// n / d for n < 2^31: no division in the kernels, whose code mostly runs once (a division is some 150 bytes of it, and code that runs
// for the first time costs about 85 ns per 64 bytes; some twenty of them a call of conv_fused_kernel: first layers 0.4 to 1.5 us a
// call, 64 x 3 x 7 x 7 on 16 224 x 224 images 20.7 -> 19.7, two of 104 x 104 8.6 -> 8.1; other channel counts 0.2 to 0.9 us).
struct Reciprocal {
    uint32_t magic, shift;
    __device__ __forceinline__ uint32_t operator()(uint32_t n) const { return __umulhi(2u * n, magic) >> shift; }
};

struct ConvParams {
    const uint32_t* tables;
    const anszp_chunk_t* chunks;        // the layer's first chunk
    const uint32_t* stream_hdr;
    const uint32_t* payload;
    const anszp_layer_t* layers;
    const float* scales;
    const uint16_t* x;
    void* y;
    uint32_t* status;
    uint64_t n_stream_hdr, payload_words, n_scales;
    uint32_t layer_id, table_log, n_streams, rows_per_chunk, chunks_per_panel;
    uint32_t in_h, in_w, cin, cout, kh, kw, stride, pad, out_h, out_w;
    // element strides that tell the two activation layouts apart (see anszp_conv_args_t):
    //   x element (image b, pixel i, channel c) = b * in_h*in_w*cin + i * x_pixel + (c / 8) * x_block + c % 8
    //   y element (image b, pixel i, channel o) = b * out_h*out_w*cout + i * y_pixel + (o / 8) * y_block + o % 8
    // NHWC: pixel = channels, block = 8;  blocks of 8 channels: pixel = 8, block = 8 * pixels per image
    uint32_t x_pixel, x_block, y_pixel, y_block;
    uint32_t y_bf16, K, row_stride, n_pixels, n_mtiles;   // n_mtiles: panels of 16 * MR rows
    uint32_t k_magic;                                     // floor(2^32 / K) + 1: i / K = mulhi(i, k_magic) for i * K < 2^32
    RowReciprocal row_of;                                 // the same with 24-bit factors, for all elements of a chunk
    uint32_t panel_off;                                   // first byte of the panel in LDS (behind the table and the staging room)
    uint32_t patch_off;                                   // kGenericPatch: first byte of the staged rows
    uint32_t row_pitch;                                   // kGenericPatch: bytes from one staged image row to the next
    // conv_sliced_kernel: slices of the reduction; wavefronts that share one (k_groups * t_groups = 12) and wave / t_groups =
    // wave * t_groups_inv >> 16; column tiles of a wavefront (the first wave_tiles_rest have one more), of a round; units of a
    // slice; bytes of x and y
    uint32_t k_groups, t_groups, t_groups_inv, wave_tiles, wave_tiles_rest, round_tiles, slice_units, x_bytes, y_bytes;
    uint32_t x_image, y_image;                            // elements of an image
    uint32_t columns, first_column;                       // pixels in a row of them; the one that is the first output column (kShift
                                                          // without padding: 1, with a pixel on either side that has no output)
    // n / d = mulhi(2 n, magic) >> shift for n < 2^31 (d: columns, output rows, panels, blocks of 32 input channels)
    uint32_t columns_magic, columns_shift, out_h_magic, out_h_shift, n_mtiles_magic, n_mtiles_shift, blocks_magic, blocks_shift;
    __device__ __forceinline__ uint32_t n_mtiles_by(uint32_t n) const { return __umulhi(2u * n, n_mtiles_magic) >> n_mtiles_shift; }
    // conv_fused_kernel's: by output columns and rows; by channels and kernel columns (a k's tap and row), kGenericPatch: by pieces of
    // an image row, words of its edges, padded rows of an image
    Reciprocal by_out_w, by_out_h, by_cin, by_kw, by_pieces, by_edges, by_padded_h;
    uint32_t pixels_per_split, block_pixels;              // multiples of 16: the pixels of a workgroup; of one block (<= 64)
};

__device__ __forceinline__ void report(uint32_t* status, uint32_t bits) {
    atomicOr(&status[0], bits);
    atomicAdd(&status[1], 1u);
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
#pragma unroll
    for (int d = 1; d < int(kWave); d <<= 1) v |= __shfl_xor(v, d, kWave);
    return v;
}

// Exclusive prefix sum over the 64 lanes of a wavefront; *total receives the sum.  Data-parallel-primitive
// moves: within rows of 16 lanes by 1, 2, 4 and 8 (lanes without a source add zero), then lane 15 of rows 0
// and 2 to the rows after them, then lane 31 to the upper half.
__device__ __forceinline__ uint32_t wave_exclusive_sum(uint32_t v, uint32_t* total) {
    int x = static_cast<int>(v);
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);      // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);      // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);      // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);      // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2 and 3
    *total = static_cast<uint32_t>(__builtin_amdgcn_readlane(x, kWave - 1));
    return static_cast<uint32_t>(x) - v;
}

// What a wavefront fetches of a chunk before it decodes it: the stream headers (lane k: stream k), the chunk's
// words as two 16-byte pieces per lane (kStageWords words in all) and the up to three words behind the last
// whole piece.
struct ChunkData {
    uint32_t hdr;
    words4 q0, q1;
    uint32_t tail;
};

// A chunk's descriptor as the wavefront uses it (uniform values), checked against the layer and the buffers.
struct ChunkDesc {
    uint32_t n_symbols, payload_words, stream_offset;
    uint64_t payload_offset;
    bool ok, staged;             // staged: the chunk's words (and two zero words behind them) fit the wavefront's LDS room
};

// LDS byte addresses as numbers: a load or store through one is an LDS instruction with the rest of the address in
// its offset field.
template <class T>
__device__ __forceinline__ T lds_load(uint32_t at) { return *reinterpret_cast<const __attribute__((address_space(3))) T*>(static_cast<uintptr_t>(at)); }
template <class T>
__device__ __forceinline__ void lds_store(uint32_t at, T v) { *reinterpret_cast<__attribute__((address_space(3))) T*>(static_cast<uintptr_t>(at)) = v; }

__device__ __forceinline__ uint32_t lds_address(const void* shared) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)shared));
}

// One chunk into the LDS panel: symbol i of the chunk belongs to panel row i / K, column i % K.  One lane per
// stream (Sec. III-B) walks the automaton of Sec. II-A through the table's look-ahead entries (anszp_layout.h):
// one look-up stands for up to eight symbols, all but the last the layer's dominant symbol, which the panel
// already holds everywhere (the caller fills it), so a look-up writes one panel element.  With T the bits the entry
// of index 2X + b consumes, the next index is base + (the next T + 1 stream bits, first bit most significant) and the
// bit position moves on by T.  Returns the lane's error bits.
//
// The chunk's words were fetched into `d` (16-byte loads issued long before) and go to `stage` (LDS, this
// wavefront's own) when they fit, so that the loop waits for no global load; a larger chunk is read word by word
// in place.  What a look-up costs is instructions (three wavefronts share a SIMD) and LDS accesses (twelve share the
// LDS), so the staged words are kept bit-reversed, the first word at the highest address: with c the bits left
// down from there, words c / 32 + 1 and c / 32 funnel-shifted by c mod 32 are the next 32 stream bits, first bit
// on top, and they last for two look-ups (2 * 12 + 1 bits).  16 vector instructions and 2.5 LDS accesses a look-up where
// least significant bits first, a window per look-up and the clamps of every index took 28 and 3.  A wavefront with a SIMD to
// itself, or nearly, is bound by the chain of them: the next entry is asked for after four, and the twelve that place the
// symbols are issued while it is on its way (behind them: 53 layers of a ResNet-50 on 16 images 688 us, 661 so).
// P16: the panel holds bf16 values q - z (two bytes per weight) instead of the symbols q.
template <bool P16>
__device__ uint32_t decode_chunk_to_panel(const ConvParams& p, const ChunkDesc& c, const ChunkData& d, const uint32_t ahead,
                                          uint32_t ahead_mask, const uint32_t stage, const uint32_t rows, uint32_t lane, int32_t zero_point) {
    const uint32_t N = p.n_streams;
    const uint32_t L = 1u << p.table_log;
    const uint32_t X0 = d.hdr & (L - 1u);
    const uint32_t n_words = d.hdr >> 16;
    uint32_t total_words;
    const uint32_t first_word = wave_exclusive_sum(n_words, &total_words);
    uint32_t err = (total_words != c.payload_words) ? ANSZP_ST_BAD_DESC : 0u;

    const uint32_t word_limit = c.payload_words;      // reads beyond the chunk see zeros
    constexpr uint32_t kElem = P16 ? 2u : 1u;
    const uint32_t n = lane < N ? c.n_symbols : 0u;   // a lane without a stream never runs
    const float zf = static_cast<float>(zero_point);
    // (|q - z| <= 255 has at most 8 significant bits: the upper half of its binary32 form is exact)
    auto put = [&](uint32_t where, uint32_t entry) {
        if constexpr (P16) lds_store<uint16_t>(where, static_cast<uint16_t>(__float_as_uint(static_cast<float>((entry >> 16) & 0xFFu) - zf) >> 16));
        else lds_store<uint8_t>(where, static_cast<uint8_t>(entry >> 16));
    };
    // where what lies beyond the chunk goes (an entry that would carry a stream past its end: corrupt data only): the
    // first column of padding behind the chunk's last row
    const uint32_t beyond = rows + ((p.rows_per_chunk - 1u) * p.row_stride + p.K) * kElem;
    // what the checks at a stream's end look at: the position behind its last symbol, index * 8 of the next entry, bits read
    uint32_t ended_at = 0, at = 0, bits_read = 0;
    if (c.staged) {
        // word i at top - 4 - 4 * i
        const uint32_t quads = word_limit >> 2, top = stage + 4u * kStageWords;
        auto reversed = [](words4 q) { return words4{__brev(q.w), __brev(q.z), __brev(q.y), __brev(q.x)}; };
        if (lane < quads) lds_store<words4>(top - 16u - 16u * lane, reversed(d.q0));
        if (lane + kWave < quads) lds_store<words4>(top - 16u - 16u * (lane + kWave), reversed(d.q1));
        const uint32_t tail_at = (quads << 2) + lane;
        if (lane < 3u && tail_at < word_limit) lds_store<uint32_t>(top - 4u - 4u * tail_at, __brev(d.tail));
        if (lane < 2u) lds_store<uint32_t>(top - 4u - 4u * (word_limit + lane), 0u);     // what a stream reads beyond the chunk
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // LDS serves a wavefront's accesses in order
        __builtin_amdgcn_wave_barrier();
        // b bits into the chunk the next 32 bits, first bit on top, are the two words at and above (left / 32) * 4, funnel-
        // shifted by left mod 32, with left = 8 * top - 32 - b (anszp_panel.h)
        const uint32_t begin = 8u * top - 32u - 32u * min(first_word, word_limit);
        uint32_t left = begin;
        at = ((2u * X0 + (lds_load<uint32_t>(stage_address(begin)) >> 31)) * 8u) & ahead_mask;     // entry 2 X0 + first stream bit
        auto walk = [&](auto one_row) {
            // one row: positions are LDS addresses; several: elements of the chunk, put in their row by a division
            constexpr bool kOneRow = decltype(one_row)::value;
            const uint32_t step = kOneRow ? N * kElem : N;
            const uint32_t end = kOneRow ? rows + n * kElem : n;
            uint32_t pos = kOneRow ? rows + lane * kElem : lane;
            const uint32_t gap = (p.row_stride - p.K) * kElem;
            auto advance = [&](uint32_t window, words2 e) {          // to the next entry; returns the bits consumed
                const uint32_t v = window >> (e.x & 31u);            // the next T + 1 stream bits
                at = (e.y + 8u * v) & ahead_mask;
                const uint32_t T = (e.x >> 24) & 15u;
                left -= T;
                return T;
            };
            auto place = [&](uint32_t entry) {                       // the entry's symbols
                pos = __umul24((entry >> 28) & 7u, step) + pos;      // past its dominant ones
                uint32_t where = pos;
                if constexpr (!kOneRow) {
                    uint32_t row;                                    // pos / K (anszp_panel.h)
                    asm("v_mul_hi_u32_u24 %0, %2, %1" : "=v"(row) : "v"(pos << p.row_of.shift), "s"(p.row_of.magic));
                    where = __umul24(row, gap) + (pos * kElem + rows);
                }
                put(min(where, beyond), entry);
                pos += step;
            };
            // The next entry (and, every second time, the next window's words) is asked for as soon as its index is known, and the
            // symbols of the one at hand are placed while it is on its way: what a stream's end leaves asked for is not used.
            if (pos < end) {
                words2 e = lds_load<words2>(ahead + at);
                uint32_t word = stage_address(left);
                uint32_t lo = lds_load<uint32_t>(word), hi = lds_load<uint32_t>(word + 4u);
                do {
                    const uint32_t window = __builtin_amdgcn_alignbit(hi, lo, left);
                    const uint32_t T = advance(window, e);
                    const words2 second = lds_load<words2>(ahead + at);
                    __builtin_amdgcn_sched_barrier(0);
                    place(e.x);
                    if (pos < end) {
                        advance(window << T, second);
                        e = lds_load<words2>(ahead + at);
                        word = stage_address(left);
                        lo = lds_load<uint32_t>(word);
                        hi = lds_load<uint32_t>(word + 4u);
                        __builtin_amdgcn_sched_barrier(0);
                        place(second.x);
                    }
                } while (pos < end);
            }
            ended_at = kOneRow ? (pos - rows) / kElem : pos;
        };
        if (p.rows_per_chunk == 1u) walk(std::true_type{});
        else walk(std::false_type{});
        bits_read = begin - left;
    } else {
        const uint32_t* words = p.payload + c.payload_offset;
        auto word_at = [&](uint32_t i) { return i < word_limit ? words[i] : 0u; };
        uint32_t bit = first_word << 5, elem = lane;
        at = ((2u * X0 + (word_at(min(first_word, word_limit)) & 1u)) * 8u) & ahead_mask;
        while (elem < n) {
            const uint32_t wi = min(bit >> 5, word_limit);
            const words2 e = lds_load<words2>(ahead + at);
            const uint32_t window = __builtin_amdgcn_alignbit(word_at(wi + 1u), word_at(wi), bit);
            at = (e.y + 8u * (__brev(window) >> (e.x & 31u))) & ahead_mask;
            bit += (e.x >> 24) & 15u;
            elem += ((e.x >> 28) & 7u) * N;
            const uint32_t row = p.K > 1u ? __umulhi(elem, p.k_magic) : elem;
            put(min(rows + (row * (p.row_stride - p.K) + elem) * kElem, beyond), e.x);
            elem += N;
        }
        ended_at = elem;
        bits_read = bit - (first_word << 5);
    }
    // a stream ends where an entry ends, in state 0 (the index of the next entry is 2 X + peeked bit),
    // having read exactly its words
    if (lane < N) {
        // the lane's elements are lane, lane + N, ...: it has produced exactly its symbols if it stands on the
        // first of them that is no element of the chunk
        if (ended_at - c.n_symbols >= N) err |= ANSZP_ST_BAD_LENGTH;
        if ((at >> 4) != 0u) err |= ANSZP_ST_BAD_STATE;
        if ((bits_read + 31u) >> 5 != n_words) err |= ANSZP_ST_BAD_LENGTH;
    }
    return err;                                       // this lane's
}

// Eight symbols -> eight bf16 values q - z.  |q - z| <= 255 has at most 8 significant bits, so the
// upper half of its binary32 form is the exact bf16 value.
__device__ __forceinline__ bf16x8 weights_of(words2 q, float z) {
    auto byte = [](uint32_t w, uint32_t i) { return static_cast<float>((w >> (8u * i)) & 0xFFu); };   // v_cvt_f32_ubyte<i>
    const float f0 = byte(q.x, 0) - z, f1 = byte(q.x, 1) - z, f2 = byte(q.x, 2) - z, f3 = byte(q.x, 3) - z;
    const float f4 = byte(q.y, 0) - z, f5 = byte(q.y, 1) - z, f6 = byte(q.y, 2) - z, f7 = byte(q.y, 3) - z;
    auto pack = [](float lo, float hi) {              // upper halves of two binary32 values, lo in bits 0..15
        return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
    };
    words4 w = {pack(f0, f1), pack(f2, f3), pack(f4, f5), pack(f6, f7)};
    return __builtin_bit_cast(bf16x8, w);
}

// The accumulators of one block of up to 64 pixels times the scale(s), to y.  D operand layout: lane holds
// column lane % 16, rows 4 * (lane / 16) + 0..3 of each row tile: four consecutive output channels.
template <uint32_t MR>
__device__ __forceinline__ void store_tiles(const ConvParams& p, const anszp_layer_t& lay, uint32_t mtile, uint32_t kg,
                                            const floatx4 (&acc)[MR][4], const bool (&valid)[4], const uint32_t (&out_at)[4]) {
    const bool per_channel = lay.channel_len != 0;
#pragma unroll
    for (uint32_t m = 0; m < MR; ++m) {
        const uint32_t o = (mtile * MR + m) * kRows + 4u * kg;
        float sc[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            sc[i] = lay.scale;
            if (per_channel) {
                const uint64_t ch = lay.scales_offset + o + i;
                sc[i] = ch < p.n_scales ? p.scales[ch] : 0.0f;
            }
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            if (valid[q]) {
                const floatx4 out = {acc[m][q][0] * sc[0], acc[m][q][1] * sc[1], acc[m][q][2] * sc[2], acc[m][q][3] * sc[3]};
                const uint32_t at = out_at[q] + (o >> 3) * p.y_block + (o & 7u);
                if (p.y_bf16) {                                   // round to nearest even (v_cvt_pk_bf16_f32)
                    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
                    const bf16x4 r = {static_cast<__bf16>(out[0]), static_cast<__bf16>(out[1]),
                                      static_cast<__bf16>(out[2]), static_cast<__bf16>(out[3])};
                    *reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(p.y) + at) = r;
                } else {
                    *reinterpret_cast<floatx4*>(static_cast<float*>(p.y) + at) = out;
                }
            }
        }
    }
}

// What a kernel tap outside the image reads (kTapsRing: every load is unconditional).
__device__ __attribute__((aligned(64))) const uint32_t zero_page[16] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};

// kTapsRing: the loads of one ring slot (QT activation vectors) issued by hand, and the wait for them.  When a
// slot is used, LATER loads have been asked for after its own, so the wait is for all but LATER loads; it names the
// slot's registers as its results, so that nothing which uses them can be moved ahead of it.  (The compiler, left
// to count loads that cross the loop's back edge, waits for every load at the head of the loop.)
template <uint32_t QT>
__device__ __forceinline__ void ring_request(words4 (&slot)[QT], const uint16_t* const (&from)[QT]) {
#pragma unroll
    for (uint32_t q = 0; q < QT; ++q) asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(slot[q]) : "v"(from[q]) : "memory");
}
template <uint32_t QT, uint32_t LATER>
__device__ __forceinline__ void ring_arrived(words4 (&slot)[QT]) {
    static_assert(QT >= 1 && QT <= 4 && LATER < 64, "one to four vectors per slot; the counter has six bits");
    if constexpr (QT == 1) asm volatile("s_waitcnt vmcnt(%1)" : "+v"(slot[0]) : "n"(LATER) : "memory");
    if constexpr (QT == 2) asm volatile("s_waitcnt vmcnt(%2)" : "+v"(slot[0]), "+v"(slot[1]) : "n"(LATER) : "memory");
    if constexpr (QT == 3) asm volatile("s_waitcnt vmcnt(%3)" : "+v"(slot[0]), "+v"(slot[1]), "+v"(slot[2]) : "n"(LATER) : "memory");
    if constexpr (QT == 4) asm volatile("s_waitcnt vmcnt(%4)" : "+v"(slot[0]), "+v"(slot[1]), "+v"(slot[2]), "+v"(slot[3]) : "n"(LATER) : "memory");
}

// The panel and the range of pixels of this workgroup.
// The chip hands consecutive workgroups to its eight dies in turn and every die has its own L2: workgroup
// blockIdx.x is the (blockIdx.x / 8)-th of die blockIdx.x % 8.  Numbering the workgroups die after die, the
// panels of one range of pixels follow each other on one die, whose L2 then fetches those activations once
// for all of them.  (Any one-to-one numbering is correct; this one is for the cache.)
__device__ __forceinline__ uint32_t unit_of_workgroup() {
    constexpr uint32_t kDies = 8;
    const uint32_t per_die = gridDim.x / kDies, extra = gridDim.x % kDies, die = blockIdx.x % kDies;
    return die * per_die + min(die, extra) + blockIdx.x / kDies;
}

// Phase 1: panel `mtile` (ROWS weight rows) into LDS; the caller's barrier follows.  meanwhile(): called while the
// first loads are on their way.  Returns the layer's quantizer.
template <uint32_t ROWS, bool P16, class MEANWHILE>
__device__ __forceinline__ anszp_layer_t decode_panel(const ConvParams& p, uint8_t* lds, uint32_t mtile, MEANWHILE&& meanwhile) {
    const uint32_t L = 1u << p.table_log;
    const uint32_t ahead_bytes = 16u * L;                         // 2 L look-ahead entries of two words
    uint8_t* ahead = lds + kStageBytes;
    uint8_t* panel = lds + p.panel_off;
    constexpr uint32_t kElem = P16 ? 2u : 1u;                     // bytes per panel element
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // ---- phase 1: the layer's look-ahead entries into LDS, then this workgroup's weight rows.
    // Every global read that depends only on the kernel's arguments is issued before any is waited for: the
    // descriptors of this wavefront's chunks (lane i: its i-th chunk, panel chunk wave + i * kWaves), the layer's
    // quantizer, the triple of the last state (it carries the layer's dominant symbol if there is one), the
    // table (one 16-byte row per state: the entries for both values of the peeked bit; up to six rows per thread).
    const uint32_t cpp = p.chunks_per_panel;
    const anszp_chunk_t* panel_chunks = p.chunks + uint64_t(mtile) * cpp;
    const anszp_chunk_t held = panel_chunks[min(wave + min(lane, kMaxMine - 1u) * kWaves, cpp - 1u)];
    const uint32_t* table_src = p.tables + p.layer_id * table_stride_words(p.table_log);
    const anszp_layer_t lay = p.layers[p.layer_id];
    const uint32_t top = table_src[table_triples_offset(p.table_log) + L - 1u];
    constexpr uint32_t kTableLoads = ((1u << ANSZP_MAX_TABLE_LOG) + kThreads - 1u) / kThreads;
    const words4* tsrc = reinterpret_cast<const words4*>(table_src + table_lookahead_offset(p.table_log));
    words4 tv[kTableLoads];
#pragma unroll
    for (uint32_t u = 0; u < kTableLoads; ++u) tv[u] = tsrc[min(tid + u * kThreads, L - 1u)];

    auto desc_of = [&](uint32_t i) {                              // this wavefront's i-th chunk (i uniform)
        ChunkDesc c;
        const uint32_t layer_id = __builtin_amdgcn_readlane(held.layer_id, i);
        c.n_symbols = __builtin_amdgcn_readlane(held.n_symbols, i);
        c.payload_words = __builtin_amdgcn_readlane(held.payload_words, i);
        c.stream_offset = __builtin_amdgcn_readlane(held.stream_offset, i);
        c.payload_offset = uint64_t(uint32_t(__builtin_amdgcn_readlane(uint32_t(held.payload_offset), i))) |
                           uint64_t(uint32_t(__builtin_amdgcn_readlane(uint32_t(held.payload_offset >> 32), i))) << 32;
        c.ok = layer_id == p.layer_id && c.n_symbols == p.rows_per_chunk * p.K && (c.payload_offset & 3u) == 0 &&
               c.payload_offset <= p.payload_words && c.payload_words <= p.payload_words - c.payload_offset &&
               uint64_t(c.stream_offset) + p.n_streams <= p.n_stream_hdr;
        c.staged = c.payload_words + 2u <= kStageWords;           // two zero words behind the chunk's own
        return c;
    };
    auto fetch = [&](const ChunkDesc& c, ChunkData& d) {          // from clamped, always valid addresses
        d.hdr = 0u;
        d.q0 = d.q1 = words4{0u, 0u, 0u, 0u};
        d.tail = 0u;
        if (!c.ok) return;                                        // uniform
        if (lane < p.n_streams) d.hdr = p.stream_hdr[c.stream_offset + lane];
        const uint32_t quads = c.payload_words >> 2;
        if (c.staged && c.payload_words) {
            const uint32_t* words = p.payload + c.payload_offset;
            if (quads) {
                d.q0 = reinterpret_cast<const words4*>(words)[min(lane, quads - 1u)];
                d.q1 = reinterpret_cast<const words4*>(words)[min(lane + kWave, quads - 1u)];
            }
            const uint32_t tail_at = (quads << 2) + lane;
            if (lane < 3u && tail_at < c.payload_words) d.tail = words[tail_at];
        }
    };
    const uint32_t n_mine = wave < cpp ? (cpp - wave + kWaves - 1u) / kWaves : 0u;
    ChunkDesc cur{};
    ChunkData cur_data{};
    if (n_mine) {
        cur = desc_of(0u);
        fetch(cur, cur_data);
    }
    meanwhile();
    {
        // (done while the table is still on its way: only the quantizer and the last state's triple are needed)
        // The panel starts as the layer's dominant symbol everywhere (decoding writes only the other symbols);
        // also the columns from K to a row's end and the 64 bytes behind the last row, which the contraction
        // reads (the last 32 k of a row tile or of a kernel tap) against activations that are zero: as bf16
        // values they must be finite, whatever an earlier kernel left in LDS.
        const uint32_t dominant = top >> 24;
        uint32_t fill = dominant * 0x01010101u;
        if constexpr (P16) {
            const uint32_t h = __float_as_uint(static_cast<float>(int32_t(dominant) - int32_t(lay.zero_point))) >> 16;
            fill = h | h << 16;
        }
        const uint32_t panel_quads = (ROWS * p.row_stride * kElem + 64u) / 16u;
        for (uint32_t i = tid; i < panel_quads; i += kThreads) reinterpret_cast<words4*>(panel)[i] = words4{fill, fill, fill, fill};
    }
#pragma unroll
    for (uint32_t u = 0; u < kTableLoads; ++u)
        if (tid + u * kThreads < L) reinterpret_cast<words4*>(ahead)[tid + u * kThreads] = tv[u];
    __syncthreads();
    uint32_t err = (lay.channel_len != 0 && lay.channel_len != p.K) ? ANSZP_ST_BAD_DESC : 0u;   // scales per output channel only
    for (uint32_t i = 0; i < n_mine; ++i) {
        // the next chunk's words are asked for before this one is decoded
        ChunkDesc nxt{};
        ChunkData nxt_data{};
        if (i + 1u < n_mine) {
            nxt = desc_of(i + 1u);
            fetch(nxt, nxt_data);
        }
        const uint32_t j = wave + i * kWaves;
        // (LDS addresses count from 0: the kernels' only LDS is what their launch asks for, which begins there)
        if (!cur.ok) err |= ANSZP_ST_BAD_DESC;                    // its rows stay the dominant symbol
        else err |= decode_chunk_to_panel<P16>(p, cur, cur_data, kStageBytes, ahead_bytes - 8u, wave * (kStageWords * 4u),
                                               p.panel_off + j * p.rows_per_chunk * p.row_stride * kElem, lane, int32_t(lay.zero_point));
        cur = nxt;
        cur_data = nxt_data;
    }
    err = wave_or(err);
    if (err && lane == 0) report(p.status, err);
    return lay;
}

// A panel of symbol bytes widened in place to bf16 values q - z (the table and the staging room are free by then; the
// widened panel starts at the beginning of LDS): every thread takes its 16-byte pieces into registers, all wait, then
// every piece is written back as 32 bytes, all wait.
template <uint32_t MR>
__device__ __forceinline__ void widen_panel(const ConvParams& p, uint8_t* lds, const anszp_layer_t& lay) {
    const uint32_t tid = threadIdx.x;
    const uint32_t n_pieces = (kRows * MR * p.row_stride + 64u) / 16u;     // the host made sure: <= kWidenPieces * kThreads
    const float zf = static_cast<float>(lay.zero_point);
    words4 held_q[kWidenPieces];
#pragma unroll
    for (uint32_t u = 0; u < kWidenPieces; ++u)
        held_q[u] = reinterpret_cast<const words4*>(lds + p.panel_off)[min(tid + u * kThreads, n_pieces - 1u)];
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kWidenPieces; ++u) {
        const uint32_t i = tid + u * kThreads;
        if (i < n_pieces) {
            bf16x8* dst = reinterpret_cast<bf16x8*>(lds + 32u * i);
            dst[0] = weights_of(words2{held_q[u].x, held_q[u].y}, zf);
            dst[1] = weights_of(words2{held_q[u].z, held_q[u].w}, zf);
        }
    }
    __syncthreads();
}

// MR: MFMA row tiles per workgroup.  Every wavefront multiplies all 16 * MR panel rows with its columns, so
// an activation vector loaded once feeds MR MFMAs.
// P16: the panel is kept as bf16 (short rows: K <= 576), so that the contraction reads its A operands as they are.
// KIND: how the contraction addresses the activations.
enum { kTaps = 0,        // input channels a multiple of 8: a lane's 8 consecutive k lie under one kernel tap
       kPointwise = 1,   // as kTaps with a 1 x 1 kernel and no padding: one pixel per column, nothing outside the image
       kGeneric = 2,     // any number of input channels (NHWC): every activation is addressed on its own
       kTapsRing = 3,          // as kTaps with input channels a multiple of 32 * D: D steps' activations in flight
       kGenericPatch = 4 };    // as kGeneric when image rows are whole words, 16 bytes or more: the image rows under a round
                               // of pixels are staged in LDS, zero padding included, and gathered from there
// D (kTapsRing only): steps of 32 input channels whose activation loads are in flight at any time.
template <int KIND, uint32_t MR, bool P16, uint32_t D>
__global__ __launch_bounds__(kThreads) void conv_fused_kernel(ConvParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t* panel = lds + p.panel_off;
    constexpr uint32_t kElem = P16 ? 2u : 1u;                     // bytes per panel element
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t unit = unit_of_workgroup(), split = p.n_mtiles_by(unit), mtile = unit - split * p.n_mtiles;
    const anszp_layer_t lay = decode_panel<kRows * MR, P16>(p, lds, mtile, [] {});
    __syncthreads();
    // kGeneric: what every k of the reduction means, worked out once (the table and the staging room are free now):
    // two words per k, the offset of its activation from the one under the first tap's first channel, and its
    // kernel row | kernel column << 8 (a column no image has for the k beyond K)
    [[maybe_unused]] uint32_t* k_table = reinterpret_cast<uint32_t*>(lds);
    if constexpr (KIND == kGeneric) {
        for (uint32_t k = tid; k < ((p.K + 31u) & ~31u); k += kThreads) {
            const uint32_t tap = p.by_cin(k), c = k - tap * p.cin;
            const uint32_t r = p.by_kw(tap), sx = tap - r * p.kw;
            k_table[2u * k] = (r * p.in_w + sx) * p.cin + c;
            k_table[2u * k + 1u] = k < p.K ? (r | sx << 8) : 0xFFFFFF00u;
        }
        __syncthreads();
    }

    if constexpr (KIND == kGenericPatch) {
        // ---- phase 2 for any number of input channels (NHWC) when an image row is a number of words: the
        // workgroup's column tiles are taken in rounds of up to four per wavefront, dealt out evenly; the image rows under a
        // round's pixels go to LDS as they are, 16 bytes at a time, each behind 32 bytes whose upper part is the
        // left zero padding, followed by the right one; rows above and below an image are zeros.  A lane then
        // gathers its 8 k per column from LDS: the pixel's place plus an offset per k that is worked out once (a
        // table in LDS in front of the rows).  Nothing tests for the image's border.
        const uint32_t col = lane & 15u, kg = lane >> 4;          // MFMA operand layout: row or column, group of 8 k
        const uint8_t* a_row = panel + (col * p.row_stride + 8u * kg) * kElem;
        const uint32_t tile_stride = kRows * p.row_stride * kElem;
        const float zf = static_cast<float>(lay.zero_point);
        const uint32_t S = p.stride, Hp = p.in_h + 2u * p.pad;
        const uint32_t Kp = (p.K + 31u) & ~31u;
        // (a row is a whole number of words, its last piece may repeat some of the one before)
        const uint32_t row_bytes = p.in_w * p.cin * 2u, pieces_per_row = (row_bytes + 15u) / 16u;
        const uint32_t edge_words = (p.row_pitch - row_bytes) / 4u;        // the words of a row that hold no image: eight in front, the others behind
        uint32_t* k_offset = reinterpret_cast<uint32_t*>(lds);    // [Kp]: bytes from a pixel's first tap, first channel, to k's activation
        uint8_t* rows_at = lds + p.patch_off;
        for (uint32_t k = tid; k < Kp; k += kThreads) {
            const uint32_t tap = p.by_cin(k), c = k - tap * p.cin;
            const uint32_t r = p.by_kw(tap), sx = tap - r * p.kw;
            k_offset[k] = k < p.K ? r * p.row_pitch + (sx * p.cin + c) * 2u : 0u;
        }
        const uint32_t split_begin = split * p.pixels_per_split;
        const uint32_t split_end = min(split_begin + p.pixels_per_split, p.n_pixels);
        const uint32_t tiles = (split_end - split_begin + 15u) / 16u;
        const uint32_t n_rounds = (tiles + 4u * kWaves - 1u) / (4u * kWaves);
        const uint32_t round_tiles = n_rounds ? (tiles + n_rounds - 1u) / n_rounds : 0u;
        constexpr uint32_t kPieces = kPatchPieces;
        for (uint32_t round = 0; round < n_rounds; ++round) {
            const uint32_t t0 = round * round_tiles;
            if (t0 >= tiles) break;
            const uint32_t tn = min(round_tiles, tiles - t0);
            const uint32_t round0 = split_begin + 16u * t0, round_end = min(round0 + 16u * tn, split_end);
            // the staged rows: flat index b * Hp + padded row, from the first pixel's first tap to the last pixel's last
            auto row_under = [&](uint32_t pix) {                  // (flat output row b * out_h + ho)
                const uint32_t row = p.by_out_w(pix), b = p.by_out_h(row);
                return b * Hp + (row - b * p.out_h) * S;
            };
            const uint32_t pr0 = row_under(round0), pr_last = row_under(round_end - 1u) + p.kh - 1u;
            const uint32_t n_rows = pr_last - pr0 + 1u;
            const uint32_t n_pieces = n_rows * pieces_per_row;
            if (n_pieces > kPieces * kThreads) {                  // the host sized the rounds so that this cannot happen
                if (tid == 0) report(p.status, ANSZP_ST_INTERNAL);
                return;                                           // uniform
            }
            __syncthreads();                                      // the previous round's rows have been read (and k_offset written)
            words4 held_x[kPieces];
            uint32_t dst[kPieces];
#pragma unroll
            for (uint32_t u = 0; u < kPieces; ++u) {
                const uint32_t i = tid + u * kThreads;
                held_x[u] = words4{0u, 0u, 0u, 0u};
                dst[u] = 0xFFFFFFFFu;
                if (i < n_pieces) {
                    const uint32_t row = p.by_pieces(i), piece = i - row * pieces_per_row;
                    const uint32_t pra = pr0 + row;
                    const uint32_t b = p.by_padded_h(pra), h = pra - b * Hp - p.pad;         // unsigned: above the image wraps around
                    const uint32_t in_row = min(piece * 16u, row_bytes - 16u);
                    dst[u] = row * p.row_pitch + 32u + in_row;
                    if (h < p.in_h) held_x[u] = *reinterpret_cast<const words4_word_aligned*>(p.x + (b * p.in_h + h) * p.in_w * p.cin + in_row / 2u);
                }
            }
            for (uint32_t i = tid; i < n_rows * edge_words; i += kThreads) {
                const uint32_t row = p.by_edges(i), e = i - row * edge_words;
                *reinterpret_cast<uint32_t*>(rows_at + row * p.row_pitch + e * 4u + (e < 8u ? 0u : row_bytes)) = 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < kPieces; ++u)
                if (dst[u] != 0xFFFFFFFFu) *reinterpret_cast<words4_word_aligned*>(rows_at + dst[u]) = held_x[u];
            __syncthreads();

            const uint32_t w_begin = t0 + tn * wave / kWaves, w_end = t0 + tn * (wave + 1u) / kWaves;   // this wavefront's tiles
            const uint32_t pix0 = split_begin + 16u * w_begin, block_end = min(split_begin + 16u * w_end, split_end);
            auto block = [&](auto tiles_here) {
                constexpr uint32_t QT = decltype(tiles_here)::value;
                bool valid[4] = {false, false, false, false};
                uint32_t out_at[4] = {0u, 0u, 0u, 0u};
                uint32_t at_rows[QT];                             // byte of the pixel's first tap, first channel (may lie in the left padding)
#pragma unroll
                for (uint32_t q = 0; q < QT; ++q) {
                    const uint32_t pix = pix0 + q * 16u + col;
                    valid[q] = pix < block_end;
                    const uint32_t n = valid[q] ? pix : pix0;     // a column beyond the block stands on its first pixel
                    const uint32_t t = p.by_out_w(n), wo = n - t * p.out_w;
                    const uint32_t b = p.by_out_h(t), ho = t - b * p.out_h;
                    at_rows[q] = (b * Hp + ho * S - pr0) * p.row_pitch + 32u + (wo * S * p.cin) * 2u - p.pad * p.cin * 2u;
                    out_at[q] = b * p.out_h * p.out_w * p.cout + (ho * p.out_w + wo) * p.y_pixel;
                }
                floatx4 acc[MR][4];
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m)
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) acc[m][q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                for (uint32_t k0 = 0; k0 < Kp; k0 += 32u) {
                    const uint32_t kbase = k0 + 8u * kg;
                    const words4 off_lo = *reinterpret_cast<const words4*>(k_offset + kbase);
                    const words4 off_hi = *reinterpret_cast<const words4*>(k_offset + kbase + 4u);
                    const uint32_t off[8] = {off_lo.x, off_lo.y, off_lo.z, off_lo.w, off_hi.x, off_hi.y, off_hi.z, off_hi.w};
                    words4 b[QT];
#pragma unroll
                    for (uint32_t q = 0; q < QT; ++q) {
                        uint32_t v[8];
#pragma unroll
                        for (uint32_t j = 0; j < 8; ++j) {
                            v[j] = *reinterpret_cast<const uint16_t*>(rows_at + at_rows[q] + off[j]);
                            if (kbase + j >= p.K) v[j] = 0u;      // beyond the reduction (the last step only)
                        }
                        b[q] = words4{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16};
                    }
#pragma unroll
                    for (uint32_t m = 0; m < MR; ++m) {
                        bf16x8 a;
                        if constexpr (P16) a = *reinterpret_cast<const bf16x8*>(a_row + m * tile_stride + k0 * 2u);
                        else a = weights_of(*reinterpret_cast<const words2*>(a_row + m * tile_stride + k0), zf);
#pragma unroll
                        for (uint32_t q = 0; q < QT; ++q)
                            acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b[q]), acc[m][q], 0, 0, 0);
                    }
                }
                store_tiles<MR>(p, lay, mtile, kg, acc, valid, out_at);
            };
            switch (w_end - w_begin) {                            // uniform
                case 1: block(std::integral_constant<uint32_t, 1>{}); break;
                case 2: block(std::integral_constant<uint32_t, 2>{}); break;
                case 3: block(std::integral_constant<uint32_t, 3>{}); break;
                case 4: block(std::integral_constant<uint32_t, 4>{}); break;
                default: break;
            }
        }
        return;
    }

    if constexpr (KIND == kTapsRing) {
        // ---- phase 2 for kernels of several taps whose input channels are a multiple of 32 * D: steps of 32 k, kernel
        // taps outermost, in groups of D steps that never straddle a tap; rounds of up to four column tiles per wavefront,
        // dealt out evenly.  A column whose pixel lies outside the image under a tap reads zero_page for that tap (with a
        // step stride of zero), so every load is unconditional.
        const uint32_t col = lane & 15u, kg = lane >> 4;          // MFMA operand layout: row or column, group of 8 k
        if constexpr (!P16) widen_panel<MR>(p, lds, lay);         // (the host keeps this kind for panels that can be widened)
        const uint8_t* a_row = (P16 ? panel : lds) + (col * p.row_stride + 8u * kg) * 2u;
        const uint32_t tile_stride = kRows * p.row_stride * 2u;
        const uint32_t groups_per_tap = p.cin / (32u * D);
        const uint32_t n_groups = p.kh * p.kw * groups_per_tap;
        const uint32_t split_begin = split * p.pixels_per_split;
        const uint32_t split_end = min(split_begin + p.pixels_per_split, p.n_pixels);
        const uint32_t tiles = (split_end - split_begin + 15u) / 16u;
        const uint32_t n_rounds = (tiles + 4u * kWaves - 1u) / (4u * kWaves);
        const uint32_t round_tiles = n_rounds ? (tiles + n_rounds - 1u) / n_rounds : 0u;
        const uint16_t* zeros = reinterpret_cast<const uint16_t*>(zero_page);
        auto block = [&](uint32_t pix0, uint32_t block_end, auto tiles_here) {
            constexpr uint32_t QT = decltype(tiles_here)::value;
            bool valid[4] = {false, false, false, false};
            uint32_t out_at[4] = {0u, 0u, 0u, 0u};
            int32_t h0[QT], w0[QT];
            uint32_t img[QT];
#pragma unroll
            for (uint32_t q = 0; q < QT; ++q) {
                const uint32_t pix = pix0 + q * 16u + col;
                valid[q] = pix < block_end;
                const uint32_t n = valid[q] ? pix : pix0;         // a column beyond the block stands on its first pixel
                const uint32_t t = p.by_out_w(n), wo = n - t * p.out_w;
                const uint32_t b = p.by_out_h(t), ho = t - b * p.out_h;
                h0[q] = int32_t(ho * p.stride) - int32_t(p.pad);
                w0[q] = int32_t(wo * p.stride) - int32_t(p.pad);
                img[q] = b * p.in_h * p.in_w * p.cin;
                out_at[q] = b * p.out_h * p.out_w * p.cout + (ho * p.out_w + wo) * p.y_pixel;
            }
            floatx4 acc[MR][4];
#pragma unroll
            for (uint32_t m = 0; m < MR; ++m)
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) acc[m][q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            // where the requests of the group being asked for read: the tap's pixel of every column, and how far it
            // is from one step's vector to the next's (nothing, on the zero page)
            const uint16_t* tap_ptr[QT];
            uint32_t tap_step[QT];
            auto enter_tap = [&](uint32_t tap) {
                const uint32_t r = p.by_kw(tap), sx = tap - r * p.kw;
#pragma unroll
                for (uint32_t q = 0; q < QT; ++q) {
                    const int32_t h = h0[q] + int32_t(r), w = w0[q] + int32_t(sx);
                    const bool inside = uint32_t(h) < p.in_h && uint32_t(w) < p.in_w;
                    tap_ptr[q] = inside ? p.x + (img[q] + (uint32_t(h) * p.in_w + uint32_t(w)) * p.x_pixel + kg * p.x_block) : zeros;
                    tap_step[q] = inside ? 4u * p.x_block : 0u;
                }
            };
            words4 ring[D][QT];
            auto request = [&](uint32_t d, uint32_t step_in_tap) {
                const uint16_t* from[QT];
#pragma unroll
                for (uint32_t q = 0; q < QT; ++q) from[q] = tap_ptr[q] + __umul24(step_in_tap, tap_step[q]);
                ring_request<QT>(ring[d], from);
            };
            auto multiply = [&](uint32_t k_first, uint32_t d) {   // k_first: the step's first k (its panel column)
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m) {
                    const bf16x8 a = *reinterpret_cast<const bf16x8*>(a_row + m * tile_stride + k_first * 2u);
#pragma unroll
                    for (uint32_t q = 0; q < QT; ++q)
                        acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, ring[d][q]), acc[m][q], 0, 0, 0);
                }
            };
            enter_tap(0u);
#pragma unroll
            for (uint32_t d = 0; d < D; ++d) request(d, d);
            uint32_t tap = 0, group_in_tap = 0;                   // of the group being multiplied
            for (uint32_t g = 0; g + 1u < n_groups; ++g) {        // every group but the last
                uint32_t next_tap = tap, next_in_tap = group_in_tap + 1u;
                if (next_in_tap == groups_per_tap) {              // uniform
                    next_in_tap = 0;
                    ++next_tap;
                    enter_tap(next_tap);
                }
                const uint32_t k_group = tap * p.cin + group_in_tap * (32u * D);
#pragma unroll
                for (uint32_t d = 0; d < D; ++d) {
                    ring_arrived<QT, (D - 1u) * QT>(ring[d]);
                    multiply(k_group + 32u * d, d);
                    request(d, next_in_tap * D + d);
                }
                tap = next_tap;
                group_in_tap = next_in_tap;
            }
            const uint32_t k_group = tap * p.cin + group_in_tap * (32u * D);
            static_assert(D == 2 || D == 4, "written out for two and four slots");
            if constexpr (D == 2) {
                ring_arrived<QT, QT>(ring[0]);
                multiply(k_group, 0u);
                ring_arrived<QT, 0u>(ring[1]);
                multiply(k_group + 32u, 1u);
            } else {
                ring_arrived<QT, 3u * QT>(ring[0]);
                multiply(k_group, 0u);
                ring_arrived<QT, 2u * QT>(ring[1]);
                multiply(k_group + 32u, 1u);
                ring_arrived<QT, QT>(ring[2]);
                multiply(k_group + 64u, 2u);
                ring_arrived<QT, 0u>(ring[3]);
                multiply(k_group + 96u, 3u);
            }
            store_tiles<MR>(p, lay, mtile, kg, acc, valid, out_at);
        };
        for (uint32_t round = 0; round < n_rounds; ++round) {
            const uint32_t t0 = round * round_tiles;
            if (t0 >= tiles) break;
            const uint32_t tn = min(round_tiles, tiles - t0);
            const uint32_t w_begin = t0 + tn * wave / kWaves, w_end = t0 + tn * (wave + 1u) / kWaves;   // this wavefront's tiles
            const uint32_t pix0 = split_begin + 16u * w_begin, block_end = min(split_begin + 16u * w_end, split_end);
            switch (w_end - w_begin) {                            // uniform
                case 1: block(pix0, block_end, std::integral_constant<uint32_t, 1>{}); break;
                case 2: block(pix0, block_end, std::integral_constant<uint32_t, 2>{}); break;
                case 3: block(pix0, block_end, std::integral_constant<uint32_t, 3>{}); break;
                case 4: block(pix0, block_end, std::integral_constant<uint32_t, 4>{}); break;
                default: break;
            }
        }
        return;
    }

    // ---- phase 2: the panel times the activations
    const uint32_t col = lane & 15u, kg = lane >> 4;              // MFMA operand layout: row or column, group of 8 k
    const uint8_t* a_row = panel + (col * p.row_stride + 8u * kg) * kElem;  // A: lane holds row lane % 16 of a row tile, k = 8 * (lane / 16) + 0..7
    const uint32_t tile_stride = kRows * p.row_stride * kElem;
    const float zf = static_cast<float>(lay.zero_point);
    auto a_operand = [&](const uint8_t* at) {                     // 8 consecutive k of this lane's row
        if constexpr (P16) return *reinterpret_cast<const bf16x8*>(at);
        else return weights_of(*reinterpret_cast<const words2*>(at), zf);
    };
    const uint32_t Kp = (p.K + 31u) & ~31u;
    // The workgroup's pixels are dealt out to its wavefronts in blocks of block_pixels, round robin, so that at
    // any time the wavefronts work on neighbouring pixels (kernel taps of neighbours share input rows).  A block
    // is 64 pixels unless the workgroup has fewer than 64 per wavefront: then it is narrower and the column
    // tiles beyond it are switched off, rather than wavefronts left without work.
    const uint32_t split_end = min((split + 1u) * p.pixels_per_split, p.n_pixels);

    for (uint32_t pix0 = split * p.pixels_per_split + wave * p.block_pixels; pix0 < split_end; pix0 += kWaves * p.block_pixels) {
        const uint32_t block_end = min(pix0 + p.block_pixels, split_end);
        // B: lane holds column lane % 16 of each of the block's four column tiles
        uint32_t pix[4];
        int32_t h0[4], w0[4];
        uint32_t img[4], out_at[4];                              // first element of the image in x; of the pixel in y
        bool valid[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            pix[q] = pix0 + q * 16u + col;
            valid[q] = pix[q] < block_end;
            const uint32_t n = valid[q] ? pix[q] : 0u;
            const uint32_t t = p.by_out_w(n), wo = n - t * p.out_w;
            const uint32_t b = p.by_out_h(t), ho = t - b * p.out_h;
            h0[q] = int32_t(ho * p.stride) - int32_t(p.pad);
            w0[q] = int32_t(wo * p.stride) - int32_t(p.pad);
            img[q] = b * p.in_h * p.in_w * p.cin;
            out_at[q] = b * p.out_h * p.out_w * p.cout + (ho * p.out_w + wo) * p.y_pixel;
        }
        floatx4 acc[MR][4];
#pragma unroll
        for (uint32_t m = 0; m < MR; ++m)
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) acc[m][q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

        if constexpr (KIND == kPointwise) {
            // One pixel per column for the whole reduction: a step of 32 input channels is one address
            // addition per column.  The next step's activation vectors are requested before this step's MFMAs.
            const uint32_t n_steps = (p.cin + 31u) / 32u;
            const uint16_t* px[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                px[q] = p.x + (valid[q] ? img[q] + (uint32_t(h0[q]) * p.in_w + uint32_t(w0[q])) * p.x_pixel : 0u) + kg * p.x_block;
            auto load_step = [&](uint32_t step, words4 (&b)[4]) {
                const bool live = step < n_steps && step * 32u + 8u * kg < p.cin;   // the last step may be partly beyond the channels
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    b[q] = words4{0u, 0u, 0u, 0u};
                    if (live && valid[q]) b[q] = *reinterpret_cast<const words4*>(px[q] + step * 4u * p.x_block);
                }
            };
            words4 cur[4], nxt[4];
            load_step(0u, cur);
            for (uint32_t step = 0; step < n_steps; ++step) {
                load_step(step + 1u, nxt);
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m) {
                    const bf16x8 a = a_operand(a_row + m * tile_stride + step * 32u * kElem);
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q)
                        acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, cur[q]), acc[m][q], 0, 0, 0);
                }
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) cur[q] = nxt[q];
            }
        } else if constexpr (KIND == kTaps) {
            // Steps of 32 k: kernel taps outermost, 32 input channels at a time inside a tap.
            const uint32_t steps_per_tap = (p.cin + 31u) / 32u;
            const uint32_t n_steps = p.kh * p.kw * steps_per_tap;
            struct Cursor { uint32_t r, s, c0, a_off; };          // a_off: the step's first k (its panel column)
            auto advance = [&](Cursor& c) {
                c.c0 += 32u;
                if (c.c0 >= p.cin) {
                    c.c0 = 0;
                    c.a_off += p.cin;
                    if (++c.s == p.kw) { c.s = 0; ++c.r; }
                }
            };
            // where each column's pixel under the load cursor's kernel tap lies (recomputed when the cursor
            // enters a tap), so that a step costs one address addition per column
            const uint16_t* tap_ptr[4];
            bool tap_inside[4];
            auto enter_tap = [&](const Cursor& c) {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const int32_t h = h0[q] + int32_t(c.r), w = w0[q] + int32_t(c.s);
                    tap_inside[q] = valid[q] && uint32_t(h) < p.in_h && uint32_t(w) < p.in_w;
                    const uint32_t at = tap_inside[q] ? img[q] + (uint32_t(h) * p.in_w + uint32_t(w)) * p.x_pixel : 0u;
                    tap_ptr[q] = p.x + at + kg * p.x_block;           // this lane's block of 8 channels of the step's first 32
                }
            };
            auto load_step = [&](const Cursor& c, bool in_range, words4 (&b)[4]) {
                if (c.c0 == 0) enter_tap(c);                            // wavefront-uniform
                const bool live = in_range && c.c0 + 8u * kg < p.cin;   // the last 32 k of a tap may be partly beyond it
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    b[q] = words4{0u, 0u, 0u, 0u};
                    if (live && tap_inside[q]) b[q] = *reinterpret_cast<const words4*>(tap_ptr[q] + (c.c0 >> 3) * p.x_block);
                }
            };
            // a ring of kDepth steps' activation vectors: a step's slot is refilled, for the step kDepth
            // later, as soon as its MFMAs are issued.  Two steps: a deeper ring buys nothing as long as the
            // compiler waits for all outstanding loads before a step's MFMAs, and its registers are better
            // spent on a third wavefront per SIMD.
            constexpr uint32_t kDepth = 2;
            words4 ring[kDepth][4];
            Cursor ld{0u, 0u, 0u, 0u}, use{0u, 0u, 0u, 0u};
#pragma unroll
            for (uint32_t d = 0; d < kDepth; ++d) { load_step(ld, d < n_steps, ring[d]); advance(ld); }
            for (uint32_t base = 0; base < n_steps; base += kDepth) {
#pragma unroll
                for (uint32_t d = 0; d < kDepth; ++d) {
                    if (base + d < n_steps) {
#pragma unroll
                        for (uint32_t m = 0; m < MR; ++m) {
                            const bf16x8 a = a_operand(a_row + m * tile_stride + (use.a_off + use.c0) * kElem);
#pragma unroll
                            for (uint32_t q = 0; q < 4; ++q)
                                acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, ring[d][q]), acc[m][q], 0, 0, 0);
                        }
                    }
                    advance(use);
                    load_step(ld, base + d + kDepth < n_steps, ring[d]);
                    advance(ld);
                }
            }
        } else {
            // where each column's pixel lies under the first kernel tap (possibly outside the image: only used
            // together with a tap that is inside)
            uint32_t corner[4];
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) corner[q] = img[q] + uint32_t((h0[q] * int32_t(p.in_w) + w0[q]) * int32_t(p.cin));
            for (uint32_t k0 = 0; k0 < Kp; k0 += 32u) {
                const uint32_t kbase = k0 + 8u * kg;
                uint16_t bv[4][8];
                words2 kt[8];                                     // this lane's 8 k of the step: offset, kernel row and column
#pragma unroll
                for (uint32_t j = 0; j < 8; j += 2) {
                    const words4 two = *reinterpret_cast<const words4*>(k_table + 2u * (kbase + j));
                    kt[j] = words2{two.x, two.y};
                    kt[j + 1] = words2{two.z, two.w};
                }
#pragma unroll
                for (uint32_t j = 0; j < 8; ++j) {
                    const uint32_t r = kt[j].y & 0xFFu, s = kt[j].y >> 8;          // s = 0xFFFFFF beyond K: outside every image
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        const int32_t h = h0[q] + int32_t(r), w = w0[q] + int32_t(s);
                        const bool inside = valid[q] && uint32_t(h) < p.in_h && uint32_t(w) < p.in_w;
                        bv[q][j] = inside ? p.x[corner[q] + kt[j].x] : uint16_t(0);   // NHWC only
                    }
                }
                words4 b[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
                    b[q] = words4{uint32_t(bv[q][0]) | uint32_t(bv[q][1]) << 16, uint32_t(bv[q][2]) | uint32_t(bv[q][3]) << 16,
                                  uint32_t(bv[q][4]) | uint32_t(bv[q][5]) << 16, uint32_t(bv[q][6]) | uint32_t(bv[q][7]) << 16};
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m) {
                    const bf16x8 a = a_operand(a_row + m * tile_stride + k0 * kElem);
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q)
                        acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b[q]), acc[m][q], 0, 0, 0);
                }
            }
        }

        store_tiles<MR>(p, lay, mtile, kg, acc, valid, out_at);
    }
}

// The convolution of layers whose input channels are a multiple of 8 and whose kernels are 1 x 1 without padding
// (kPoint) or three taps wide (kRow; stride 1: kShift): nearly all of a network's.  TAIL: the channels are no multiple of 32,
// so that the last unit of a kernel row has fewer (a kernel of its own, because the condition on every load is worth a few
// per cent).  Such layers were left to the loops without slices and rings before: 28 drawn calls of 72 to 1,624 channels 1.0 to
// 4.2 times as fast (3 x 3 x 496 on two 23 x 23 images 57 -> 17 us, 1 x 1 from 816 channels on one 47 x 47 image 46 -> 19), 8 to 24
// channels, where most of a unit is empty, 1.02 to 1.8.
//
// Phase 2: a step is a kernel tap and 32 input channels, a unit the steps of a kernel row with the same 32 channels.
// kRow asks for the row's three taps together: they read the same pixels shifted by one, or alternate halves of the
// same lines (stride 2), and the L1 then fetches a line once for them.  kShift asks for the middle tap only (and one
// vector that holds the pixels before the first and behind the last): the other two are the neighbouring lanes' values,
// moved by one lane, zero at the ends of a row of pixels.  With padding those are the zeros around the image; without,
// a row has a pixel more on either side, whose middle tap is the image's first or last column and which has no output.  A load of 64 lanes of 16 bytes keeps a CU's address path busy for about
// 34 clocks, more than the multiplications it feeds take when a panel has one row tile (K = 4608): 3 x 3 x 512 at 7 x 7
// loads 4 vectors where kRow loads 9.  The workgroup's column tiles are dealt to t_groups
// wavefronts, QT or one fewer each, the units to k_groups slices; t_groups * k_groups = 12.  A wavefront multiplies its
// tiles with its slice, and the slices' sums are added up through LDS (the panel is no longer needed then).  What the
// slices are for: a panel row tile read from LDS serves all of a wavefront's column tiles, so fewer tile ranges mean
// fewer LDS reads, and with fewer tiles than wavefronts none of them idles.
//
// What bounds these launches (12 to 25 us each) is largely code that runs for the first time: a CU fetches it 64 bytes at
// a time from the L2, about 85 ns each, which is as long as ten instructions take once they are there (measured: 2.5 us
// for the tiles' addresses, 0.35 us the second time).  So the code is kept short: no divisions (the host passes
// reciprocals), no conditions on a pixel or unit (loads go through a buffer descriptor: what lies outside the image, belongs
// to no pixel or to no unit has an offset beyond the buffer or an empty buffer and reads as zero without memory traffic;
// stores that belong to no pixel are dropped the same way), one kernel per number of tiles, the slices' sums in a loop.
// A load that reads nothing still takes its 25 to 34 clocks of the address path, though, so the last units of a slice have
// code of their own that asks for no more (as many again as are in flight otherwise, and their multiplications: 840 calls
// whose best choice takes 9 to 500 us became 4 to 20 % faster where a wavefront has few units or rounds, none slower; 1 x 1
// from 32 channels to 592 on eight 59 x 59 images 31 -> 27 us).
//
// The first units' activations are asked for before the panel is decoded, behind the loads that decoding waits for, where the
// registers hold them meanwhile (kEarly: all but 4 row tiles x 3 column tiles of three taps and 4 column tiles of nine
// vectors): a ResNet-50's convolutions, each repeated, 696 -> 674 us on 16 images and 1286 -> 1263 on 64, 0.1 to 1.2 us a call.
//
// Measured against rings of loads without slices (a call among others, MI355X): 3 x 3 x 512 channels, one 7 x 7 image 21.8 ->
// 12.4 us; 1 x 1 from 1024 channels, 64 14 x 14 images 21.4 -> 16.8; 3 x 3 x 128 channels, 64 28 x 28 images 28.5 -> 25.5; a
// ResNet-50's 53 convolutions on 16 images, one call each 900 -> 692.
// Every lane's neighbour's words within rows of 16 lanes: of the lane before (BEFORE) or after, the first (last) lane's
// from `beyond`, which holds them in the row's last (first) lane if it is a tile of its own (ROTATE), else in the lane
// itself; and-ed with `mask`.  (Moves and masks in one: the lane without a source keeps what the first instruction
// wrote.  The wait states are those between writing a register and reading it from another lane or
// in a matrix instruction.)
template <bool BEFORE, bool ROTATE>
__device__ __forceinline__ words4 neighbours(const words4& tile, const words4& beyond, uint32_t mask) {
    words4 v;
#define ANSZP_NEIGHBOURS(FIRST, FIRST_MOVE, MOVE)                                                                          \
    asm("s_nop 1\n"                                                                                                        \
        FIRST " %0, %8, %12" FIRST_MOVE FIRST " %1, %9, %12" FIRST_MOVE FIRST " %2, %10, %12" FIRST_MOVE FIRST " %3, %11, %12" FIRST_MOVE   \
        "v_and_b32_dpp %0, %4, %12" MOVE "v_and_b32_dpp %1, %5, %12" MOVE "v_and_b32_dpp %2, %6, %12" MOVE "v_and_b32_dpp %3, %7, %12" MOVE \
        "s_nop 1\n"                                                                                                        \
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])                                                                \
        : "v"(tile[0]), "v"(tile[1]), "v"(tile[2]), "v"(tile[3]), "v"(beyond[0]), "v"(beyond[1]), "v"(beyond[2]), "v"(beyond[3]), "v"(mask))
#define ANSZP_MOVE(HOW) " " HOW " row_mask:0xf bank_mask:0xf\n"
    if constexpr (BEFORE && ROTATE) ANSZP_NEIGHBOURS("v_and_b32_dpp", ANSZP_MOVE("row_ror:1"), ANSZP_MOVE("row_shr:1"));
    if constexpr (BEFORE && !ROTATE) ANSZP_NEIGHBOURS("v_and_b32", "\n", ANSZP_MOVE("row_shr:1"));
    if constexpr (!BEFORE && ROTATE) ANSZP_NEIGHBOURS("v_and_b32_dpp", ANSZP_MOVE("row_ror:15"), ANSZP_MOVE("row_shl:1"));
    if constexpr (!BEFORE && !ROTATE) ANSZP_NEIGHBOURS("v_and_b32", "\n", ANSZP_MOVE("row_shl:1"));
#undef ANSZP_MOVE
#undef ANSZP_NEIGHBOURS
    return v;
}

template <uint32_t ROWS, bool P16, uint32_t MODE, uint32_t QT, bool TAIL>
__global__ __launch_bounds__(kThreads) void conv_sliced_kernel(ConvParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr uint32_t MR = ROWS < kRows ? 1u : ROWS / kRows;     // row tiles
    constexpr bool kHalf = ROWS < kRows;                          // half a row tile: its lower rows are the upper ones again, and not stored
    constexpr uint32_t NS = MODE == kPoint ? 1u : 3u;             // steps of a unit
    constexpr uint32_t NF = MODE == kRow ? 3u : 1u;               // vectors of a unit that are loaded per column tile
    constexpr uint32_t kSlots = units_in_flight(MR, MODE, QT);
    // the first round's activations are asked for before the panel is decoded
    constexpr bool kEarly = MODE == kPoint || (MODE == kShift ? MR * QT < 12u : MR * QT < 12u && QT < 4u);
    constexpr uint32_t kOutside = 0x80000000u;                    // an offset beyond any x or y (the host: fewer than 2^31 bytes)
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t unit = unit_of_workgroup(), split = p.n_mtiles_by(unit), mtile = unit - split * p.n_mtiles;
    const uint32_t col = lane & 15u, kg = lane >> 4;              // MFMA operand layout: row or column, group of 8 k
    const uint32_t wk = (wave * p.t_groups_inv) >> 16, wt = wave - wk * p.t_groups;
    const uint32_t split_begin = split * p.pixels_per_split;
    const uint32_t split_end = min(split_begin + p.pixels_per_split, p.n_pixels);

    // B: lane holds column lane % 16 of each of the wavefront's QT column tiles.  Where the taps of the first kernel row read
    // (byte of x; kOutside: outside the image), that row, byte of y (kOutside: no pixel)
    uint32_t from[NF][QT], out_at[QT];
    int32_t h0[QT];
    [[maybe_unused]] uint32_t edge_from = kOutside;               // kShift: of the pixel before the first column (lanes 0) and
    [[maybe_unused]] int32_t edge_h0 = 0;                         // behind the last (lanes 15)
    [[maybe_unused]] uint32_t not_left[QT], not_right[QT];        // all bits, or none in a row's first, last column
    const uint32_t y_elem = p.y_bf16 ? 1u : 2u;                   // log2 bytes
    // returns the pixel's byte of y; kShift: wo is a column (p.first_column: output column 0)
    auto pixel_of = [&](uint32_t pix, uint32_t end, uint32_t& b, uint32_t& ho, uint32_t& wo) {
        const uint32_t t = __umulhi(2u * pix, p.columns_magic) >> p.columns_shift;
        wo = pix - t * p.columns;
        b = __umulhi(2u * t, p.out_h_magic) >> p.out_h_shift;
        ho = t - b * p.out_h;
        if constexpr (MODE == kShift) {
            const uint32_t w = wo - p.first_column;
            const uint32_t at = (b * p.y_image + (ho * p.out_w + w) * p.y_pixel + (kg >> 1) * p.y_block + 4u * (kg & 1u)) << y_elem;
            return ((pix < end) & (w < p.out_w) & (!kHalf || kg < 2u)) ? at : kOutside;
        }
        // D: lane holds column lane % 16, rows 4 * (lane / 16) + 0..3 of a row tile
        const uint32_t at = (b * p.y_image + (ho * p.out_w + wo) * p.y_pixel + (kg >> 1) * p.y_block + 4u * (kg & 1u)) << y_elem;
        return ((pix < end) & (!kHalf || kg < 2u)) ? at : kOutside;
    };
    // a round's tiles dealt evenly: QT or one fewer each
    auto first_tile = [&](uint32_t g) { return g * p.wave_tiles + min(g, p.wave_tiles_rest); };
    const bool has_last = first_tile(wt + 1u) - first_tile(wt) == QT;
    auto place = [&](uint32_t t0) __attribute__((always_inline)) {                               // of the round from tile t0 on
        const uint32_t pix0 = split_begin + 16u * (t0 + first_tile(wt)), end = min(split_begin + 16u * (t0 + first_tile(wt + 1u)), split_end);
#pragma unroll
        for (uint32_t q = 0; q < QT; ++q) {
            const uint32_t pix = pix0 + q * 16u + col;
            uint32_t b, ho, wo;
            out_at[q] = pixel_of(pix, end, b, ho, wo);
            h0[q] = int32_t(ho * p.stride) - int32_t(p.pad);
            // (kShift: stride 1; the middle tap's column, w0 of the others)
            const int32_t w0 = MODE == kShift ? int32_t(wo - p.first_column) + 1 - int32_t(p.pad) : int32_t(wo * p.stride) - int32_t(p.pad);
            const uint32_t corner = (b * p.x_image + uint32_t(h0[q] * int32_t(p.in_w) + w0) * p.x_pixel + kg * p.x_block) * 2u;
            if constexpr (MODE == kShift) {                       // (a column that is not stored may be a neighbour's neighbour)
                from[0][q] = ((pix < p.n_pixels) & (uint32_t(w0) < p.in_w)) ? corner : kOutside;
                not_left[q] = wo != 0u ? 0xFFFFFFFFu : 0u;
                not_right[q] = wo + 1u != p.columns ? 0xFFFFFFFFu : 0u;
            } else {
#pragma unroll
                for (uint32_t sx = 0; sx < NS; ++sx)
                    from[sx][q] = ((uint32_t(w0 + int32_t(sx)) < p.in_w) & (pix < end)) ? corner + sx * p.x_pixel * 2u : kOutside;
            }
        }
        if constexpr (MODE == kShift) {
            const uint32_t pix = col == 0u ? pix0 - 1u : pix0 + 16u * QT;      // (before pixel 0: beyond all; a tile that is not there
                                                                  // is loaded all the same)
            uint32_t b, ho, wo;
            pixel_of(min(pix, p.n_pixels - 1u), 0u, b, ho, wo);
            edge_h0 = int32_t(ho) - int32_t(p.pad);
            const int32_t w0 = int32_t(wo - p.first_column) + 1 - int32_t(p.pad);
            const bool is_edge = (col == 0u) | (col == 15u);
            edge_from = (is_edge & (pix < p.n_pixels) & (uint32_t(w0) < p.in_w))
                            ? (b * p.x_image + uint32_t(edge_h0 * int32_t(p.in_w) + w0) * p.x_pixel + kg * p.x_block) * 2u : kOutside;
        }
    };
    const uint32_t blocks = TAIL ? (p.cin + 31u) / 32u : p.cin / 32u, units = (MODE != kPoint ? p.kh : 1u) * blocks;
    const uint32_t u_begin = wk * p.slice_units, n = min(p.slice_units, units - min(u_begin, units));
    // TAIL: the last block has fewer than 32 channels; the lanes of those that are missing read outside there (the weights they
    // meet are the next tap's or the row's padding: finite)
    [[maybe_unused]] const bool beyond_tail = 8u * kg >= p.cin % 32u;
    const uint32_t row0 = MODE != kPoint ? __umulhi(2u * u_begin, p.blocks_magic) >> p.blocks_shift : 0u;
    // the cursors of the loads and of the multiplications: kernel row and block of 32 channels of the next unit
    uint32_t row, cb, use_cb, k_use, asked;
    words4 ring[kSlots][NF][QT];
    [[maybe_unused]] words4 edge[kSlots];
    auto request = [&](uint32_t slot) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.x), 0, asked < n ? p.x_bytes : 0u, 0x00020000);
        const uint32_t at = asked < n ? cb * 8u * p.x_block : 0u;      // (an empty buffer's check must not overflow)
        // (what is outside stays beyond the buffer: no row is 2^31 bytes away)
        const uint32_t row_at = MODE == kPoint ? 0u : row * p.in_w * p.x_pixel * 2u;
        [[maybe_unused]] const bool is_tail = TAIL && cb + 1u == blocks;
        auto in_row = [&](int32_t first_row, uint32_t where) {
            const uint32_t v = MODE == kPoint ? where : uint32_t(first_row + int32_t(row)) < p.in_h ? where + row_at : kOutside;
            if constexpr (TAIL) return is_tail && beyond_tail ? kOutside : v;
            return v;
        };
#pragma unroll
        for (uint32_t q = 0; q < QT; ++q)
#pragma unroll
            for (uint32_t f = 0; f < NF; ++f) ring[slot][f][q] = __builtin_amdgcn_raw_buffer_load_b128(x, in_row(h0[q], from[f][q]), at, 0);
        if constexpr (MODE == kShift) edge[slot] = __builtin_amdgcn_raw_buffer_load_b128(x, in_row(edge_h0, edge_from), at, 0);
        ++asked;
        ++cb;
        if constexpr (MODE != kPoint) {
            const bool next_row = cb == blocks;               // (without a branch)
            cb = next_row ? 0u : cb;
            row += next_row ? 1u : 0u;
        }
    };
    auto request_first = [&]() __attribute__((always_inline)) {
        row = row0;
        cb = use_cb = u_begin - row0 * blocks;
        k_use = row0 * NS * p.cin + cb * 32u;
        asked = 0;
#pragma unroll
        for (uint32_t d = 0; d < kSlots; ++d) request(d);
    };
    const anszp_layer_t lay = decode_panel<ROWS, P16>(p, lds, mtile, [&]() __attribute__((always_inline)) {
        place(0u);
        if constexpr (kEarly) request_first();
    });
    __syncthreads();
    if constexpr (!P16) widen_panel<MR>(p, lds, lay);

    const uint32_t a_at = lds_address(lds) + (P16 ? p.panel_off : 0u) + ((kHalf ? col & 7u : col) * p.row_stride + 8u * kg) * 2u;
    const uint32_t tile_stride = kRows * p.row_stride * 2u;
    const __amdgpu_buffer_rsrc_t y_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, p.y_bytes, 0x00020000);
    const bool per_channel = lay.channel_len != 0;
    auto store = [&](uint32_t m, uint32_t at, const floatx4 sum) {
        const uint32_t tile = mtile * MR + m;                     // (o = 16 * tile + 4 * kg + i, of half a row tile 8 * tile + ..)
        float sc[4] = {lay.scale, lay.scale, lay.scale, lay.scale};
        if (per_channel) {
#pragma unroll 1
            for (uint32_t i = 0; i < 4; ++i) {
                const uint64_t ch = lay.scales_offset + tile * (kHalf ? ROWS : kRows) + 4u * kg + i;
                const float v = ch < p.n_scales ? p.scales[ch] : 0.0f;
                sc[0] = i == 0u ? v : sc[0]; sc[1] = i == 1u ? v : sc[1]; sc[2] = i == 2u ? v : sc[2]; sc[3] = i == 3u ? v : sc[3];
            }
        }
        const floatx4 out = {sum[0] * sc[0], sum[1] * sc[1], sum[2] * sc[2], sum[3] * sc[3]};
        const uint32_t tile_at = ((kHalf ? 1u : 2u) * tile * p.y_block) << y_elem;
        if (p.y_bf16) {                                           // round to nearest even (v_cvt_pk_bf16_f32)
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            const bf16x4 r = {static_cast<__bf16>(out[0]), static_cast<__bf16>(out[1]), static_cast<__bf16>(out[2]), static_cast<__bf16>(out[3])};
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(words2, r), y_rsrc, at, tile_at, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(words4, out), y_rsrc, at, tile_at, 0);
        }
    };
    for (uint32_t t0 = 0;;) {
        floatx4 acc[MR][QT];
#pragma unroll
        for (uint32_t m = 0; m < MR; ++m)
#pragma unroll
            for (uint32_t q = 0; q < QT; ++q) acc[m][q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (!kEarly) request_first();
        auto use = [&](uint32_t d) {                              // the unit in slot d
            uint32_t a_step = a_at + k_use * 2u;
#pragma unroll
            for (uint32_t sx = 0; sx < NS; ++sx) {
                auto operand = [&](uint32_t q) {                  // (q is a constant once unrolled)
                    if constexpr (MODE != kShift) return ring[d][sx][q];
                    if (sx == 1u) return ring[d][0][q];
                    if (sx == 0u) return q ? neighbours<true, true>(ring[d][0][q], ring[d][0][q ? q - 1u : 0u], not_left[q])
                                           : neighbours<true, false>(ring[d][0][q], edge[d], not_left[q]);
                    return q + 1u < QT ? neighbours<false, true>(ring[d][0][q], ring[d][0][q + 1u < QT ? q + 1u : q], not_right[q])
                                       : neighbours<false, false>(ring[d][0][q], edge[d], not_right[q]);
                };
                bf16x8 a[MR];
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m) a[m] = lds_load<bf16x8>(a_step + m * tile_stride);
                auto multiply = [&](uint32_t q) {
                    const bf16x8 b = __builtin_bit_cast(bf16x8, operand(q));
#pragma unroll
                    for (uint32_t m = 0; m < MR; ++m) acc[m][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[m][q], 0, 0, 0);
                };
#pragma unroll
                for (uint32_t q = 0; q + 1u < QT; ++q) multiply(q);
                if (has_last) multiply(QT - 1u);                  // (uniform)
                a_step += p.cin * 2u;
            }
            ++use_cb;
            k_use += 32u;
            if constexpr (MODE != kPoint) {
                const bool next_row = use_cb == blocks;
                use_cb = next_row ? 0u : use_cb;
                k_use += next_row ? (TAIL ? NS * p.cin - 32u * blocks : 2u * p.cin) : 0u;
            }
        };
        uint32_t done = 0;
#pragma unroll 1
        for (; done + kSlots < n; done += kSlots) {
#pragma unroll
            for (uint32_t d = 0; d < kSlots; ++d) {
                use(d);
                request(d);
            }
        }
#pragma unroll
        for (uint32_t d = 0; d < kSlots; ++d)
            if (done + d < n) use(d);                             // (uniform: between the loads a branch would cost the compiler
                                                                  // its count of them, and every use would wait for all)
        if (p.k_groups == 1u) {
#pragma unroll
            for (uint32_t m = 0; m < MR; ++m)
#pragma unroll
                for (uint32_t q = 0; q < QT; ++q) store(m, out_at[q], acc[m][q]);
            t0 += p.round_tiles;
            if (split_begin + 16u * t0 >= split_end) break;
            place(t0);
            if constexpr (kEarly) request_first();
        } else {
            // One round.  Every wavefront leaves its sums in LDS, 1 KiB per tile and row tile ([slice][tile range][q][m]);
            // the wavefronts then take the blocks in turn, add up the slices' and store.
            const uint32_t block_bytes = kWave * 16u, slice_bytes = p.t_groups * QT * MR * block_bytes;
            __syncthreads();                                      // every wavefront has read what it needs of the panel
            const uint32_t mine = lds_address(lds) + wk * slice_bytes + wt * (QT * MR * block_bytes) + lane * 16u;
#pragma unroll
            for (uint32_t q = 0; q < QT; ++q)
#pragma unroll
                for (uint32_t m = 0; m < MR; ++m) lds_store<floatx4>(mine + (q * MR + m) * block_bytes, acc[m][q]);
            __syncthreads();
            const uint32_t n_blocks = p.t_groups * QT * MR;
#pragma unroll 1
            for (uint32_t i = wave; i < n_blocks; i += kWaves) {
                const uint32_t m = i % MR, tq = i / MR, g = tq / QT, q = tq - g * QT;        // (constants)
                const uint32_t tile = first_tile(g) + q, pix = split_begin + 16u * tile + col;
                uint32_t b, ho, wo;
                const uint32_t at = pixel_of(pix, tile < first_tile(g + 1u) ? split_end : 0u, b, ho, wo);
                uint32_t part = lds_address(lds) + i * block_bytes + lane * 16u;
                floatx4 sum = lds_load<floatx4>(part);
#pragma unroll 1
                for (uint32_t j = 1; j < p.k_groups; ++j) {
                    part += slice_bytes;
                    sum += lds_load<floatx4>(part);
                }
                store(m, at, sum);
            }
            break;
        }
    }
}

typedef void (*ConvKernel)(ConvParams);
template <uint32_t ROWS, bool P16, uint32_t MODE, bool TAIL>
ConvKernel sliced_kernel(uint32_t qt) {
    if constexpr (most_tiles(ROWS < kRows ? 1u : ROWS / kRows, MODE) == 4u) {
        if (qt == 4u) return conv_sliced_kernel<ROWS, P16, MODE, 4, TAIL>;
    }
    return qt == 3u ? conv_sliced_kernel<ROWS, P16, MODE, 3, TAIL> : qt == 2u ? conv_sliced_kernel<ROWS, P16, MODE, 2, TAIL> : conv_sliced_kernel<ROWS, P16, MODE, 1, TAIL>;
}
template <uint32_t ROWS, bool P16, bool TAIL>
ConvKernel sliced_kernel(uint32_t mode, uint32_t qt) {
    return mode == kPoint ? sliced_kernel<ROWS, P16, kPoint, TAIL>(qt) : mode == kShift ? sliced_kernel<ROWS, P16, kShift, TAIL>(qt) : sliced_kernel<ROWS, P16, kRow, TAIL>(qt);
}
template <bool TAIL>
ConvKernel sliced_kernel(uint32_t rows, bool p16, uint32_t mode, uint32_t qt) {
    if (rows < kRows) return sliced_kernel<kRows / 2u, true, TAIL>(mode, qt);
    return p16 ? (rows == 64u ? sliced_kernel<64, true, TAIL>(mode, qt) : rows == 32u ? sliced_kernel<32, true, TAIL>(mode, qt) : sliced_kernel<16, true, TAIL>(mode, qt))
               : (rows == 64u ? sliced_kernel<64, false, TAIL>(mode, qt) : rows == 32u ? sliced_kernel<32, false, TAIL>(mode, qt) : sliced_kernel<16, false, TAIL>(mode, qt));
}

template <bool TAIL>
bool allow_all_lds() {
    for (uint32_t mode = kPoint; mode <= kRow; ++mode)
        for (const uint32_t rows : {8u, 16u, 32u, 64u})
            for (uint32_t qt = 1; qt <= most_tiles(std::max(1u, rows / kRows), mode); ++qt)
                for (const bool p16 : {false, true})
                    if (hipFuncSetAttribute(reinterpret_cast<const void*>(sliced_kernel<TAIL>(rows, p16, mode, qt)), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
                        return false;
    return true;
}

int launch_sliced(const ConvParams& p, uint32_t rows, bool p16, uint32_t mode, uint32_t qt, int device, uint32_t groups, uint32_t lds_bytes, hipStream_t s) {
    const bool tail = p.cin % 32u != 0u;
    const ConvKernel kernel = tail ? sliced_kernel<true>(rows, p16, mode, qt) : sliced_kernel<false>(rows, p16, mode, qt);
    // the kernels may use all of the CU's LDS: said for all of them by a device's first call, because which one a layer gets
    // depends on the batch too, and a call may be captured whose layer ran before with another batch (concurrent first callers
    // at worst both say it)
    static std::atomic<bool> allowed[64];
    if (device < 0 || device >= 64) return ANSZP_E_HIP;
    if (!allowed[device].load(std::memory_order_acquire)) {
        if (!allow_all_lds<false>() || !allow_all_lds<true>()) return ANSZP_E_HIP;
        allowed[device].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), std::max(lds_bytes, kLeastLds), s, p);
    return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
}

Reciprocal reciprocal(uint32_t d) {
    const uint32_t shift = d > 1u ? 32u - uint32_t(__builtin_clz(d - 1u)) : 0u;
    return {uint32_t((1ull << (31 + shift)) / d + 1u), shift};
}

// The whole call in launches of at most `images` images.
int conv_sliced(ConvParams p, const anszp_conv_args_t& a, uint32_t images, uint32_t cus, int device, hipStream_t s) {
    p.x_image = a.in_h * a.in_w * a.cin;
    p.y_image = p.out_h * p.out_w * a.cout;
    p.panel_off = kStageBytes + (16u << a.table_log);
    auto magic = [](uint32_t d, uint32_t& m, uint32_t& shift) {
        const Reciprocal r = reciprocal(d);
        m = r.magic;
        shift = r.shift;
    };
    magic(p.out_h, p.out_h_magic, p.out_h_shift);
    magic((a.cin + 31u) / 32u, p.blocks_magic, p.blocks_shift);
    for (uint32_t first = 0; first < a.batch; first += images) {
        const uint32_t n = std::min(images, a.batch - first);
        p.x = a.x + uint64_t(first) * p.x_image;
        p.y = static_cast<uint8_t*>(a.y) + uint64_t(first) * p.y_image * (p.y_bf16 ? 2u : 4u);
        p.x_bytes = uint32_t(uint64_t(n) * p.x_image * 2u);
        p.y_bytes = uint32_t(uint64_t(n) * p.y_image * (p.y_bf16 ? 2u : 4u));
        const CallPlan call = plan_call(a, p.K, p.row_stride, p.out_h, p.out_w, n, cus);
        const SlicedPlan& plan = call.plan;
        if (!plan.mr) return ANSZP_E_RANGE;
        p.first_column = call.first_column;
        p.columns = call.columns;
        magic(p.columns, p.columns_magic, p.columns_shift);
        p.n_pixels = n * p.out_h * p.columns;
        p.n_mtiles = a.cout / plan.rows;
        magic(p.n_mtiles, p.n_mtiles_magic, p.n_mtiles_shift);
        p.chunks_per_panel = plan.rows / a.rows_per_chunk;
        p.pixels_per_split = 16u * plan.tiles_per_split;
        p.k_groups = plan.k_groups;
        p.t_groups = kWaves / plan.k_groups;
        p.t_groups_inv = 65536u / p.t_groups + 1u;
        p.wave_tiles = plan.round_tiles / p.t_groups;
        p.wave_tiles_rest = plan.round_tiles % p.t_groups;
        p.round_tiles = plan.round_tiles;
        p.slice_units = plan.slice_units;
        const int rc = launch_sliced(p, plan.rows, plan.p16, call.mode, plan.qt, device, p.n_mtiles * plan.splits, plan.lds_bytes, s);
        if (rc != ANSZP_OK) return rc;
    }
    return ANSZP_OK;
}

constexpr uint32_t kMaxK16 = 576;          // up to here 64 rows fit as bf16 (73 KiB), and no conversion is left in the loop

}  // namespace

extern "C" int anszp_conv_fused(const anszp_conv_args_t* a, void* stream) {
    if (!a || !a->tables || !a->chunks || !a->stream_hdr || !a->layers || !a->x || !a->y || !a->status) return ANSZP_E_NULL;
    if (a->payload_words && !a->payload) return ANSZP_E_NULL;
    if (a->table_log < 1 || a->table_log > ANSZP_MAX_TABLE_LOG || a->n_streams < 1 || a->n_streams > 64) return ANSZP_E_RANGE;
    if (a->layer_id >= a->n_tables) return ANSZP_E_RANGE;
    if (a->y_dtype != ANSZP_OUT_F32 && a->y_dtype != ANSZP_OUT_BF16) return ANSZP_E_RANGE;
    if (!a->batch || !a->in_h || !a->in_w || !a->cin || !a->cout || !a->kh || !a->kw || !a->stride) return ANSZP_E_RANGE;
    if (a->in_h > 32768u || a->in_w > 32768u || a->cin > 65536u || a->kh > 64u || a->kw > 64u || a->pad > 64u) return ANSZP_E_RANGE;
    if (a->cout % kRows) return ANSZP_E_RANGE;
    const uint64_t K = uint64_t(a->cin) * a->kh * a->kw;
    if (K > kMaxK) return ANSZP_E_RANGE;
    if (a->in_h + 2u * a->pad < a->kh || a->in_w + 2u * a->pad < a->kw) return ANSZP_E_RANGE;
    const uint32_t R = a->rows_per_chunk;
    if (R == 0 || R > kRows || (kRows % R)) return ANSZP_E_RANGE;
    const uint32_t out_h = (a->in_h + 2u * a->pad - a->kh) / a->stride + 1u;
    const uint32_t out_w = (a->in_w + 2u * a->pad - a->kw) / a->stride + 1u;
    const uint64_t n_pixels = uint64_t(a->batch) * out_h * out_w;
    if (n_pixels >= (1ull << 31) || uint64_t(a->batch) * a->in_h * a->in_w >= (1ull << 31)) return ANSZP_E_RANGE;
    if (uint64_t(a->batch) * a->in_h * a->in_w * a->cin >= (1ull << 32) || n_pixels * a->cout >= (1ull << 32))
        return ANSZP_E_RANGE;                                    // elements of x and y are addressed with 32 bits
    if (a->x_layout > ANSZP_ACT_C8 || a->y_layout > ANSZP_ACT_C8) return ANSZP_E_RANGE;
    if (a->x_layout == ANSZP_ACT_C8 && (a->cin % 8u) != 0) return ANSZP_E_RANGE;
    if (a->n_chunks < a->cout / R) return ANSZP_E_RANGE;
    if ((reinterpret_cast<uintptr_t>(a->x) | reinterpret_cast<uintptr_t>(a->y) | reinterpret_cast<uintptr_t>(a->payload) |
         reinterpret_cast<uintptr_t>(a->tables)) & 15u) return ANSZP_E_RANGE;

    ConvParams p{};
    p.tables = a->tables; p.chunks = a->chunks; p.stream_hdr = a->stream_hdr; p.payload = a->payload;
    p.layers = a->layers; p.scales = a->scales; p.x = a->x; p.y = a->y; p.status = a->status;
    p.y_bf16 = a->y_dtype == ANSZP_OUT_BF16;
    p.n_stream_hdr = a->n_stream_hdr; p.payload_words = a->payload_words; p.n_scales = a->scales ? a->n_scales : 0;
    p.layer_id = a->layer_id; p.table_log = a->table_log; p.n_streams = a->n_streams;
    p.rows_per_chunk = R;
    p.in_h = a->in_h; p.in_w = a->in_w; p.cin = a->cin; p.cout = a->cout; p.kh = a->kh; p.kw = a->kw;
    p.stride = a->stride; p.pad = a->pad; p.out_h = out_h; p.out_w = out_w;
    p.x_pixel = a->x_layout == ANSZP_ACT_C8 ? 8u : a->cin;
    p.x_block = a->x_layout == ANSZP_ACT_C8 ? 8u * a->in_h * a->in_w : 8u;
    p.y_pixel = a->y_layout == ANSZP_ACT_C8 ? 8u : a->cout;
    p.y_block = a->y_layout == ANSZP_ACT_C8 ? 8u * out_h * out_w : 8u;
    p.K = uint32_t(K);
    p.k_magic = uint32_t((uint64_t(1) << 32) / K) + 1u;           // unused for K = 1
    p.row_of = row_reciprocal(uint32_t(K));
    const uint32_t row_stride = ((uint32_t(K) + 31u) & ~31u) + kRowPad, table_bytes = 16u << a->table_log;      // (the look-ahead entries)
    p.row_stride = row_stride;
    p.n_pixels = uint32_t(n_pixels);

    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return ANSZP_E_HIP;
    const uint32_t cus = device_cus(device);
    const bool generic = (a->cin % 8u) != 0;
    const bool pointwise = !generic && a->kh == 1 && a->kw == 1 && a->pad == 0;
    if (!generic && (pointwise || a->kw == 3)) {
        // buffer offsets are 31 bits: as many images at a time as x and y of that size allow (all of them, but for very large calls)
        const uint64_t x_image = uint64_t(a->in_h) * a->in_w * a->cin, y_image = uint64_t(out_h) * out_w * a->cout;
        const uint64_t most = ((1ull << 31) - 1u) / std::max(2u * x_image, (p.y_bf16 ? 2u : 4u) * y_image);
        if (most) return conv_sliced(p, *a, uint32_t(std::min<uint64_t>(most, a->batch)), cus, device, static_cast<hipStream_t>(stream));
    }
    // Row tiles per workgroup: as many of 4, 2, 1 as divide the output channels and leave the panel room in LDS
    // beside the table and the staging buffers (more rows per activation vector loaded).
    const uint32_t fixed_bytes = kStageBytes + table_bytes + 64u;
    const bool p16 = K <= kMaxK16;                              // short rows: the panel as bf16
    const uint32_t elem = p16 ? 2u : 1u;
    uint32_t mr = 4;
    while (mr > 1 && ((a->cout % (kRows * mr)) != 0 || fixed_bytes + kRows * mr * row_stride * elem > kLdsLimit)) mr >>= 1;
    const uint32_t n_mtiles = a->cout / (kRows * mr);
    p.chunks_per_panel = kRows * mr / R;
    p.n_mtiles = n_mtiles;
    const Reciprocal by_panels = reciprocal(n_mtiles);
    p.n_mtiles_magic = by_panels.magic;
    p.n_mtiles_shift = by_panels.shift;
    p.by_out_w = reciprocal(out_w);
    p.by_out_h = reciprocal(out_h);
    p.by_cin = reciprocal(a->cin);
    p.by_kw = reciprocal(a->kw);
    // Every workgroup decodes its panel once, so few, long-lived workgroups: as many as are resident at once,
    // which is one per CU (twelve wavefronts of more than 128 VGPRs fill a CU's four SIMDs whatever the LDS
    // would allow).  A panel's pixels are dealt out in column tiles of 16, evenly over the workgroups that
    // share the panel.
    const uint32_t lds_bytes = fixed_bytes + kRows * mr * row_stride * elem;
    const uint32_t n_tiles = uint32_t((n_pixels + 15u) / 16u);
    uint32_t splits = (cus + n_mtiles - 1u) / n_mtiles;
    if (splits > n_tiles) splits = n_tiles;
    if (splits == 0) splits = 1;
    const uint32_t tiles_per_split = (n_tiles + splits - 1u) / splits;
    splits = (n_tiles + tiles_per_split - 1u) / tiles_per_split;
    p.pixels_per_split = 16u * tiles_per_split;
    const uint32_t tiles_per_wave = (tiles_per_split + kWaves - 1u) / kWaves;
    p.block_pixels = 16u * (tiles_per_wave < 4u ? tiles_per_wave : 4u);

    // (fixed_bytes counts 64 bytes beyond the panel: the last 32 k of a kernel tap may reach past the end of the last row)
    const uint32_t panel_bytes = kRows * mr * row_stride * elem;
    uint32_t lds_total = lds_bytes;
    p.panel_off = kStageBytes + table_bytes;
    bool generic_patch = false;
    if (generic) {
        // image rows that are multiples of 16 bytes, or of whole words where the reduction is more than one step of 32 k (NHWC; with every
        // activation on its own and from LDS, us, both with the divisions that are reciprocals now: 64 x 3 x 7 x 7 on 60 212 x 212 images 91.5, 47.0, on one of 134 x 134 12.1, 8.1; of 50
        // calls with 1 to 60 channels and kernels of 1 to 7 the 18 of at most 32 k that could change took 0.1 to 0.6 longer, but for three,
        // the 20 others went 1.07 to 2.1 times as fast, one 1.00): the rows under a round of pixels staged in LDS, if the most
        // rows a round can need fit below the panel (after the table of k offsets) and in pieces per thread
        const uint32_t Kp = (uint32_t(K) + 31u) & ~31u;
        const uint64_t row_bytes = uint64_t(a->in_w) * a->cin * 2u;
        const uint64_t row_pitch = (32u + row_bytes + uint64_t(a->pad) * a->cin * 2u + 15u) & ~uint64_t(15);
        if (a->x_layout == ANSZP_ACT_NHWC && (row_bytes % 16u == 0 || (row_bytes % 4u == 0 && row_bytes >= 16u && K > 32u)) && uint64_t(a->pad) * a->cin * 2u <= 32u && row_pitch < (1u << 20) && uint64_t(a->batch) * (a->in_h + 2u * a->pad) < (1ull << 31)) {
            const uint32_t S = a->stride, Hp = a->in_h + 2u * a->pad;
            const int64_t gap = int64_t(Hp) - int64_t(out_h) * S;
            const uint64_t tiles = (p.pixels_per_split + 15u) / 16u;
            const uint64_t n_rounds = (tiles + 4u * kWaves - 1u) / (4u * kWaves);
            const uint64_t round = ((tiles + n_rounds - 1u) / n_rounds) * 16u;
            const uint64_t rows_out = (round + out_w - 2u) / out_w + 1u;
            const uint64_t crossings = std::min<uint64_t>(a->batch - 1u, (rows_out + out_h - 2u) / out_h);
            const uint64_t rows = (rows_out - 1u) * S + a->kh + crossings * uint64_t(gap > 0 ? gap : 0);
            const uint64_t k_table_bytes = (uint64_t(Kp) * 4u + 63u) & ~uint64_t(63);
            const uint64_t below = std::max<uint64_t>(p.panel_off, k_table_bytes + rows * row_pitch);
            if (rows * ((row_bytes + 15u) / 16u) <= kPatchPieces * kThreads && below + panel_bytes + 64u <= kLdsLimit) {
                generic_patch = true;
                p.row_pitch = uint32_t(row_pitch);
                p.by_pieces = reciprocal(uint32_t((row_bytes + 15u) / 16u));
                p.by_edges = reciprocal(uint32_t((row_pitch - row_bytes) / 4u));
                p.by_padded_h = reciprocal(Hp);
                p.patch_off = uint32_t(k_table_bytes);
                p.panel_off = uint32_t((below + 15u) & ~uint64_t(15));
                lds_total = p.panel_off + panel_bytes + 64u;
            }
        }
        if (!generic_patch) {                                     // room for the table of the k below the panel
            const uint32_t k_table_bytes = Kp * 8u;
            if (p.panel_off < k_table_bytes) {
                p.panel_off = k_table_bytes;
                lds_total = p.panel_off + panel_bytes + 64u;
                if (lds_total > kLdsLimit) return ANSZP_E_RANGE;
            }
        }
    }
    // other kernels of several taps: the ring of loads, if the channels allow whole groups of steps per tap and a
    // step's stride fits a 24-bit multiplication
    const bool taps_ring = !generic && !pointwise && (a->cin % 64u) == 0 && 4ull * p.x_block < (1u << 24) &&
                           (p16 || (panel_bytes + 64u <= kWidenPieces * kThreads * 16u && 2u * (panel_bytes + 64u) <= kLdsLimit));
    if (taps_ring && !p16 && lds_total < 2u * (panel_bytes + 64u)) lds_total = 2u * (panel_bytes + 64u);
    const uint32_t taps_depth = taps_ring ? ((a->cin % 128u) == 0 ? 4u : 2u) : 0u;
    const int kind = generic_patch ? kGenericPatch : generic ? kGeneric : taps_ring ? kTapsRing : pointwise ? kPointwise : kTaps;
    void (*kernel)(ConvParams) = nullptr;
#define ANSZP_CONV_PICK(KIND, D)                                                                                       \
    (p16 ? (mr == 4 ? conv_fused_kernel<KIND, 4, true, D> : mr == 2 ? conv_fused_kernel<KIND, 2, true, D> : conv_fused_kernel<KIND, 1, true, D>) \
         : (mr == 4 ? conv_fused_kernel<KIND, 4, false, D> : mr == 2 ? conv_fused_kernel<KIND, 2, false, D> : conv_fused_kernel<KIND, 1, false, D>))
    kernel = kind == kGeneric ? ANSZP_CONV_PICK(kGeneric, 0) : kind == kPointwise ? ANSZP_CONV_PICK(kPointwise, 0)
           : kind == kTaps ? ANSZP_CONV_PICK(kTaps, 0) : kind == kGenericPatch ? ANSZP_CONV_PICK(kGenericPatch, 0)
           : taps_depth == 4 ? ANSZP_CONV_PICK(kTapsRing, 4) : ANSZP_CONV_PICK(kTapsRing, 2);
#undef ANSZP_CONV_PICK
    // the kernels may use all of the CU's LDS: said once per kernel and device (a table of atomics:
    // concurrent callers at worst both say it)
    static std::atomic<bool> lds_allowed[2][6][3][64];
    const uint32_t slot = mr == 4 ? 2u : mr == 2 ? 1u : 0u;
    const uint32_t kernel_no = kind == kTapsRing && taps_depth == 4 ? 5u : uint32_t(kind);
    if (device < 0 || device >= 64) return ANSZP_E_HIP;
    if (!lds_allowed[p16][kernel_no][slot][device].load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                int(kLdsLimit)) != hipSuccess) return ANSZP_E_HIP;
        lds_allowed[p16][kernel_no][slot][device].store(true, std::memory_order_relaxed);
    }
    lds_total = std::max(lds_total, kLeastLds);                   // (what kStageMask leaves of an address is always there)
    hipLaunchKernelGGL(kernel, dim3(n_mtiles * splits), dim3(kThreads), lds_total, static_cast<hipStream_t>(stream), p);
    return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
}
