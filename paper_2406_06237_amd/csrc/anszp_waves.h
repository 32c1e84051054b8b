// Many short chunks: a wavefront per chunk, the table shared by a workgroup (internal to the library; included by the
// decode kernels' source, whose names it uses).
//
// The look-ahead kernel stages a table for every one or two chunks and spreads a chunk's work over several wavefronts, so
// that one chunk is done as soon as possible.  With several rounds of such workgroups per CU neither pays: what counts is
// what a CU gets done, and staging (up to 64 KiB of entries per workgroup, 4 us) is most of it where chunks are short.
// Here a workgroup fills a CU and takes a share of the chunks; it stages a layer's entries once, and every
// wavefront takes the next chunk by itself: its stream words to LDS (first bit on top), look-ups (walk_entries), symbols to a
// buffer in LDS that holds the dominant symbol as background (a look-up writes the last of its symbols), and from there,
// converted, 16 bytes per lane to memory.  A chunk longer than the buffer is decoded in windows of the buffer's length:
// lanes stop at its end, and what a last look-up wrote behind it (up to 8 symbols of each stream) begins the next.
// No wavefront waits for another but at a change of layer.
//
// The shares: descriptors may come in any order and chunks of any size.  Where layers follow each other and their chunks
// have like numbers of words, as a packer leaves them, a share is a run of consecutive descriptors.  Every workgroup looks at
// the same sample of the descriptors to see whether that holds.  If not, it sorts them (by layer, in LDS) and takes a share of
// equal weight, so that a layer's chunks meet in few workgroups and long chunks do not meet in one (waves_share).
// A chunk with more words than its wavefront's part of LDS holds waits for a second turn, of fewer wavefronts with more each.
// Measured with a plan, bf16 out, 64 streams, 48 layers (look-ahead kernel -> here):
//   layers in a row: chunks of 2,048 symbols, 2^12 states, 1,104 of them 20 -> 9.8 us, 2,304 33 -> 15.5, 9,600 224 -> 31; 4,096 symbols
//   of 2 bits, 2^10 states, 9,600 144 -> 36; 16,384 symbols, 2^12 states, 1,104 31 -> 26, 2,304 52 -> 45.
//   descriptors in any order: 30 -> 19, 53 -> 26, 228 -> 58; 149 -> 63; 47 -> 33, 88 -> 54 (all as descriptors in a row 32, 52, 225;
//   264; 102, 186).  Working out the shares takes a call 8 us, finding out that it need not 0.3.
//   chunks of 8,192 symbols of half a bit and some of 8 bits in a row, 2^12 states: 9,000 and 300 215 -> 75, 2,200 and 100 33 -> 33 (as
//   descriptors in a row, with words that did not fit read from memory, 328 and 76); 1,000 and 60 21 -> 31, of 32,768 symbols
//   36 -> 76 (198): a long chunk has one wavefront here, seven there.
//   9,600 chunks of 2,048 symbols, 1,000 of them layers of their own: 220 -> 75 (268).
#ifndef ANSZP_WAVES_H
#define ANSZP_WAVES_H

#include "anszp_walk.h"

constexpr uint32_t kWavesLookers = 4u;                     // wavefronts that look at a sample of the descriptors
constexpr uint32_t kWavesKeys = 1024u;                     // layers are told apart by so many of their number's values while they are sorted
constexpr uint32_t kWavesList = 1024u;                     // chunks of a share that are listed at once
constexpr uint32_t kWavesListBytes = kWavesList * 2u;      // at the end of LDS
constexpr uint32_t kWavesLeastUnits = 16u, kWavesMostUnits = 1023u;
constexpr uint32_t kWavesWindow = 15000u;                  // units listed at once: with what moves a window's ends (at most 15 mean
static_assert((kWavesWindow + 2u * 15u * 32u) / kWavesLeastUnits + 2u <= kWavesList, "a window's chunks fit the list");      // chunks each)
constexpr uint32_t kWavesSorted = 16384u;                  // most chunks sorted at once (64 KiB)

// How far (in chunks) a share's ends may move to where a layer ends: a layer more in a share is a table more to stage and,
// with fewer chunks than wavefronts, a chunk's time more.
__device__ __forceinline__ uint32_t waves_reach(uint32_t share, uint32_t waves) {
    return min(15u, share < waves ? min(share / 2u + 1u, (waves - share + 1u) / 2u) : share / 8u);
}

// A workgroup's share of the descriptors base .. base + count - 1 (count <= kWavesSorted) where they are in no useful order
// or of very different sizes: laid out layer after layer (a layer: stage_units, then its chunks in the order of their descriptors)
// they have a length in units, of which every workgroup takes an equal piece.  Lists the piece's chunks (numbers from
// base on, 16 bits, layer after layer, a layer's largest first) at `list`; all threads get how many there are.  A piece too
// long for the list comes in several windows: `more` says that there is another.  What decides where a piece ends is
// worked out from the same numbers by both workgroups it lies between (sums, and an order by number: no atomics' order), so
// every chunk is in one share.
__device__ __forceinline__ uint32_t waves_share(const DecodeParams& p, const WavesShape& shape, uint8_t* lds, uint16_t* list, uint32_t base, uint32_t count,
                                                uint32_t window, bool& more) {
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6), threads = blockDim.x, waves = threads / kWave;
    uint32_t* const code = reinterpret_cast<uint32_t*>(lds);                   // key << 20 | units of every chunk
    uint32_t* const sum = code + kWavesSorted;                                  // units of every key's chunks
    uint32_t* const sorts = sum + kWavesKeys;                                   // of the listed: what they are sorted by
    uint16_t* const listed = reinterpret_cast<uint16_t*>(sorts + kWavesList);
    uint32_t* const part = sorts + kWavesList + kWavesList / 2u;                // wavefronts' sums, two rows
    uint32_t* const bound = part + 32u;                                         // key and units to skip of both ends; where that is; how many are listed
    __syncthreads();                                        // (what lies there has been used)
    for (uint32_t k = tid; k < kWavesKeys; k += threads) sum[k] = 0u;
    if (tid < 8u) bound[tid] = tid < 4u ? (tid & 1u ? 0u : kWavesKeys) : tid < 6u ? count : 0u;       // (an end nobody finds is the last one)
    __syncthreads();
    for (uint32_t i = tid; i < count; i += threads) {
        const uint32_t layer = p.chunks[base + i].layer_id, words = p.chunks[base + i].payload_words;
        const uint64_t cost = (uint64_t(words) + shape.fixed) * shape.unit_scale >> 16;
        const uint32_t units = min(max(static_cast<uint32_t>(min(cost, uint64_t(kWavesMostUnits))), kWavesLeastUnits), kWavesMostUnits);
        const uint32_t key = min(layer, p.n_tables) % kWavesKeys;
        code[i] = key << 20 | units;
        atomicAdd(&sum[key], units);
    }
    __syncthreads();
    // where every key's chunks begin, and the ends of this share among them
    const uint32_t share = count / gridDim.x, reach = 32u * waves_reach(share, waves);
    const uint32_t stage = min(shape.stage_units, 16u * share);                 // (no share may be nothing but tables)
    {
        const uint32_t per = (kWavesKeys + threads - 1u) / threads, k0 = tid * per, k1 = min(k0 + per, kWavesKeys);
        uint32_t mine = 0, all;
        for (uint32_t k = k0; k < k1; ++k) mine += sum[k] ? sum[k] + stage : 0u;
        uint32_t at = wave_exclusive_sum(mine, &all);
        if (lane == 0) part[wave] = all;
        __syncthreads();
        uint32_t total = 0;
        for (uint32_t w = 0; w < waves; ++w) {
            at += w < wave ? part[w] : 0u;
            total += part[w];
        }
        const uint32_t lo = static_cast<uint32_t>(uint64_t(total) * blockIdx.x / gridDim.x), hi = static_cast<uint32_t>(uint64_t(total) * (blockIdx.x + 1u) / gridDim.x);
        const uint32_t x0 = lo + min(window * kWavesWindow, hi - lo), x1 = x0 + min(kWavesWindow, hi - x0);
        more = x1 < hi;
        for (uint32_t k = k0; k < k1; ++k) {
            const uint32_t s = sum[k];
            if (!s) continue;
            const uint32_t size = s + stage;
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e) {
                const uint32_t d = (e ? x1 : x0) - at;      // (wraps around below)
                if (d >= size) continue;
                const bool to_start = d < stage + reach, to_end = size - d < reach;
                bound[2u * e] = !to_start && to_end ? k + 1u : k;
                bound[2u * e + 1u] = to_start || to_end ? 0u : d - stage;
            }
            at += size;
        }
    }
    __syncthreads();
    const uint32_t key0 = bound[0], skip0 = bound[1], key1 = bound[2], skip1 = bound[3];
    if (skip0 | skip1) {                                    // inside a layer: the first of its chunks that is beyond that many units of it
        const uint32_t per = (count + threads - 1u) / threads | 1u, i0 = tid * per, i1 = min(i0 + per, count);
        uint32_t s0 = 0, s1 = 0, all0, all1;
        for (uint32_t i = i0; i < i1; ++i) {
            const uint32_t c = code[i], key = c >> 20, units = c & 0xFFFFFu;
            s0 += key == key0 ? units : 0u;
            s1 += key == key1 ? units : 0u;
        }
        s0 = wave_exclusive_sum(s0, &all0);
        s1 = wave_exclusive_sum(s1, &all1);
        if (lane == 0) { part[wave] = all0; part[16u + wave] = all1; }
        __syncthreads();
        for (uint32_t w = 0; w < wave; ++w) { s0 += part[w]; s1 += part[16u + w]; }
        uint32_t found0 = count, found1 = count;
        for (uint32_t i = i0; i < i1; ++i) {
            const uint32_t c = code[i], key = c >> 20, units = c & 0xFFFFFu;
            if (key == key0) {
                if (s0 >= skip0) found0 = min(found0, i);
                s0 += units;
            }
            if (key == key1) {
                if (s1 >= skip1) found1 = min(found1, i);
                s1 += units;
            }
        }
        if (found0 < count) atomicMin(&bound[4], found0);
        if (found1 < count) atomicMin(&bound[5], found1);
        __syncthreads();
    }
    const uint32_t from0 = skip0 ? bound[4] : 0u, upto1 = skip1 ? bound[5] : 0u;
    for (uint32_t i = tid; i < count; i += threads) {
        const uint32_t c = code[i], key = c >> 20;
        if ((key > key0 || (key == key0 && i >= from0)) && (key < key1 || (key == key1 && i < upto1))) {
            const uint32_t slot = atomicAdd(&bound[6], 1u);
            if (slot < kWavesList) {
                sorts[slot] = c ^ 0xFFFFFu;
                listed[slot] = static_cast<uint16_t>(i);
            }
        }
    }
    __syncthreads();
    const uint32_t n = min(bound[6], kWavesList);
    for (uint32_t j = tid; j < n; j += threads) {
        const uint32_t v = sorts[j];
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t q = 0; q < n; ++q) rank += sorts[q] < v || (sorts[q] == v && q < j) ? 1u : 0u;
        list[rank] = listed[j];
    }
    __syncthreads();
    return n;
}

// Most words of a chunk that `own` bytes of LDS hold beside the least buffer.
__device__ __forceinline__ uint32_t waves_words(uint32_t own) { return (own - kWavesLeastRoom - kWavesBehind - 16u) / 4u - kWavesPad; }

// What a run of chunks of one layer shares.
struct WavesLayer {
    const uint32_t* src;                                    // the table as it comes
    anszp_layer_t lay;
    uint32_t layer_id, bg;                                  // the buffers' background: four times the dominant symbol
};

// Stages the table of layer `layer_id` and finds how many of the chunks index_of(first) ... index_of(last - 1) in a row are of
// that layer (ctl[1]) and the most words of those that have more than `fits` (ctl[2], or 0).  beside() is called while the table
// is on its way; ctl[3] is 0 before it.
template <class INDEX_OF, class BESIDE>
__device__ __forceinline__ WavesLayer waves_stage(const DecodeParams& p, uint8_t* lds, uint32_t* ctl, uint32_t layer_id, uint32_t first, uint32_t last, uint32_t fits,
                                                  INDEX_OF&& index_of, BESIDE&& beside) {
    const uint32_t tid = threadIdx.x, threads = blockDim.x, L = 1u << p.table_log, table_at = lds_address(lds);
    const uint32_t look = min(last - first, threads);
    __syncthreads();                                        // (the run before this one is done)
    if (tid == 0) { ctl[0] = 0u; ctl[1] = look; ctl[2] = 0u; ctl[3] = 0u; }
    __syncthreads();
    const bool known = layer_id < p.n_tables;
    WavesLayer w;
    w.src = p.tables + size_t(known ? layer_id : 0u) * table_stride_words(p.table_log);
    const uint4* const entries = reinterpret_cast<const uint4*>(w.src + table_lookahead_offset(p.table_log));
    for (uint32_t i = tid; i < L; i += threads) reinterpret_cast<uint4*>(lds)[i] = walk_entry_pair(entries[i], table_at);
    beside();
    if (tid < look) {
        const anszp_chunk_t& c = p.chunks[index_of(first + tid)];
        if (c.layer_id != layer_id) atomicMin(&ctl[1], tid);
        else if (c.payload_words > fits) atomicMax(&ctl[2], c.payload_words);
    }
    w.lay = p.layers[known ? layer_id : 0u];
    w.layer_id = layer_id;
    w.bg = (w.src[table_triples_offset(p.table_log) + L - 1u] >> 24) * 0x01010101u;
    __syncthreads();
    return w;
}

// The chunks index_of(first) ... index_of(first + run - 1) with at most `fits` words (LONG: those with more), each by the next
// of `active` wavefronts that has time (ctl[0] counts them), in `own` bytes of LDS.
template <int OUT, bool LONG, class INDEX_OF>
__device__ __forceinline__ void waves_decode(const DecodeParams& p, uint8_t* lds, uint32_t* ctl, const WavesLayer& w, uint32_t own, uint32_t active, uint32_t fits,
                                             uint32_t first, uint32_t run, INDEX_OF&& index_of) {
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6);
    const uint32_t L = 1u << p.table_log, N = p.n_streams, table_bytes = 16u << p.table_log, table_at = lds_address(lds);
    const anszp_layer_t& lay = w.lay;
    const uint32_t* const src = w.src;
    const bool per_channel = lay.channel_len != 0u;
    const uint32_t bg = w.bg;
    // (a zero word, the chunk's words from a multiple of 16 bytes on, zeros)
    uint8_t* const place = lds + table_bytes + kWavesCtl + wave * own;
    uint32_t* const words = reinterpret_cast<uint32_t*>(place) + 3;
    const uint32_t q0 = 8u * lds_address(words) + 31u;      // bit b of the chunk is at q = q0 + b
    if (LONG && wave >= active) return;
    for (;;) {
        // (What lane 0 alone does at the end of a turn must not be joined with this: the compiler, seeing the same
        // condition, led the other lanes around both, found their number to be 0 and had them take chunk 0 for ever.)
        uint32_t who = lane, mine = 0;
        asm volatile("" : "+v"(who), "+v"(mine));
        if (who == 0u) mine = atomicAdd(&ctl[0], 1u);
        mine = uniform(mine);
        if (mine >= run) break;
        const anszp_chunk_t c = p.chunks[uniform(index_of(first + mine))];
        if ((c.payload_words > fits) != LONG) continue;
        if (!chunk_in_bounds(p, c) || !scales_in_bounds(p, lay, c)) {
            if (lane == 0) report(p.status, ANSZP_ST_BAD_DESC);
            continue;
        }
        if (c.n_symbols > (1u << 24) || c.payload_words > waves_words(own)) {      // the plain loop, like any chunk beyond its kernel's reach
            const uint32_t err = decode_chunk_stepwise<OUT>(p, c, lay, WordTable{src + table_triples_offset(p.table_log)}, lane);
            if (err && lane == 0) report(p.status, err);
            continue;
        }
        const uint32_t hdr = lane < N ? p.stream_hdr[c.stream_offset + lane] : 0u;
        const uint32_t total = c.payload_words;
        const uint32_t* const payload = p.payload + c.payload_offset;
        const uint32_t skew = static_cast<uint32_t>(c.out_offset) & 7u, n = c.n_symbols + skew;
        const uint32_t words_bytes = (4u * (total + kWavesPad) + 15u) & ~15u;
        uint8_t* const buf = place + words_bytes;
        const uint32_t buf_at = lds_address(buf), room = min((own - words_bytes - kWavesBehind) & ~15u, (n + 15u) & ~15u);
        {
            // (several loads under way: a long chunk would take a trip to memory for every KiB)
            constexpr uint32_t kLoads = LONG ? 8u : 2u;
            const uint32_t quads = total / 4u;
            for (uint32_t i0 = 0; i0 < quads; i0 += kLoads * kWave) {
                uint4 v[kLoads];
#pragma unroll
                for (uint32_t u = 0; u < kLoads; ++u) v[u] = reinterpret_cast<const uint4*>(payload)[min(i0 + u * kWave + lane, quads - 1u)];
#pragma unroll
                for (uint32_t u = 0; u < kLoads; ++u)
                    if (i0 + u * kWave + lane < quads)
                        reinterpret_cast<uint4*>(words + 1)[i0 + u * kWave + lane] = make_uint4(__brev(v[u].x), __brev(v[u].y), __brev(v[u].z), __brev(v[u].w));
            }
            const uint32_t i = 4u * quads + lane;           // the last words, and the zeros
            if (i < total + kWavesPad - 4u) words[1u + i] = i < total ? __brev(payload[i]) : 0u;
            if (lane == 0u) words[0] = 0u;
        }
        for (uint32_t i = lane * 16u; i < room + kWavesBehind; i += kWave * 16u) *reinterpret_cast<uint4*>(buf + i) = make_uint4(bg, bg, bg, bg);
        uint32_t all_words;
        const uint32_t first_word = wave_exclusive_sum(hdr >> 16, &all_words);
        uint32_t err = all_words != total ? ANSZP_ST_BAD_DESC : 0u;
        const uint32_t len = (lane < N && c.n_symbols > lane) ? (c.n_symbols - lane + N - 1u) / N : 0u;
        const uint64_t out_elem0 = c.out_offset - skew, layer_elem0 = out_elem0 - lay.out_base;
        const bool wide = per_channel && c.out_offset - lay.out_base + c.n_symbols >= (1ull << 32);      // (store8 numbers a layer's elements in 32 bits)
        // The streams: entry, bit, and the next symbol's position (counted from the multiple of 8 elements of the output
        // below the chunk's first).  The chunk's words end at q_end; a lane that has no more symbols stays behind every end.
        const uint32_t first_bit = 32u * min(first_word, total), q_end = q0 + 32u * total + 1u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t q = q0 + first_bit, at = table_at + 8u * (2u * (hdr & (L - 1u)) + (words[1u + (first_bit >> 5)] >> 31));
        uint32_t next = len ? skew + lane : n;
        for (uint32_t from = 0; from < n; from += room) {
            const uint32_t end = min(n - from, room);
            // an entry's last symbol is N positions before the stream's next
            uint32_t to = buf_at + next - from - N;
            const uint32_t to_end = buf_at + end - N;
            walk_entries<kWalkSpread, LONG>(at, q, to, q_end, to_end, N);      // (long chunks: few wavefronts at a time)
            next = to + N + from - buf_at;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // kStore symbols of a lane at a time, so that a wavefront's 16-byte stores lie one behind the other (fp32 with eight, two
            // stores side by side in every lane: 6,154 chunks of 6,192 symbols 82 us, 56 so)
            constexpr uint32_t kStore = OUT == ANSZP_OUT_F32 ? 4u : 8u;
            typedef typename std::conditional<OUT == ANSZP_OUT_F32, uint32_t, uint2>::type symbols_t;
            auto read = [&](uint32_t i) { return *reinterpret_cast<const symbols_t*>(buf + i); };
            auto clear = [&](uint32_t i) {
                if constexpr (OUT == ANSZP_OUT_F32) *reinterpret_cast<uint32_t*>(buf + i) = bg;
                else *reinterpret_cast<uint2*>(buf + i) = make_uint2(bg, bg);
            };
            auto store = [&](uint32_t i, const symbols_t s) {
                const uint32_t pos = from + i;
                if (__builtin_expect(pos >= skew && i + kStore <= end && !wide, 1)) {
                    if constexpr (OUT == ANSZP_OUT_F32) {
                        if (per_channel) Flusher<OUT, true>::store4(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                        else Flusher<OUT, false>::store4(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                    } else {
                        if (per_channel) Flusher<OUT, true>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                        else Flusher<OUT, false>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                    }
                } else {
#pragma unroll 1
                    for (uint32_t j = pos < skew ? skew - pos : 0u; j < kStore && i + j < end; ++j) {
                        uint32_t word;
                        if constexpr (OUT == ANSZP_OUT_F32) word = s;
                        else word = j < 4u ? s.x : s.y;
                        const uint32_t sym = (word >> (8u * (j & 3u))) & 0xFFu;
                        if (per_channel) Flusher<OUT, true>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                        else Flusher<OUT, false>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                    }
                }
            };
            if constexpr (LONG) {                           // (two reads under way; the second may lie behind the window, where there is room)
                for (uint32_t i = lane * kStore; i < end; i += 2u * kWave * kStore) {
                    const uint32_t i1 = i + kWave * kStore;
                    const symbols_t s0 = read(i), s1 = read(i1);
                    clear(i);
                    if (i1 < end) clear(i1);
                    store(i, s0);
                    if (i1 < end) store(i1, s1);
                }
            } else {                                        // (twice the code costs a call 0.2 us)
                for (uint32_t i = lane * kStore; i < end; i += kWave * kStore) {
                    const symbols_t s0 = read(i);
                    clear(i);
                    store(i, s0);
                }
            }
            // what last look-ups wrote behind the window: the next one's, or nothing's (a corrupt stream)
            {
                uint8_t* const behind = buf + ((end + 7u) & ~7u) + lane * 8u;
                const uint2 s = *reinterpret_cast<const uint2*>(behind);
                *reinterpret_cast<uint2*>(behind) = make_uint2(bg, bg);
                __builtin_amdgcn_wave_barrier();
                if (end == room && from + room < n) *reinterpret_cast<uint2*>(buf + lane * 8u) = s;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        // Every stream ends with an entry, in state 0, its words read and no more.
        if (lane < N) {
            if (next != (len ? skew + lane + len * N : n) || at - table_at >= 16u) err |= ANSZP_ST_BAD_STATE;
            if (((q - q0 - first_bit + 31u) >> 5) != hdr >> 16) err |= ANSZP_ST_BAD_LENGTH;
        }
        err = wave_or(err);
        if (err && lane == 0) report(p.status, err);
    }
}

// The chunks that do not fit a wavefront's part of `area`, with as many wavefronts at a time as have room for the longest.
template <int OUT, class INDEX_OF>
__device__ __forceinline__ void waves_decode_long(const DecodeParams& p, uint8_t* lds, uint32_t* ctl, const WavesLayer& w, uint32_t area, uint32_t longest, uint32_t fits,
                                                  uint32_t first, uint32_t run, INDEX_OF&& index_of) {
    const uint32_t need = 4u * (min(longest, kWavesLds / 4u) + kWavesPad) + kWavesLeastRoom + kWavesBehind + 32u;
    const uint32_t active = min(max(area / need, 1u), blockDim.x / kWave);
    __syncthreads();                                        // (the chunks that fit are done)
    if (threadIdx.x == 0) ctl[0] = 0u;
    __syncthreads();
    waves_decode<OUT, true>(p, lds, ctl, w, area / active & ~15u, active, fits, first, run, index_of);
}

template <int OUT>
__global__ __launch_bounds__(1024) void decode_waves(DecodeParams p, WavesShape shape) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kWavesLds];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6), threads = blockDim.x;
    const uint32_t table_bytes = 16u << p.table_log;
    // 0: chunks of the run taken; 1: the run's length; 2: words of its longest chunk of those that need a turn of their own, or 0;
    // 3: not a regular set
    uint32_t* const ctl = reinterpret_cast<uint32_t*>(lds + table_bytes);
    const uint32_t share = p.n_chunks / gridDim.x, waves = threads / kWave, last_chunk = p.n_chunks - 1u;
    // The workgroups' shares of a regular set: consecutive chunks, as alike in number as they can be, but that a share ends with a
    // layer where one ends nearby.  (Lanes 0..31 look around the share's first chunk, the others around its end; both neighbours find
    // the same.)
    const uint32_t reach = waves_reach(share, waves);
    const uint32_t border = blockIdx.x + lane / 32u;        // (n_chunks * border / gridDim.x, in 32 bits)
    const uint32_t nominal = border * share + border * (p.n_chunks - share * gridDim.x) / gridDim.x;
    const uint32_t look_at = nominal + lane % 32u - reach;  // (wraps around below 0: beyond every chunk)
    bool ends = false;
    if (lane % 32u <= 2u * reach && look_at - 1u < last_chunk) ends = p.chunks[look_at].layer_id != p.chunks[look_at - 1u].layer_id;
    // Is it one?  Four wavefronts look at 32 pairs of neighbours each, spread evenly over all descriptors.
    const uint32_t pair = 32u * wave + lane / 2u;
    const uint32_t sample = static_cast<uint32_t>(uint64_t(pair) * (last_chunk - 1u) / (32u * kWavesLookers - 1u)) + lane % 2u;
    uint32_t sample_layer = 0, sample_words = 0;
    if (wave < kWavesLookers) {
        sample_layer = p.chunks[sample].layer_id;
        sample_words = p.chunks[sample].payload_words;
    }
    const uint64_t found = __ballot(ends);
    auto share_begins = [&](uint32_t half) {
        const uint32_t b = __builtin_amdgcn_readlane(nominal, 32u * half), m = static_cast<uint32_t>(found >> (32u * half));
        if (b == 0u || b == p.n_chunks || m == 0u) return b;
        const uint32_t below = m & ((2u << reach) - 1u), above = m >> reach;         // at or below, at or above the middle
        const uint32_t down = below ? reach - (31u - static_cast<uint32_t>(__clz(below))) : 32u;
        const uint32_t up = above ? static_cast<uint32_t>(__ffs(above)) - 1u : 32u;
        return down <= up ? b - down : b + up;
    };
    const uint32_t first = share_begins(0u), last = share_begins(1u);
    const uint32_t own = shape.own, fits = waves_words(own), area = kWavesLds - table_bytes - kWavesCtl;
    // More than 8 of 32 pairs of two layers or five in a row (layers of one chunk), words that do not fit, three times the mean
    // chunk's cost: not a regular set.
    auto look = [&] {
        if (wave >= kWavesLookers) return;
        const uint32_t other = __builtin_amdgcn_update_dpp(0, sample_layer, 0xB1, 0xF, 0xF, false);       // the pair's other one's
        uint32_t sum;
        wave_exclusive_sum(min(sample_words, fits), &sum);
        const uint64_t ends_in = __ballot(sample_layer != other);
        if ((__popcll(ends_in) > 16 || (ends_in & ends_in >> 2 & ends_in >> 4 & ends_in >> 6 & ends_in >> 8) != 0ull || __ballot(sample_words > fits) != 0ull || sum > kWave * (3u * shape.mean + 2u * shape.fixed)) && lane == 0)
            ctl[3] = 1u;
    };
    if (__builtin_expect(first == last, 0)) {               // (no share: only to find out)
        if (tid == 0) ctl[3] = 0u;
        __syncthreads();
        look();
        __syncthreads();
    }
    for (uint32_t at_chunk = first; at_chunk < last;) {
        auto itself = [](uint32_t i) { return i; };
        const bool at_first = at_chunk == first;
        const WavesLayer w = waves_stage(p, lds, ctl, p.chunks[at_chunk].layer_id, at_chunk, last, fits, itself, [&] { if (at_first) look(); });
        const uint32_t run = ctl[1], longest = ctl[2];
        if (ctl[3]) break;
        waves_decode<OUT, false>(p, lds, ctl, w, own, waves, fits, at_chunk, run, itself);
        if (__builtin_expect(longest != 0u, 0)) waves_decode_long<OUT>(p, lds, ctl, w, area, longest, fits, at_chunk, run, itself);
        at_chunk += run;
    }
    if (__builtin_expect(ctl[3] == 0u, 1)) return;
    // So many descriptors at a time, all workgroups the same ones, and of a share of those as much as the list holds.
    uint16_t* const list = reinterpret_cast<uint16_t*>(lds + kWavesLds - kWavesListBytes);
    const uint32_t sorted_area = area - kWavesListBytes, sorted_own = sorted_area / waves & ~15u, sorted_fits = waves_words(sorted_own);
    const uint32_t at_once = min(32u * gridDim.x, kWavesSorted), blocks = (p.n_chunks + at_once - 1u) / at_once;
    for (uint32_t block = 0; block < blocks; ++block) {
        const uint32_t base = static_cast<uint32_t>(uint64_t(p.n_chunks) * block / blocks), end = static_cast<uint32_t>(uint64_t(p.n_chunks) * (block + 1u) / blocks);
        auto listed = [&](uint32_t i) { return base + list[i]; };
        bool more = true;
        for (uint32_t window = 0; more; ++window) {
            const uint32_t n = uniform(waves_share(p, shape, lds, list, base, end - base, window, more));
            for (uint32_t at_chunk = 0; at_chunk < n;) {
                const WavesLayer w = waves_stage(p, lds, ctl, p.chunks[uniform(listed(at_chunk))].layer_id, at_chunk, n, sorted_fits, listed, [] {});
                const uint32_t run = ctl[1], longest = ctl[2];
                waves_decode<OUT, false>(p, lds, ctl, w, sorted_own, waves, sorted_fits, at_chunk, run, listed);
                if (longest) waves_decode_long<OUT>(p, lds, ctl, w, sorted_area, longest, sorted_fits, at_chunk, run, listed);
                at_chunk += run;
            }
        }
    }
}

#endif
