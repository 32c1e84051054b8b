// Few chunks: a workgroup per chunk (internal to the library; included by the decode kernels'
// source, whose names it uses).
//
// The look-ahead kernel lets a chunk's walk, the placing of its symbols and the stores run beside each other, which takes
// hand-overs through LDS, blocks with a boundary between them and a start that deals out tasks.  A call of few short chunks is over
// before that pays: here all wavefronts stage the table and the words, one walks the streams from end to end
// (walk_entries) into a buffer that holds the whole chunk, and all convert and store it.  A longer chunk comes in windows, in two
// buffers in turn: while one wavefront walks a window the others store the one before and fill its buffer with the background.
// What bounds it: memory's latency three times in a row (arguments, descriptor, table and words: about 2 us with the launch),
// 45 ns a look-up, and the stores at the end.  One chunk of 4,096 symbols (2^10 states) 6.7 -> 4.6 us, 249 of 8,192 (2^12) 8.2 -> 6.2;
// choose_kernel (anszp_choose.h) has the line between this kernel and the look-ahead kernel, with both sides.
// Windows: lanes meet at a window's end, the fastest wait for the slowest (windows of 16,384 symbols: 15 % of a walk of 1.5 bits), so
// they are few and long, and the last one, whose stores nothing hides, is a quarter of the chunk where LDS allows.  Sets that hold chunks
// much longer than their mean, 2^12 states, bf16 and fp32, look-ahead kernel with a plan -> walk, stores and filling one after the other
// -> here: 230 of 2,000 symbols and 10 of 65,536 16.4, 16.6 -> 16.4, 18.4 -> 15.8, 16.5 us; 50 layers of 500 to 90,000 in chunks of 65,536 18.6 ->
// 19.7 -> 18.3; 440 and 40 (2^10 states, two on a CU) 17.7, 17.8 -> 18.2, 20.2 -> 16.2, 17.0; 200 of 1,000 and one of 262,144 53, 53 -> 65, 73 ->
// 56, 56, one of 1,048,576 101, 102 -> 149, 179 -> 108, 109: there the look-ups' 5 ns remain.
#ifndef ANSZP_FEW_H
#define ANSZP_FEW_H

#include "anszp_walk.h"

constexpr uint32_t kFewThreads = 512u;
constexpr uint32_t kFewTableLoads = (1u << ANSZP_MAX_TABLE_LOG) / kFewThreads;          // 16-byte loads per thread
constexpr uint32_t kFewWhole = 24576u;                     // symbols of a chunk that comes in one window (440 of 1,000 and 10 of 32,768, fp32: 18.3 us with 32,768)

template <int OUT, uint32_t LDS>
__global__ __launch_bounds__(kFewThreads) void decode_few(DecodeParams p) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6);
    const uint32_t number = unit_of_workgroup(blockIdx.x);
    if (number >= p.n_chunks) return;
    const anszp_chunk_t c = p.chunks[number];
    if (!chunk_in_bounds(p, c)) {
        if (tid == 0) report(p.status, ANSZP_ST_BAD_DESC);
        return;
    }
    const uint32_t L = 1u << p.table_log, N = p.n_streams, table_bytes = 16u << p.table_log, table_at = lds_address(lds);
    const uint32_t total = c.payload_words, quads = total / 4u;
    const uint32_t* const src = p.tables + c.layer_id * table_stride_words(p.table_log);
    const uint32_t* const payload = p.payload + c.payload_offset;
    // everything that depends on the descriptor alone is asked for at once
    const uint4* const entries = reinterpret_cast<const uint4*>(src + table_lookahead_offset(p.table_log));
    uint4 tv[kFewTableLoads];
#pragma unroll
    for (uint32_t u = 0; u < kFewTableLoads; ++u)
        if (u * kFewThreads < L) tv[u] = entries[min(tid + u * kFewThreads, L - 1u)];
    constexpr uint32_t kWordLoads = 2u;
    uint4 wv[kWordLoads];
    const uint4* const rows = quads ? reinterpret_cast<const uint4*>(payload) : entries;
#pragma unroll
    for (uint32_t u = 0; u < kWordLoads; ++u) wv[u] = rows[quads ? min(tid + u * kFewThreads, quads - 1u) : 0u];
    const uint32_t last_at = 4u * quads + tid;              // the last words, and zeros
    const uint32_t last = last_at < total ? payload[last_at] : 0u;
    const uint32_t hdr = wave == 0u && lane < N ? p.stream_hdr[c.stream_offset + lane] : 0u;
    const anszp_layer_t lay = p.layers[c.layer_id];
    const uint32_t bg = (src[table_triples_offset(p.table_log) + L - 1u] >> 24) * 0x01010101u;     // four times the dominant symbol
    if (!scales_in_bounds(p, lay, c)) {
        if (tid == 0) report(p.status, ANSZP_ST_BAD_DESC);
        return;
    }
    // LDS: table | a zero word, the chunk's words from a multiple of 16 bytes on, zeros | buffer, or two of them
    const uint32_t skew = static_cast<uint32_t>(c.out_offset) & 7u, n = c.n_symbols + skew;        // (see decode_waves)
    const uint32_t area = LDS - table_bytes, words_bytes = (4u * (min(total, LDS) + kWavesPad) + 15u) & ~15u;
    if (c.n_symbols > (1u << 24) || words_bytes + 2u * (kWavesBehind + kFewLeastRoom) > area) {    // the plain loop, like any chunk beyond its kernel's reach
        if (wave) return;
        const uint32_t err = decode_chunk_stepwise<OUT>(p, c, lay, WordTable{src + table_triples_offset(p.table_log)}, lane);
        if (err && lane == 0) report(p.status, err);
        return;
    }
    uint32_t* const words = reinterpret_cast<uint32_t*>(lds + table_bytes) + 3;
    uint8_t* const buf = lds + table_bytes + words_bytes;
    // one window where the chunk is short, else windows of a length that two of them fit
    const uint32_t left = area - words_bytes, one = (n + 15u) & ~15u;
    const bool whole = one <= kFewWhole && one + kWavesBehind <= left;
    const uint32_t room = whole ? one : min(3u * (n / 4u), left / 2u - kWavesBehind) & ~15u, buffer = room + kWavesBehind;
    const bool per_channel = lay.channel_len != 0u;
    auto reversed = [](const uint4& v) { return make_uint4(__brev(v.x), __brev(v.y), __brev(v.z), __brev(v.w)); };
#pragma unroll
    for (uint32_t u = 0; u < kFewTableLoads; ++u)
        if (tid + u * kFewThreads < L) reinterpret_cast<uint4*>(lds)[tid + u * kFewThreads] = walk_entry_pair(tv[u], table_at);
#pragma unroll
    for (uint32_t u = 0; u < kWordLoads; ++u)
        if (tid + u * kFewThreads < quads) reinterpret_cast<uint4*>(words + 1)[tid + u * kFewThreads] = reversed(wv[u]);
    for (uint32_t i = tid + kWordLoads * kFewThreads; i < quads; i += kFewThreads) reinterpret_cast<uint4*>(words + 1)[i] = reversed(rows[i]);
    if (last_at < total + kWavesPad - 4u) words[1u + last_at] = __brev(last);
    if (tid == 0) words[0] = 0u;
    for (uint32_t i = tid * 16u; i < (whole ? buffer : 2u * buffer); i += kFewThreads * 16u) *reinterpret_cast<uint4*>(buf + i) = make_uint4(bg, bg, bg, bg);
    uint32_t all_words;
    const uint32_t first_word = wave_exclusive_sum(hdr >> 16, &all_words), first_bit = 32u * min(first_word, total);
    uint32_t err = all_words != total ? ANSZP_ST_BAD_DESC : 0u;
    const uint32_t len = (lane < N && c.n_symbols > lane) ? (c.n_symbols - lane + N - 1u) / N : 0u;
    const uint64_t out_elem0 = c.out_offset - skew, layer_elem0 = out_elem0 - lay.out_base;
    const bool wide = per_channel && c.out_offset - lay.out_base + c.n_symbols >= (1ull << 32);    // (store8 numbers a layer's elements in 32 bits)
    __syncthreads();
    // The walking wavefront's lanes: entry, bit, and the next symbol's position (as in decode_waves).
    const uint32_t q0 = 8u * lds_address(words) + 31u, q_end = q0 + 32u * total + 1u;
    uint32_t q = q0 + first_bit, at = table_at + 8u * (2u * (hdr & (L - 1u)) + (words[1u + (first_bit >> 5)] >> 31));
    uint32_t next = len ? skew + lane : n;
    constexpr uint32_t kStore = OUT == ANSZP_OUT_F32 ? 4u : 8u;
    typedef typename std::conditional<OUT == ANSZP_OUT_F32, uint32_t, uint2>::type symbols_t;
    // the `end` symbols of the window that begins at `from`, by `threads` threads; REFILL: the buffer holds the background afterwards
    auto store = [&](uint8_t* at_buf, uint32_t from, uint32_t end, uint32_t thread, uint32_t threads, auto refill) {
        for (uint32_t i = thread * kStore; i < end; i += threads * kStore) {
            const symbols_t s = *reinterpret_cast<const symbols_t*>(at_buf + i);
            if constexpr (decltype(refill)::value) {
                if constexpr (OUT == ANSZP_OUT_F32) *reinterpret_cast<uint32_t*>(at_buf + i) = bg;
                else *reinterpret_cast<uint2*>(at_buf + i) = make_uint2(bg, bg);
            }
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
        }
    };
    auto walk = [&](const uint8_t* at_buf, uint32_t from, uint32_t end) {
        const uint32_t buf_at = lds_address(at_buf);
        uint32_t to = buf_at + next - from - N;            // an entry's last symbol is N positions before the stream's next
        __builtin_amdgcn_s_setprio(3);
        walk_entries<kWalkSpread, true>(at, q, to, q_end, buf_at + end - N, N);
        __builtin_amdgcn_s_setprio(0);
        next = to + N + from - buf_at;
    };
    if (__builtin_expect(whole, 1)) {
        if (wave == 0u && n) walk(buf, 0u, n);
        __syncthreads();
        store(buf, 0u, n, tid, kFewThreads, std::false_type{});
    } else {
        uint2 behind = make_uint2(bg, bg);                 // what last look-ups wrote behind the window before
        uint8_t* cur = buf;
#pragma unroll 1
        for (uint32_t from = 0; from < n; from += room) {
            uint8_t* const other = cur == buf ? buf + buffer : buf;
            const uint32_t end = min(n - from, room);
            if (wave == 0u) {
                if (from) *reinterpret_cast<uint2*>(cur + lane * 8u) = behind;
                walk(cur, from, end);
                behind = *reinterpret_cast<const uint2*>(cur + room + lane * 8u);          // (room: a multiple of 16)
                *reinterpret_cast<uint2*>(cur + room + lane * 8u) = make_uint2(bg, bg);
            } else if (from) {
                store(other, from - room, room, tid - kWave, kFewThreads - kWave, std::true_type{});
            }
            __syncthreads();
            if (from + room >= n) store(cur, from, end, tid, kFewThreads, std::false_type{});
            cur = other;
        }
    }
    if (wave) return;
    // Every stream ends with an entry, in state 0, its words read and no more.
    if (lane < N) {
        if (next != (len ? skew + lane + len * N : n) || at - table_at >= 16u) err |= ANSZP_ST_BAD_STATE;
        if (((q - q0 - first_bit + 31u) >> 5) != hdr >> 16) err |= ANSZP_ST_BAD_LENGTH;
    }
    err = wave_or(err);
    if (err && lane == 0) report(p.status, err);
}

#endif
