// Many short chunks: a wavefront per chunk, the table shared by a workgroup (internal to the library; included by the
// decode kernels' source, whose names it uses).
//
// The look-ahead kernel stages a table for every one or two chunks and spreads a chunk's work over several wavefronts, so
// that one chunk is done as soon as possible.  With several rounds of such workgroups per CU neither pays: what counts is
// what a CU gets done, and staging (up to 64 KiB of entries per workgroup, 4 us) is most of it where chunks are short.
// Here a workgroup fills a CU and takes a run of consecutive chunks; it stages a layer's entries once, and every
// wavefront takes the next chunk by itself: its stream words to LDS (first bit on top), look-ups (walk_entries), symbols to a
// buffer in LDS that holds the dominant symbol as background (a look-up writes the last of its symbols), and from there,
// converted, 16 bytes per lane to memory.  A chunk longer than the buffer is decoded in windows of the buffer's length:
// lanes stop at its end, and what a last look-up wrote behind it (up to 8 symbols of each stream) begins the next.
// No wavefront waits for another but at a change of layer.
// Measured with a plan, bf16 out, 64 streams (look-ahead kernel -> here): chunks of 2,048 symbols, 2^12 states 1,100 of them
// 20 -> 9 us, 2,300 32 -> 13, 10,000 222 -> 19; 4,096 symbols of 2 bits, 2^10 states 2,300 26 -> 13, 10,000 151 -> 30 (3.1 TB/s of
// the bytes there are); 16,384 symbols, 2^12 states 1,100 29 -> 21, 4,000 131 -> 45.  With shares cut regardless of
// layers 48 layers of 11 to 23 chunks took 1.4 to 1.8 times as long (1,100 chunks of 16,384: 38, 21.6 as it is).
#ifndef ANSZP_WAVES_H
#define ANSZP_WAVES_H

#include "anszp_walk.h"

constexpr uint32_t kWavesLds = 160u * 1024u - 64u;
constexpr uint32_t kWavesCtl = 64u;                        // behind the table: what the wavefronts of a run share
constexpr uint32_t kWavesPad = 12u;                        // words beside a chunk's: one before, zeros behind (see kSplitPad)
constexpr uint32_t kWavesBehind = kLookaheadMaxSymbols * ANSZP_MAX_STREAMS + 16u;      // bytes behind the buffer
constexpr uint32_t kWavesRoom = 2048u, kWavesLeastRoom = 512u;    // symbols in the buffer beside a mean chunk's words; beside any chunk's

// Wavefronts per workgroup and the LDS each has for a chunk's words and the buffer (waves == 0: not a launch for this
// kernel).  As many wavefronts as leave room for a quarter more words than the mean chunk has beside kWavesRoom
// symbols; chunks of up to a good deal more still fit, with a shorter buffer.
struct WavesShape { uint32_t waves, own; };
inline WavesShape waves_shape(uint32_t table_log, uint64_t mean_words) {
    for (uint32_t waves : {16u, 12u, 8u}) {
        if (table_log == ANSZP_MAX_TABLE_LOG && waves == 16u) continue;
        const uint32_t own = (kWavesLds - (16u << table_log) - kWavesCtl) / waves & ~15u;
        if (4u * (mean_words * 5u / 4u + 16u + kWavesPad) + kWavesRoom + kWavesBehind <= own) return WavesShape{waves, own};
    }
    return WavesShape{0u, 0u};
}

template <int OUT>
__global__ __launch_bounds__(1024) void decode_waves(DecodeParams p, uint32_t own) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kWavesLds];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid >> 6), threads = blockDim.x;
    const uint32_t L = 1u << p.table_log, N = p.n_streams, table_bytes = 16u << p.table_log, table_at = lds_address(lds);
    uint32_t* const ctl = reinterpret_cast<uint32_t*>(lds + table_bytes);          // 0: chunks of the run taken; 1: the run's length
    uint32_t* const words = reinterpret_cast<uint32_t*>(lds + table_bytes + kWavesCtl + wave * own);
    const uint32_t most = (own - kWavesLeastRoom - kWavesBehind - 16u) / 4u - kWavesPad;      // words of a chunk
    const uint32_t q0 = 8u * lds_address(words) + 31u;      // bit b of the chunk is at q = q0 + b
    // The workgroups' shares: consecutive chunks, as alike in number as they can be, but that a share ends with a layer where
    // one ends nearby: a layer more in a share is a table more to stage and, with fewer chunks than wavefronts, a chunk's time
    // more.  (Lanes 0..31 look around the share's first chunk, the others around its end; both neighbours find the same.)
    const uint32_t share = p.n_chunks / gridDim.x, waves = threads / kWave;
    const uint32_t reach = min(15u, share < waves ? min(share / 2u + 1u, (waves - share + 1u) / 2u) : share / 8u);
    const uint32_t nominal = static_cast<uint32_t>(uint64_t(blockIdx.x + lane / 32u) * p.n_chunks / gridDim.x);
    const uint32_t look_at = nominal + lane % 32u - reach;  // (wraps around below 0: beyond every chunk)
    bool ends = false;
    if (lane % 32u <= 2u * reach && look_at - 1u < p.n_chunks - 1u) ends = p.chunks[look_at].layer_id != p.chunks[look_at - 1u].layer_id;
    const uint64_t found = __ballot(ends);
    auto share_begins = [&](uint32_t half) {
        const uint32_t b = static_cast<uint32_t>(uint64_t(blockIdx.x + half) * p.n_chunks / gridDim.x), m = static_cast<uint32_t>(found >> (32u * half));
        if (b == 0u || b == p.n_chunks || m == 0u) return b;
        const uint32_t below = m & ((2u << reach) - 1u), above = m >> reach;         // at or below, at or above the middle
        const uint32_t down = below ? reach - (31u - static_cast<uint32_t>(__clz(below))) : 32u;
        const uint32_t up = above ? static_cast<uint32_t>(__ffs(above)) - 1u : 32u;
        return down <= up ? b - down : b + up;
    };
    const uint32_t first = uniform(share_begins(0u)), last = uniform(share_begins(1u));
    for (uint32_t at_chunk = first; at_chunk < last;) {
        // the run: the chunks from at_chunk on that belong to its layer
        const uint32_t layer_id = uniform(p.chunks[at_chunk].layer_id);
        const uint32_t look = min(last - at_chunk, threads);
        __syncthreads();                                    // (the run before this one is done)
        if (tid == 0) { ctl[0] = 0u; ctl[1] = look; }
        __syncthreads();
        const bool known = layer_id < p.n_tables;
        const uint32_t* const src = p.tables + size_t(known ? layer_id : 0u) * table_stride_words(p.table_log);
        const uint4* const entries = reinterpret_cast<const uint4*>(src + table_lookahead_offset(p.table_log));
        for (uint32_t i = tid; i < L; i += threads) reinterpret_cast<uint4*>(lds)[i] = walk_entry_pair(entries[i], table_at);
        if (tid < look && p.chunks[at_chunk + tid].layer_id != layer_id) atomicMin(&ctl[1], tid);
        const anszp_layer_t lay = p.layers[known ? layer_id : 0u];
        const uint32_t dominant = src[table_triples_offset(p.table_log) + L - 1u] >> 24;
        const bool per_channel = lay.channel_len != 0u;
        const uint32_t bg = dominant * 0x01010101u;         // the buffer's background
        __syncthreads();
        const uint32_t run = ctl[1];
        for (;;) {
            // (What lane 0 alone does at the end of a turn must not be joined with this: the compiler, seeing the same
            // condition, led the other lanes around both, found their number to be 0 and had them take chunk 0 for ever.)
            uint32_t who = lane, mine = 0;
            asm volatile("" : "+v"(who), "+v"(mine));
            if (who == 0u) mine = atomicAdd(&ctl[0], 1u);
            mine = uniform(mine);
            if (mine >= run) break;
            const anszp_chunk_t c = p.chunks[at_chunk + mine];
            if (!chunk_in_bounds(p, c) || !scales_in_bounds(p, lay, c)) {
                if (lane == 0) report(p.status, ANSZP_ST_BAD_DESC);
                continue;
            }
            if (c.n_symbols > (1u << 24)) {                 // the plain loop, like any chunk beyond its kernel's reach
                const uint32_t err = decode_chunk_stepwise<OUT>(p, c, lay, WordTable{src + table_triples_offset(p.table_log)}, lane);
                if (err && lane == 0) report(p.status, err);
                continue;
            }
            const uint32_t hdr = lane < N ? p.stream_hdr[c.stream_offset + lane] : 0u;
            const uint32_t total = c.payload_words;
            const uint32_t* const payload = p.payload + c.payload_offset;
            const uint32_t skew = static_cast<uint32_t>(c.out_offset) & 7u, n = c.n_symbols + skew;
            const bool staged = total <= most;
            const uint32_t words_bytes = (4u * ((staged ? total : 0u) + kWavesPad) + 15u) & ~15u;
            uint8_t* const buf = reinterpret_cast<uint8_t*>(words) + words_bytes;
            const uint32_t buf_at = lds_address(buf), room = min((own - words_bytes - kWavesBehind) & ~15u, (n + 15u) & ~15u);
            if (staged) {
                for (uint32_t i = lane; i < total + kWavesPad; i += kWave) words[i] = i - 1u < total ? __brev(payload[i - 1u]) : 0u;
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
            auto word = [&](uint32_t i) { return staged ? words[1u + min(i, total)] : i < total ? __brev(payload[i]) : 0u; };
            uint32_t q = q0 + first_bit, at = table_at + 8u * (2u * (hdr & (L - 1u)) + (word(first_bit >> 5) >> 31));
            uint32_t next = len ? skew + lane : n;
            for (uint32_t from = 0; from < n; from += room) {
                const uint32_t end = min(n - from, room);
                // an entry's last symbol is N positions before the stream's next
                uint32_t to = buf_at + next - from - N;
                const uint32_t to_end = buf_at + end - N;
                if (staged) {
                    walk_entries<kWalkSpread>(at, q, to, q_end, to_end, N);
                } else {
                    while (to < to_end && q < q_end) {
                        const uint32_t b = q - q0;
                        const uint64_t e = *reinterpret_cast<lds_uint64_t*>(static_cast<uintptr_t>(at));
                        const uint32_t lo = static_cast<uint32_t>(e);
                        const uint32_t window = static_cast<uint32_t>(((uint64_t(word(b >> 5)) << 32 | word((b >> 5) + 1u)) << (b & 31u)) >> 32);
                        at = ((window >> (lo & 31u)) << 3) + static_cast<uint32_t>(e >> 32);
                        q += (lo >> 8) & 15u;
                        to += (lo >> 24) * N;
                        *reinterpret_cast<__attribute__((address_space(3))) uint8_t*>(static_cast<uintptr_t>(to)) = static_cast<uint8_t>(lo >> 16);
                    }
                }
                next = to + N + from - buf_at;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (uint32_t i = lane * 8u; i < end; i += kWave * 8u) {
                    const uint32_t pos = from + i;
                    const uint2 s = *reinterpret_cast<const uint2*>(buf + i);
                    *reinterpret_cast<uint2*>(buf + i) = make_uint2(bg, bg);
                    if (__builtin_expect(pos >= skew && i + 8u <= end && !wide, 1)) {
                        if (per_channel) Flusher<OUT, true>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                        else Flusher<OUT, false>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                    } else {
#pragma unroll 1
                        for (uint32_t j = pos < skew ? skew - pos : 0u; j < 8u && i + j < end; ++j) {
                            const uint32_t sym = ((j < 4u ? s.x : s.y) >> (8u * (j & 3u))) & 0xFFu;
                            if (per_channel) Flusher<OUT, true>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                            else Flusher<OUT, false>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                        }
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
        at_chunk += run;
    }
}

#endif
