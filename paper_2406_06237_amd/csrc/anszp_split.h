// One stream decoded by a whole workgroup (internal to the library; included by the decode kernels' source, whose
// names it uses).
//
// A container with one stream per chunk has the least framing, but its decoder is one chain of dependent table
// look-ups (Sec. II-A), whatever the machine beside it.  What breaks the chain: a decoder started at any bit of the
// stream in any state falls into the true sequence by itself.  Two walks of the automaton that stand at the same bit in
// the same state are one from there on, and they meet, in every bit, with a probability of about 1 / L (measured on
// streams of 1.2 bits a symbol, 2^10 states: the distance is exponential with a mean of 1.3 L bits).  Of G walks
// started together in different states the true one meets some after about 2 L / G bits, so a few dozen starts
// hit within a fraction of that.  So:
//   1  The stream is cut into `cuts` segments of equal length in bits and a short last one.  At every cut, a group of
//      1024 / cuts threads starts in as many places and walks one segment.  Where the group stands at the next cut
//      (its first look-up at or behind it: state and bit) are the places, mostly two to ten different ones, at which
//      the true walk is expected there.  They are the nodes of a graph.
//   2  Every node is walked through its segment once more, which leads to a node of the next cut, or to a place that is
//      none: that becomes a node and is walked in the next round.  The true start is a node too, so following the links
//      from it gives the true sequence as far as they are known; rounds go on until it reaches the last segment.  A
//      round always extends it, so a stream on which nothing meets costs what a plain walk costs, and a result never
//      depends on a guess: a link stands for a walk from exactly that state and bit.
//   3  The symbols counted per segment of the true sequence give every segment its place in the output; its quarters
//      are walked again from states noted on the way, into a buffer in LDS, which leaves in 16-byte stores.
// The first walk is bound by the instructions of sixteen wavefronts, the others by one LDS round trip per look-up.
// Everything is held together by barriers: no wavefront waits for another's progress.
// Measured (one chunk, fp32 out, as one chain in the look-ahead kernel -> here, the mean of twelve): 36,864 symbols of 1.2 bits,
// 2^10 states 500 -> 50 us (42 to 60; 16 of them the first walk, about 10 a round, mostly two), 2^12 states 496 -> 80; 2.8 bits,
// 2^12 states 1424 -> 134; 12,000 symbols of 1.2 bits, 2^10 states 169 -> 36; 2,500 of them 41 -> 21.
// Where a state keeps its upper bits: half, quarter, quarter, 36,864 symbols, 2^9 states 1146 -> 154 (305 at worst; 426 and 1,872 with all
// starts in spread states).  Where it keeps them for a while, 2^12 states and short streams, the kernel may lose: 64 chunks of 12,000
// symbols, 2 alike 319 -> 445, 16 alike 472 -> 543, 200 of half, quarter, quarter 322 -> 495, the worst there is (walks that wait for their
// windows took another 10 %); 64 alike 472 -> 249, 2^9 states 16 alike 472 -> 98.
#ifndef ANSZP_SPLIT_H
#define ANSZP_SPLIT_H

#include "anszp_walk.h"

constexpr uint32_t kSplitThreads = 1024u;
constexpr uint32_t kSplitMaxCuts = 64u;
constexpr uint32_t kSplitParts = 4u;                      // parts of a segment that are written side by side
constexpr uint32_t kSplitMaxNodes = 1600u;                // no more, and as many as LDS has room for
constexpr uint32_t kSplitUnknown = 0xFFFFFFFFu, kSplitNone = 0xFFFFFFFEu;
constexpr uint32_t kSplitPad = 10u;                       // words beside the stream's: one before it, zeros behind (a walk that must stop
                                                          // at the stream's end may make four look-ups more and read three words there)

// A place in a stream: the next look-ahead entry (13 bits) and the bit it stands at, plus 31 (19 bits).
static_assert(kSplitWords * 32u + 31u + 32u < (1u << 19) && ANSZP_MAX_TABLE_LOG + 1 <= 13, "a place is one word");

struct SplitLds {
    uint32_t path[kSplitMaxCuts + 1u], start[kSplitMaxCuts + 2u];
    uint32_t n_nodes, path_cut, forced, err, kept;
    __attribute__((aligned(16))) uint32_t group[kSplitThreads];         // a cut's places, then the different ones among them
    uint32_t group_size[kSplitMaxCuts], group_first[kSplitMaxCuts];
};
// A node (eleven words, an array of them behind SplitLds): its place and cut, then what its walk found: the symbols, where it
// ended, the node that is (or kSplitUnknown, kSplitNone), and place and symbols at the ends of its parts but the last.
enum { kNodePlace, kNodeCut, kNodeCount, kNodeEnd, kNodeLink, kNodePartPlace, kNodePartCount = kNodePartPlace + kSplitParts - 1, kNodeWords = kNodePartCount + kSplitParts - 1 };

template <int OUT>
__global__ __launch_bounds__(kSplitThreads) void decode_split(DecodeParams p) {
    constexpr uint32_t kLdsBytes = 160u * 1024u - 64u;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLdsBytes];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const anszp_chunk_t c = p.chunks[blockIdx.x];
    if (!chunk_in_bounds(p, c)) {
        if (tid == 0) report(p.status, ANSZP_ST_BAD_DESC);
        return;
    }
    const anszp_layer_t lay = p.layers[c.layer_id];
    const uint32_t* const src = p.tables + c.layer_id * table_stride_words(p.table_log);
    if (!scales_in_bounds(p, lay, c)) {
        if (tid == 0) report(p.status, ANSZP_ST_BAD_DESC);
        return;
    }
    if (c.payload_words > kSplitWords || c.n_symbols > (1u << 24)) {       // the plain loop, like any chunk beyond its kernel's window
        if (tid >= kWave) return;
        const uint32_t err = decode_chunk_stepwise<OUT>(p, c, lay, WordTable{src + table_triples_offset(p.table_log)}, lane);
        if (err && lane == 0) report(p.status, err);
        return;
    }

    // ---- stage.  LDS: table | a zero word, the stream's words first bit on top, zeros | SplitLds | buffer of symbols
    const uint32_t L = 1u << p.table_log, len = c.n_symbols, n_words = c.payload_words, total = 32u * n_words;
    const uint32_t words_off = 16u << p.table_log, nodes_off = (words_off + 4u * (n_words + kSplitPad) + 15u) & ~15u;
    const uint32_t table_at = lds_address(lds);
    const uint32_t q0 = 8u * (table_at + words_off) + 31u;              // a stream's bit b is at q = q0 + b
    SplitLds& S = *reinterpret_cast<SplitLds*>(lds + nodes_off);
    uint32_t* const node = reinterpret_cast<uint32_t*>(lds + nodes_off + ((sizeof(SplitLds) + 15u) & ~15u));
    // Nodes in all and those any walk may add; the others belong to the true sequence alone, one per cut, so that it can
    // always go on.
    const uint32_t n_all = min(kSplitMaxNodes, (kLdsBytes - lds_address(node) + lds_address(lds)) / (4u * kNodeWords)), n_shared = n_all - kSplitMaxCuts;
    auto at_node = [&](uint32_t field, uint32_t id) -> uint32_t& { return node[id * kNodeWords + field]; };
    const uint32_t hdr = p.stream_hdr[c.stream_offset];
    const uint32_t dominant = src[table_triples_offset(p.table_log) + L - 1u] >> 24;
    {
        const uint4* const entries = reinterpret_cast<const uint4*>(src + table_lookahead_offset(p.table_log));
        for (uint32_t i = tid; i < L; i += kSplitThreads) {
            reinterpret_cast<uint4*>(lds)[i] = walk_entry_pair(entries[i], table_at);
        }
        const uint32_t* const words = p.payload + c.payload_offset;
        uint32_t* const to = reinterpret_cast<uint32_t*>(lds + words_off);
        for (uint32_t i = tid; i < n_words + kSplitPad; i += kSplitThreads) to[i] = i - 1u < n_words ? __brev(words[i - 1u]) : 0u;
    }
    // How many segments: as many as the rounds they cost are worth.  Walks simulated on streams of 1,500 to 36,864 symbols,
    // 0.5 to 2.8 bits each, 2^8 to 2^12 states, and a round taken for 2.5 us and 50 ns a look-up: these bounds miss the best
    // of 8, 16, 32 and 64 by 4 % on average.
    const uint32_t cuts = total < 512u ? 0u : total >= max(8u * L, 12288u) ? 64u : total >= max(4u * L, 3072u) ? 32u : 16u;
    const uint32_t per_group = cuts ? kSplitThreads / cuts : 1u;
    // (bits; the last segment has a part's length, and its cut lies before the last word's padding: a walk that gets there
    // has made no look-up behind the stream's end)
    const uint32_t seg = cuts ? kSplitParts * (total - 32u) / (kSplitParts * cuts + 1u) : 0u;
    __syncthreads();

    auto place_of = [&](uint32_t at, uint32_t q) { return (at - table_at) >> 3 | (q - q0) << 13; };
    auto at_of = [&](uint32_t place) { return table_at + ((place & 0x1FFFu) << 3); };
    auto q_of = [&](uint32_t place) { return q0 + (place >> 13); };
    auto next_bit = [&](uint32_t b) { return (reinterpret_cast<const uint32_t*>(lds + words_off)[1u + (b >> 5)] >> (~b & 31u)) & 1u; };
    const uint32_t first_place = 2u * (hdr & (L - 1u)) + next_bit(0u);

    // ---- 1: the places at the cuts
    if (tid == 0) {
        at_node(kNodePlace, 0) = first_place; at_node(kNodeCut, 0) = 0u; at_node(kNodeLink, 0) = kSplitUnknown;
        S.n_nodes = 1u;
        S.kept = 0u;
    }
    __syncthreads();
    if (cuts) {
        const uint32_t g = tid / per_group, r = tid % per_group;
        uint32_t place = kSplitUnknown;
        const bool walks = g != 0u || r == 0u;
        auto walk = [&](uint32_t state, uint32_t b) {     // from that state at that bit to the next cut; returns the state there
            uint32_t at = at_of(g == 0u ? first_place : 2u * state + next_bit(b)), q = q0 + b, count = 0;
            walk_entries<kWalkCount>(at, q, count, q0 + (g + 1u) * seg, len);
            place = place_of(at, q);
            return (at - table_at) >> 4;
        };
        bool kept = false;
        if (walks) {
            const uint32_t state = g == 0u ? hdr & (L - 1u) : ((2u * r + 1u) * L / (2u * per_group)) & (L - 1u);
            const uint32_t end = walk(state, g * seg);
            kept = max(end, state) - min(end, state) <= L / 8u;
        }
        // With frequencies that are powers of two, or nearly, a state keeps its upper bits (a quarter of the states come as close by
        // chance) and walks started in other states never meet the true one: eight of them are started again, in the stream's own
        // initial state, at eight bits in a row (a symbol may take as many).
        const uint64_t n_kept = __ballot(kept);
        if (lane == 0) atomicAdd(&S.kept, static_cast<uint32_t>(__popcll(n_kept)));
        __syncthreads();
        if (S.kept > kSplitThreads / 2u && g != 0u && r < 8u) walk(hdr & (L - 1u), g * seg + r);
        // the different ones among the group's (a group is a part of a wavefront, which reads before it writes)
        S.group[tid] = place;
        bool again = place == kSplitUnknown;
        const uint4* const others = reinterpret_cast<const uint4*>(&S.group[g * per_group]);
        for (uint32_t j = 0; j < per_group; j += 4u) {
            const uint4 o = others[j / 4u];
            again |= (o.x == place && j < r) || (o.y == place && j + 1u < r) || (o.z == place && j + 2u < r) || (o.w == place && j + 3u < r);
        }
        const uint64_t group_lanes = (per_group == 64u ? ~0ull : ((1ull << per_group) - 1ull)) << (lane - r);
        const uint64_t mine = __ballot(!again) & group_lanes;
        const uint32_t rank = static_cast<uint32_t>(__popcll(mine & ((1ull << lane) - 1ull)));
        uint32_t size = static_cast<uint32_t>(__popcll(mine)), first = 0;
        if (r == 0u) {
            first = atomicAdd(&S.n_nodes, size);
            size = first >= n_shared ? 0u : min(size, n_shared - first);
            S.group_size[g] = size;
            S.group_first[g] = first;
        }
        first = __shfl(first, lane - r, kWave);
        size = __shfl(size, lane - r, kWave);
        if (!again && rank < size) {
            S.group[g * per_group + rank] = place;
            at_node(kNodePlace, first + rank) = place;
            at_node(kNodeCut, first + rank) = g + 1u;
            at_node(kNodeLink, first + rank) = kSplitUnknown;
        }
    }
    if (tid == 0) { S.path[0] = 0u; S.path_cut = 0u; S.forced = kSplitUnknown; S.err = 0u; }
    __syncthreads();

    // ---- 2: rounds
    uint32_t done = 0;                                    // nodes below this one have been walked
    for (uint32_t round = 0; cuts != 0u && round <= kSplitMaxCuts; ++round) {
        const uint32_t n_nodes = min(S.n_nodes, n_shared), forced = S.forced;
        __syncthreads();                                  // (new nodes are added from here on)
        const uint32_t items = n_nodes - done + (forced != kSplitUnknown ? 1u : 0u);
        for (uint32_t i = tid; i < items; i += kSplitThreads) {
            const uint32_t id = done + i < n_nodes ? done + i : forced;
            const uint32_t cut = at_node(kNodeCut, id);
            if (cut >= cuts) continue;                    // at the last cut: walked when it is written
            uint32_t at = at_of(at_node(kNodePlace, id)), q = q_of(at_node(kNodePlace, id)), count = 0;
#pragma unroll 1
            for (uint32_t m = 0; m < kSplitParts; ++m) {
                walk_entries<kWalkCount, true>(at, q, count, q0 + cut * seg + (m + 1u) * seg / kSplitParts, len);
                if (m + 1u < kSplitParts) {
                    at_node(kNodePartPlace + m, id) = place_of(at, q);
                    at_node(kNodePartCount + m, id) = count;
                }
            }
            const uint32_t place = place_of(at, q);
            at_node(kNodeEnd, id) = place;
            at_node(kNodeCount, id) = count;
            uint32_t link = kSplitNone;
            const uint32_t size = S.group_size[cut];
            // (four at a time and without a way out, so that the reads do not wait for each other; behind `size` lies what was there)
            const uint4* const known = reinterpret_cast<const uint4*>(&S.group[cut * per_group]);
            uint32_t found = size;
#pragma unroll 4
            for (uint32_t j = 0; j < size; j += 4u) {
                const uint4 o = known[j / 4u];
                found = min(found, o.x == place ? j : o.y == place ? j + 1u : o.z == place ? j + 2u : o.w == place ? j + 3u : size);
            }
            if (found < size) link = S.group_first[cut] + found;
            if (link == kSplitNone) {
                const uint32_t fresh = atomicAdd(&S.n_nodes, 1u);
                if (fresh < n_shared) {
                    at_node(kNodePlace, fresh) = place; at_node(kNodeCut, fresh) = cut + 1u; at_node(kNodeLink, fresh) = kSplitUnknown;
                    link = fresh;
                }
            }
            at_node(kNodeLink, id) = link;
        }
        done = n_nodes;
        __syncthreads();
        if (tid == 0) {                                   // follow the true sequence as far as it is known
            uint32_t cut = S.path_cut, id = S.path[cut], next = kSplitUnknown;
            while (cut < cuts) {
                next = at_node(kNodeLink, id);
                if (next >= kSplitNone) break;
                id = next;
                S.path[++cut] = id;
            }
            uint32_t force = kSplitUnknown;
            if (cut < cuts && next == kSplitNone) {       // walked, and no room for its end: the true sequence's own place
                force = n_shared + cut;
                at_node(kNodePlace, force) = at_node(kNodeEnd, id); at_node(kNodeCut, force) = cut + 1u; at_node(kNodeLink, force) = kSplitUnknown;
                at_node(kNodeLink, id) = force;
                S.path[++cut] = force;
            }
            S.path_cut = cut;
            S.forced = force;
        }
        __syncthreads();
        if (S.path_cut >= cuts) break;
    }

    // ---- 3: symbols before each segment of the true sequence
    if (tid < kWave) {
        uint32_t all;
        const uint32_t before = wave_exclusive_sum(lane < cuts ? at_node(kNodeCount, S.path[lane]) : 0u, &all);
        if (lane < cuts) S.start[lane] = before;
        if (lane == 0) S.start[cuts] = all;
    }
    __syncthreads();
    const uint32_t parts = cuts * kSplitParts + 1u;
    uint32_t at = 0, q = 0, count = 0, until = 0;
    auto part_begins = [&](uint32_t i) {
        const uint32_t s = i / kSplitParts, m = i % kSplitParts;
        return S.start[s] + (m ? at_node(kNodePartCount + m - 1u, S.path[s]) : 0u);
    };
    uint32_t err = 0;
    if (tid < parts) {
        const uint32_t s = tid / kSplitParts, m = tid % kSplitParts, id = S.path[s];
        const uint32_t place = m ? at_node(kNodePartPlace + m - 1u, id) : at_node(kNodePlace, id);
        at = at_of(place);
        q = q_of(place);
        count = part_begins(tid);
        until = tid + 1u < parts ? min(part_begins(tid + 1u), len) : len;
        if (count > len) err |= ANSZP_ST_BAD_STATE;       // (a corrupt stream: more symbols than the chunk has)
    }
    // Positions count from the multiple of 8 elements of the output at or below the chunk's first element.
    const uint32_t skew = static_cast<uint32_t>(c.out_offset) & 7u, n = len + skew;
    const uint64_t out_elem0 = c.out_offset - skew, layer_elem0 = out_elem0 - lay.out_base;
    // (what the nodes held is in registers now: the buffer takes their place)
    uint8_t* const buf = reinterpret_cast<uint8_t*>(S.group);
    const uint32_t room = min((kLdsBytes - kLookaheadMaxSymbols - (lds_address(buf) - table_at)) & ~15u, (n + 15u) & ~15u);
    const bool per_channel = lay.channel_len != 0u;
    const bool wide = per_channel && c.out_offset - lay.out_base + len >= (1ull << 32);      // (store8 numbers a layer's elements in 32 bits)
    __syncthreads();
    for (uint32_t first = 0; first < n; first += room) {
        const uint32_t bg = dominant * 0x01010101u;
        // (the last look-up of a part may end behind the buffer: its symbol is the next one's)
        const uint2 late = first ? *reinterpret_cast<const uint2*>(buf + room) : make_uint2(bg, bg);
        __syncthreads();
        for (uint32_t i = tid; i <= room / 16u; i += kSplitThreads) {
            if (i < room / 16u) reinterpret_cast<uint4*>(buf)[i] = i ? make_uint4(bg, bg, bg, bg) : make_uint4(late.x, late.y, bg, bg);
            else *reinterpret_cast<uint2*>(buf + room) = make_uint2(bg, bg);
        }
        __syncthreads();
        const uint32_t end = min(n - first, room);
        if (count < until && count + skew < first + end) {
            const uint32_t to = lds_address(buf) + skew - first - 1u;      // the symbol that ends a look-up is number count - 1 after it
            uint32_t address = to + count;
            walk_entries<kWalkWrite, true>(at, q, address, q0 + total + 1u, to + min(until, first + end - skew));
            count = address - to;
        }
        __syncthreads();
        for (uint32_t run = tid * 8u; run < end; run += kSplitThreads * 8u) {
            const uint32_t pos = first + run;
            const uint2 s = *reinterpret_cast<const uint2*>(buf + run);
            if (pos >= skew && run + 8u <= end && !wide) {
                if (per_channel) Flusher<OUT, true>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
                else Flusher<OUT, false>::store8(p, lay, out_elem0 + pos, layer_elem0 + pos, s);
            } else {
#pragma unroll 1
                for (uint32_t j = pos < skew ? skew - pos : 0u; j < 8u && run + j < end; ++j) {
                    const uint32_t sym = ((j < 4u ? s.x : s.y) >> (8u * (j & 3u))) & 0xFFu;
                    if (per_channel) Flusher<OUT, true>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                    else Flusher<OUT, false>::store1(p, lay, out_elem0 + pos + j, layer_elem0 + pos + j, sym);
                }
            }
        }
        __syncthreads();
    }
    // The end of the stream: the entry that holds the last symbol ends with it and arrives in state 0, the stream's words
    // read and no more.
    if (tid + 1u == parts) {
        if (count != len || at - table_at >= 16u) err |= ANSZP_ST_BAD_STATE;
        if (((q - q0 + 31u) >> 5) != hdr >> 16) err |= ANSZP_ST_BAD_LENGTH;
        if (hdr >> 16 != n_words) err |= ANSZP_ST_BAD_DESC;
    }
    if (err) atomicOr(&S.err, err);
    __syncthreads();
    if (tid == 0 && S.err) report(p.status, S.err);
}

#endif
