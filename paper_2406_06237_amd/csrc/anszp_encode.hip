// tANS encoder on the GPU: compresses layers whose symbols are in device memory into the container
// anszp_decode reads, word for word what the host packer (anszp_pack_layer) writes.
//
// Encoding (Sec. II-A) walks a stream's symbols backwards: to encode symbol s in state x (in
// [L, 2L)) the low bits of x are dropped, and written out, until x lies in [f_s, 2 f_s); the new
// state is the (x - f_s)-th state of s, counted in increasing order, plus L.  The decoder reads the
// bits of the first symbol first, so a stream's bits are laid down from its end: the walk is done
// once to learn the stream's length and once to write.
//
// As many chunks as the chip holds workgroups at once are walked once (encode_once, further down).  More of them take three
// launches, like those nothing allocated and no scratch memory: sizes (every stream's final state and
// word count into the stream headers, every chunk's descriptor but for its payload offset), a scan
// over the chunks (payload offsets, total), the writing pass.  What the writing pass needs to know of
// the sizes pass beyond that (how many bits of a stream's last word are used) travels in fields that
// the writing pass puts right: four of the five bits in bits 12..15 of the stream's header (a state has
// at most 12 bits), the fifth bit of all the chunk's streams as one word in the descriptor's out_offset.
//
// One lane per stream, one wavefront per chunk at a time.  A workgroup of eight wavefronts takes consecutive
// chunks (as few as leave every CU two workgroups); all of it builds the encoding tables of a layer in LDS
// (anszp_spread.h), then its wavefronts walk the layer's chunks.
//
// What bounds it: a walk is a chain, per symbol one LDS read and three instructions between the state and the next
// one; a wavefront has its SIMD nearly for itself.  Whether a symbol drops k or k - 1 bits is one addition
// (x + (k << 16) - (f_s << k): the upper half is the count), symbols are asked for two batches of sixteen
// ahead, a symbol's constants half a batch ahead.  Measured on 369 chunks of 65,536 symbols (2^12 states, 64
// streams): sizes 70 us, writing 98 us (54 and 83 ns a symbol, 9 us for the tables); with a search for the bit count
// bit by bit, symbols waited for batch by batch, a second walk in the writing pass for the stream's bits and the
// tables by divisions the two took 1.55 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "anszp.h"
#include "anszp_cus.h"
#include "anszp_spread.h"

namespace {

constexpr uint32_t kWave = 64;
constexpr uint32_t kThreads = 512;          // two workgroups fit a CU at once (128 registers a lane)
constexpr uint32_t kWaves = kThreads / kWave;
constexpr uint32_t kBatch = 16;             // symbols a lane asks for at a time

struct EncParams {
    const uint8_t* symbols;
    const uint32_t* freqs;                  // one row of 256 per layer
    const anszp_pack_job_t* jobs;           // null: one layer, `one`
    anszp_pack_job_t one;
    anszp_chunk_t* chunks;
    uint32_t* stream_hdr;
    uint32_t* payload;
    unsigned long long* used;
    uint32_t* status;
    const uint32_t* prepared;               // null, or a record of encoding tables per layer (encode_prepare)
    uint32_t* finish;                       // with `prepared`: workgroups that are done, then a bit per chunk that was not written
    uint64_t n_chunks, out_offset, payload_word_offset, payload_cap_words;
    uint32_t n_layers, table_log, n_streams, layer_id, stream_offset, chunks_per_group, spin_limit;
    uint32_t longest_chunk;                 // with `prepared`: symbols
};

// A layer's encoding tables.  info[s]: what x + info.x has in its upper half is the number of bits symbol s drops
// in state x; 2 * (x >> that) + info.y is the byte of `next` that holds the new state plus L.  A symbol without a
// frequency has info.x = 0 (no other symbol has), drops nothing and leads to some state.
struct EncTables {
    __attribute__((aligned(16))) uint2 info[ANSZP_ALPHABET];
    __attribute__((aligned(16))) uint16_t next[kSpreadStates];
};
struct EncLds : EncTables {
    SpreadLds spread;
};

__device__ __forceinline__ void report(uint32_t* status, uint32_t bits) {
    atomicOr(&status[0], bits);
    atomicAdd(&status[1], 1u);
}

// f: the symbol's frequency, first: the occurrences of smaller symbols.
__device__ __forceinline__ uint2 symbol_info(uint32_t f, uint32_t first, uint32_t table_log) {
    // x in [L, 2L) drops k or k - 1 bits, k = table_log - floor(log2 f): k when x >= f << k
    const uint32_t k = f ? table_log - (31u - static_cast<uint32_t>(__clz(f))) : 0u;
    return f ? make_uint2((k << 16) - (f << k), 2u * (first - f)) : make_uint2(0u, 0u - (2u << table_log));
}

// The workgroup's encoding tables.  False (for every thread) when the frequencies do not sum to L.
__device__ __forceinline__ bool build_tables(const uint32_t* freqs, uint32_t table_log, EncTables& t, SpreadLds& spread) {
    const uint32_t tid = threadIdx.x, L = 1u << table_log;
    const bool ok = spread_states<kThreads>(freqs, table_log, spread, [&](uint32_t g, uint32_t, uint32_t, uint32_t, uint32_t state) {
        t.next[g] = static_cast<uint16_t>(L + state);
    });
    if (!ok) return false;
    if (tid < ANSZP_ALPHABET) t.info[tid] = symbol_info(spread.f[tid], spread.first[tid], table_log);
    __syncthreads();
    return true;
}

// A layer's record of encode_prepare: four words, the first of them whether the frequencies sum to L, then `info` and the
// first L states of `next`.
constexpr uint32_t kRecordInfo = 4u, kRecordNext = kRecordInfo + 2u * ANSZP_ALPHABET;
__host__ __device__ constexpr uint32_t record_words(uint32_t table_log) { return kRecordNext + (table_log > 3u ? (1u << table_log) / 2u : 4u); }

// The workgroup's encoding tables, built or taken from the layer's record.
__device__ __forceinline__ bool layer_tables(const EncParams& p, uint32_t layer, EncTables& t, SpreadLds& spread) {
    if (!p.prepared) return build_tables(p.freqs + size_t(layer) * ANSZP_ALPHABET, p.table_log, t, spread);
    typedef spread_words4 words4;
    const words4* const record = reinterpret_cast<const words4*>(p.prepared + size_t(layer) * record_words(p.table_log));
    const uint32_t units = record_words(p.table_log) / 4u;
    constexpr uint32_t kMost = (record_words(ANSZP_MAX_TABLE_LOG) / 4u + kThreads - 1u) / kThreads, kInfo = kRecordNext / 4u;
    words4 v[kMost];
    const uint32_t ok = __builtin_amdgcn_readfirstlane(record[0].x);
#pragma unroll
    for (uint32_t u = 0; u < kMost; ++u) v[u] = record[min(threadIdx.x + u * kThreads, units - 1u)];
#pragma unroll
    for (uint32_t u = 0; u < kMost; ++u) {
        const uint32_t i = threadIdx.x + u * kThreads;
        if (i >= units || i == 0u) continue;
        if (i < kInfo) reinterpret_cast<words4*>(t.info)[i - 1u] = v[u];
        else reinterpret_cast<words4*>(t.next)[i - kInfo] = v[u];
    }
    __syncthreads();
    return ok != 0u;
}

// A chunk's streams as its wavefront walks them: symbol number r of this lane's stream is chunk[r * n_streams + lane_off].
typedef const __attribute__((address_space(1))) uint8_t global_uint8_t;   // (a flat load would be waited for with the LDS reads)
struct ChunkStreams {
    global_uint8_t* chunk;                                      // uniform
    uint32_t cn, max_len;                                       // symbols of the chunk, of its longest stream (uniform)
    uint32_t lane_off;                                          // 0 for a lane without symbols: it walks along, never counted
    bool has_any, has_last;                                     // any symbol; one in row max_len - 1 (every lane has all rows before it)
};

// One stream, backwards (Sec. II-A).  WRITE: lay the bits down in `words` (the stream's n_words words, `pad` zero bits
// behind its last one); otherwise only count them.  Returns the number of bits; x: the final state plus L.
// The bits a symbol adds precede, in the stream, everything written so far; the stream is therefore built
// in reverse, padded at its start so that whole reversed words are whole words of the stream, and each
// finished word is bit-reversed into its place, from the stream's last word down to its first.
template <bool WRITE>
__device__ __forceinline__ uint32_t walk_stream(const EncTables& t, const ChunkStreams& s, uint32_t N, uint32_t L, uint32_t* words, uint32_t n_words,
                                uint32_t pad, uint32_t& x_out, bool& bad_symbol) {
    uint32_t x = L, bits = 0, lowest = 0xFFFFFFFFu;           // lowest: the smallest info.x met
    uint64_t acc = 0;
    uint32_t pair = 0, pair_bits = 0;                         // the bits of the last two symbols, on their way into acc
    uint32_t cnt = pad, at = n_words;                         // bits in acc; words still to be written
    const uint8_t* next = reinterpret_cast<const uint8_t*>(t.next);
    constexpr uint32_t kHalf = kBatch / 2u;
    auto load = [&](uint32_t hi, uint32_t (&sym)[kBatch]) {   // rows hi - 1, hi - 2, ... (hi >= kBatch)
        global_uint8_t* const row = s.chunk + uint64_t(hi - kBatch) * N;
#pragma unroll
        for (uint32_t j = 0; j < kBatch; ++j) sym[j] = (row + (kBatch - 1u - j) * N)[s.lane_off];
    };
    auto look_up = [&](const uint32_t (&sym)[kBatch], uint32_t from, uint2 (&info)[kHalf]) {
#pragma unroll
        for (uint32_t j = 0; j < kHalf; ++j) info[j] = t.info[sym[from + j]];
    };
    auto step = [&](const uint2 i) {
        const uint32_t sum = x + i.x, nb = sum >> 16;
        lowest = min(lowest, i.x);
        if constexpr (WRITE) {
            pair |= __builtin_amdgcn_ubfe(x, 0u, nb) << pair_bits;
            pair_bits += nb;
        } else {
            bits += nb;
        }
        uint32_t kept;                                        // x >> nb, the count taken from the sum's upper half as it is
        asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD" : "=v"(kept) : "v"(sum), "v"(x));
        x = *reinterpret_cast<const uint16_t*>(next + (2u * kept + i.y));
    };
    auto flush = [&]() {                                      // at least every two symbols: 24 bits, and 31 + 24 of them, fit
        if constexpr (WRITE) {
            acc |= uint64_t(pair) << cnt;
            cnt += pair_bits;
            pair = pair_bits = 0u;
            if (cnt >= 32u) {
                if (at) words[--at] = __brev(static_cast<uint32_t>(acc));
                acc >>= 32;
                cnt -= 32u;
            }
        }
    };
    auto walk = [&](const uint2 (&info)[kHalf]) {
#pragma unroll
        for (uint32_t j = 0; j < kHalf; ++j) {
            step(info[j]);
            if (j & 1u) flush();
        }
    };
    // the first batch makes the number of symbols left a multiple of a batch; only its first symbol may be missing
    // in a lane
    const uint32_t top = (s.max_len - 1u) % kBatch + 1u;
    uint32_t hi = s.max_len - top;                            // rows still to be asked for: a multiple of kBatch from here on
    uint32_t sym_a[kBatch], sym_b[kBatch] = {};
    uint2 info_0[kHalf], info_1[kHalf];
    sym_a[0] = s.chunk[(s.has_last ? (s.max_len - 1u) * N : 0u) + s.lane_off];
#pragma unroll
    for (uint32_t j = 1; j < kBatch; ++j) sym_a[j] = (s.chunk + (j < top ? uint64_t(s.max_len - 1u - j) * N : 0u))[s.lane_off];
    uint32_t left = hi;                                       // rows still to be walked behind the first batch
    if (hi) { load(hi, sym_b); hi -= kBatch; }
    look_up(sym_a, 0u, info_0);
    look_up(sym_a, kHalf, info_1);
    if (hi) { load(hi, sym_a); hi -= kBatch; }
    if (s.has_last) step(info_0[0]);
#pragma unroll
    for (uint32_t j = 1; j < kBatch; ++j) {
        if (j < top) step(j < kHalf ? info_0[j % kHalf] : info_1[j % kHalf]);         // (uniform)
        if (j & 1u) flush();
    }
    // a batch: the first half's constants are in info_0; `sym` holds the batch, `then` the one after it
    auto batch = [&](uint32_t (&sym)[kBatch], uint32_t (&then)[kBatch]) {
        look_up(sym, kHalf, info_1);
        if (hi) { load(hi, sym); hi -= kBatch; }
        walk(info_0);
        look_up(then, 0u, info_0);                            // (behind the last batch: symbols walked before, not used)
        walk(info_1);
        left -= kBatch;
    };
    look_up(sym_b, 0u, info_0);
    while (left) {
        batch(sym_b, sym_a);
        if (!left) break;
        batch(sym_a, sym_b);
    }
    if (lowest == 0u) bad_symbol = true;
    x_out = x;
    return bits;
}

// (Called by whole wavefronts, c alike for all lanes.)  The layer chunk c belongs to (jobs are in chunk order: the last one whose first_chunk is not beyond c) and the
// chunk's number within it.  False when c belongs to no layer.
__device__ bool layer_of_chunk(const EncParams& p, uint64_t c, uint32_t& layer, anszp_pack_job_t& job, uint64_t& local) {
    layer = 0;
    if (!p.jobs) {
        job = p.one;
    } else {
        // (64 jobs at a look, one per lane: a look is a round trip to memory)
        uint32_t lo = 0, hi = p.n_layers;
        do {
            const uint32_t stride = (hi - lo + kWave - 1u) / kWave, i = lo + (threadIdx.x & (kWave - 1u)) * stride;
            const uint32_t below = static_cast<uint32_t>(__popcll(__ballot(i < hi && p.jobs[min(i, hi - 1u)].first_chunk <= c)));
            if (below == 0u) return false;
            lo += (below - 1u) * stride;
            hi = min(hi, lo + stride);
        } while (hi - lo > 1u);
        layer = lo;
        job = p.jobs[lo];
    }
    local = c - job.first_chunk;
    return job.chunk_size != 0 && local < (job.n_symbols + job.chunk_size - 1) / job.chunk_size;
}

// What both passes do with a workgroup's chunks: run after run of chunks of one layer, the layer's tables, then
// chunk(job, layer, local, c, tables_ok) by one wavefront per chunk; none(c) by all threads for a chunk of no layer.
template <class CHUNK, class NONE>
__device__ __forceinline__ void for_each_chunk(const EncParams& p, EncLds& t, CHUNK&& chunk, NONE&& none) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t c = uint64_t(blockIdx.x) * p.chunks_per_group;
    const uint64_t end = min(c + p.chunks_per_group, (unsigned long long)p.n_chunks);
    while (c < end) {                                           // (alike for every thread)
        uint32_t layer;
        anszp_pack_job_t job;
        uint64_t local;
        if (!layer_of_chunk(p, c, layer, job, local)) {
            none(c);
            ++c;
            continue;
        }
        uint64_t run = (job.n_symbols + job.chunk_size - 1) / job.chunk_size - local;   // chunks of this layer from c on
        if (p.jobs && layer + 1u < p.n_layers && p.jobs[layer + 1u].first_chunk > c) run = min(run, (unsigned long long)(p.jobs[layer + 1u].first_chunk - c));
        run = min(run, (unsigned long long)(end - c));
        const bool ok = layer_tables(p, layer, t, t.spread);
        for (uint64_t i = wave; i < run; i += kWaves) chunk(job, layer, local + i, c + i, ok);
        c += run;
        // (behind the last run a wavefront is done as soon as its own chunks are: the registers of the idle ones let the
        // next workgroup onto the CU)
        if (c < end) __syncthreads();                           // the tables have been read
    }
}

__device__ __forceinline__ ChunkStreams streams_of(const EncParams& p, const anszp_pack_job_t& job, uint64_t local, uint32_t lane) {
    ChunkStreams s;
    const uint32_t N = p.n_streams;
    const uint64_t begin = local * job.chunk_size, rest = job.n_symbols - begin;
    s.cn = __builtin_amdgcn_readfirstlane(rest < job.chunk_size ? static_cast<uint32_t>(rest) : job.chunk_size);
    s.max_len = (s.cn - 1u) / N + 1u;
    s.has_any = lane < N && lane < s.cn;
    s.has_last = s.has_any && (s.cn - lane - 1u) / N + 1u == s.max_len;
    s.lane_off = s.has_any ? lane : 0u;
    const uintptr_t at = reinterpret_cast<uintptr_t>(p.symbols) + job.first_symbol + begin;
    s.chunk = reinterpret_cast<global_uint8_t*>(uintptr_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(at)))) |
                                               uintptr_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(at >> 32)))) << 32);
    return s;
}

__global__ __launch_bounds__(kThreads, 4) void encode_sizes(EncParams p) {
    __shared__ EncLds t;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t N = p.n_streams, L = 1u << p.table_log;
    for_each_chunk(p, t, [&](const anszp_pack_job_t& job, uint32_t layer, uint64_t local, uint64_t c, bool ok) {
        if (!ok && lane == 0 && local == 0) report(p.status, ANSZP_ST_BAD_FREQ);
        if (!ok && !p.jobs) return;                             // (one layer: nothing is written)
        const ChunkStreams s = streams_of(p, job, local, lane);
        uint32_t x = L, nw = 0, bits = 0;
        bool bad = false;
        if (ok) {
            bits = walk_stream<false>(t, s, N, L, nullptr, 0u, 0u, x, bad);
            if (!s.has_any) { bits = 0; x = L; bad = false; }   // no stream, or one without symbols
            nw = (bits + 31u) >> 5;
        }
        const bool too_long = nw > 0xFFFFu;
        nw = min(nw, 0xFFFFu);
        // (bits 12..15 and out_offset: how many bits there are beyond whole words, for the writing pass)
        const uint64_t fifth = __ballot((bits & 16u) != 0u);
        if (lane < N) p.stream_hdr[c * N + lane] = (x - L) | (bits & 15u) << 12 | nw << 16;
        const uint32_t chunk_words = __builtin_amdgcn_readlane(spread_wave_sum(nw), kWave - 1);
        if (__ballot(bad) && lane == 0) report(p.status, ANSZP_ST_BAD_SYMBOL);
        if (__ballot(too_long) && lane == 0) report(p.status, ANSZP_ST_NO_SPACE);
        if (lane == 0) {
            anszp_chunk_t d;
            d.layer_id = p.jobs ? layer : p.layer_id;
            d.n_symbols = ok ? s.cn : 0u;
            d.out_offset = ok ? fifth : job.first_symbol + local * job.chunk_size;
            d.payload_offset = 0;                               // by the scan
            d.payload_words = chunk_words;
            d.stream_offset = p.stream_offset + static_cast<uint32_t>(c) * N;
            p.chunks[c] = d;
        }
    }, [&](uint64_t c) {                                        // the jobs do not cover the chunks the caller counted
        if (threadIdx.x == 0) {
            report(p.status, ANSZP_ST_BAD_DESC);
            anszp_chunk_t d = {};
            p.chunks[c] = d;
        }
        if (threadIdx.x < N) p.stream_hdr[c * N + threadIdx.x] = 0u;
    });
}

// A layer without symbols: what is left to do is to look at its frequencies (one wavefront).
__global__ __launch_bounds__(kWave) void encode_nothing(EncParams p) {
    const uint32_t L = 1u << p.table_log;
    uint32_t sum = 0;
    for (uint32_t s = threadIdx.x; s < ANSZP_ALPHABET; s += kWave) sum += min(p.freqs[s], L + 1u);   // (as in spread_states)
    sum = spread_wave_sum(sum);
    if (threadIdx.x == kWave - 1u && sum != L) report(p.status, ANSZP_ST_BAD_FREQ);
}

// Payload offsets: every chunk starts on a multiple of four words.  One workgroup, chunks in order, as many at a time
// as it has threads.
__global__ __launch_bounds__(kThreads) void encode_scan(EncParams p) {
    __shared__ unsigned long long part[2][kWaves];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    unsigned long long carry = 0;
    for (uint64_t base = 0, turn = 0; base < p.n_chunks; base += kThreads, ++turn) {
        const uint64_t c = base + tid;
        unsigned long long mine = c < p.n_chunks ? ((unsigned long long)(p.chunks[c].payload_words) + 3ull) & ~3ull : 0ull;
        unsigned long long upto = mine;
#pragma unroll
        for (int d = 1; d < int(kWave); d <<= 1) {
            const unsigned long long v = __shfl_up(upto, d, kWave);
            if (lane >= uint32_t(d)) upto += v;
        }
        if (lane == kWave - 1) part[turn & 1][wave] = upto;     // (two rows: one barrier per turn)
        __syncthreads();
        unsigned long long before = carry;
        for (uint32_t w = 0; w < kWaves; ++w) {
            const unsigned long long v = part[turn & 1][w];
            if (w < wave) before += v;
            carry += v;
        }
        if (c < p.n_chunks) p.chunks[c].payload_offset = p.payload_word_offset + before + upto - mine;
    }
    if (tid == 0) {
        *p.used = carry;
        if (carry > p.payload_cap_words) report(p.status, ANSZP_ST_NO_SPACE);
    }
}

// A chunk's words, by one wavefront, from a walk of its own.  fifth: see encode_sizes.
__device__ __forceinline__ void write_chunk(const EncParams& p, const EncTables& t, const anszp_pack_job_t& job, uint64_t local, uint64_t c, uint32_t payload_words,
                                            uint64_t payload_offset, uint64_t fifth) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t N = p.n_streams, L = 1u << p.table_log;
    const ChunkStreams s = streams_of(p, job, local, lane);
    const uint32_t hdr = lane < N ? p.stream_hdr[c * N + lane] : 0u;
    const uint32_t nw = hdr >> 16;
    const uint32_t beyond = ((hdr >> 12) & 15u) | ((fifth >> lane) & 1u ? 16u : 0u);   // bits of the last word, 0: all
    if (lane < N) p.stream_hdr[c * N + lane] = hdr & 0xFFFF0FFFu;
    if (lane == 0) p.chunks[c].out_offset = p.out_offset + job.first_symbol + local * job.chunk_size;
    const uint64_t at = payload_offset - p.payload_word_offset;          // in the caller's payload region
    const uint64_t padded = (uint64_t(payload_words) + 3ull) & ~3ull;
    if (at > p.payload_cap_words || padded > p.payload_cap_words - at) return;     // no room: reported with the total
    uint32_t* words = p.payload + at + (spread_wave_sum(nw) - nw);
    uint32_t x = L, room = nw;
    bool bad = false;
    if (__ballot(nw == 0xFFFFu) != 0ull) {                  // a stream too long for its header is not written
        const uint32_t bits = walk_stream<false>(t, s, N, L, nullptr, 0u, 0u, x, bad);
        if (((bits + 31u) >> 5) != nw) room = 0u;
    }
    if (!s.has_any) room = 0u;
    walk_stream<true>(t, s, N, L, words, room, (32u - beyond) & 31u, x, bad);
    if (lane < padded - payload_words) p.payload[at + payload_words + lane] = 0u;   // up to three pad words
}

__global__ __launch_bounds__(kThreads, 4) void encode_write(EncParams p) {
    __shared__ EncLds t;
    for_each_chunk(p, t, [&](const anszp_pack_job_t& job, uint32_t, uint64_t local, uint64_t c, bool ok) {
        if (!ok) return;                                        // reported by the first pass
        const anszp_chunk_t d = p.chunks[c];
        write_chunk(p, t, job, local, c, d.payload_words, d.payload_offset, d.out_offset);
    }, [&](uint64_t) {});                                       // reported by the first pass
}

// ---- All chunks at once (no more than the chip holds workgroups): one walk of every stream.
//
// A workgroup takes one chunk.  Its wavefronts share the walk, sixteen rows of symbols at a time with a barrier between:
//   load   (four) fetch the symbols, two steps ahead, and leave their constants in LDS in the order they are needed,
//   walk   (one) goes from state to state and notes each with the symbol's constant added,
//   pack   (one) works out from that which bits were dropped and lays them down, in the order of the walk.
// What stands between two states is then all the walking wavefront does (one LDS read, three instructions: 40 ns a
// symbol; 83 with the bits laid down in between, after 54 for a walk that only counts them).  A stream's bits stay in LDS
// until it is known how many there are and where the chunk's words begin: every workgroup publishes its chunk's words
// in the chunk's descriptor and adds up those of the chunks before it (the field reads kUnknown until then).  A workgroup only
// ever waits for lower-numbered ones, which have usually been started before it.  That is not certain: each of the chip's dies
// starts its own share in order, and another stream's kernels may hold places on some of them.  So a wait ends after a bounded
// number of looks (about 25 ms), and the chunks of workgroups that gave up, like chunks with a stream longer than its place in
// LDS, are written by the launch behind this one, with a walk of their own.  (Three streams that pack beside each other, or a
// matrix product beside one, never got there: 55 us a pack of 369 chunks of 65,536 symbols, 81 on one stream.)
// Measured on 369 chunks of 65,536 symbols (2^12 states, 64 streams): 66 us, 7.5 of them the tables, 40 ns a symbol, and 1.4
// and 4 us for the launches before and behind; with a pass for the sizes, a scan and a pass that writes 71, 5 and 97 (11 of
// both for the tables then).  One layer of 2.4 M symbols in 144 chunks 24 (23, 5, 29).  (A chunk whose streams do not fit is walked twice and costs what it
// did: 200 chunks of 65,536 symbols at 4.9 bits 236, 240.)
constexpr uint32_t kRows = 16u;                             // rows of symbols between two barriers
constexpr uint32_t kRowsPerLoader = 4u;
constexpr uint32_t kBitsStride = kWave + 1u;                // words from a stream's word to its next (read by streams and by words)
constexpr uint32_t kUnknown = 0xFFFFFFFFu;                  // in a descriptor's payload_words: not published yet
constexpr uint64_t kNotWritten = 1ull << 63;                // in its out_offset: to be written by the launch behind this one
typedef __attribute__((address_space(3))) uint32_t lds_word_t;
__device__ __forceinline__ uint32_t lds_offset(const void* shared) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)shared));
}
struct OnceLds {
    EncTables tables;
    union {
        SpreadLds spread;
        struct {
            uint2 ring[2][kRows][kWave];                    // the symbols' constants: being loaded, being read by the walk
            uint32_t sums[2][kRows][kWave];                 // state plus constant: being walked, packed
        };
    };
    uint32_t first[kWave], n_words[kWave], pad[kWave], x[kWave];
    uint32_t before, gave_up, bad, over;
    uint64_t fifth;                                         // (with bits 12..15 of a header: the bits beyond whole words, for a chunk written later)
    uint32_t bits[kBitsStride];                             // (as many rows as fit: see kBitRows)
};
constexpr uint32_t kOnceLds = 80u * 1024u;                  // two workgroups per CU
constexpr uint32_t kBitRows = (kOnceLds - uint32_t(offsetof(OnceLds, bits))) / (4u * kBitsStride) - 1u;

// True for every thread when the frequencies of the one layer sum to L.
__device__ __forceinline__ bool one_layer_ok(const EncParams& p) {
    __shared__ uint32_t part[ANSZP_ALPHABET / kWave];
    const uint32_t tid = threadIdx.x, L = 1u << p.table_log;
    if (tid < ANSZP_ALPHABET) {
        const uint32_t sum = spread_wave_sum(min(p.freqs[tid], L + 1u));       // (as in spread_states)
        if (tid % kWave == kWave - 1u) part[tid / kWave] = sum;
    }
    __syncthreads();
    return part[0] + part[1] + part[2] + part[3] == L;
}

// Before it: nothing is published.  (One layer of bad frequencies: nothing is written at all.)
__global__ __launch_bounds__(kThreads) void encode_begin(EncParams p) {
    if (!p.jobs && !one_layer_ok(p)) return;
    for (uint64_t c = threadIdx.x; c < p.n_chunks; c += kThreads) p.chunks[c].payload_words = kUnknown;
}

// ---- Before a packer whose caller brings scratch memory (anszp_pack_set_device): one launch for what does not depend on the symbols.
//
// The first workgroups work out the layers' encoding tables, once for all chunks: 512 occurrences each, a thread's occurrence
// against every symbol there is.  Occurrence i of symbol s has, of symbol t's, those before it whose (2j + 1) / 2g, g = t's
// frequency, is smaller than (2i + 1) / 2f (or equal, t < s): the odd numbers up to ((2i + 1) g - (t >= s)) / f.  That is a
// dozen instructions per symbol without a barrier or a look-up, 16 symbols 1 us, where every workgroup of the packer needed
// 7.5 us for a counting sort of its own.  Beyond kDirectSymbols symbols the sort is the faster one; one workgroup then does it.
// The others clear what the packer's callers find cleared (a fill per buffer took a launch each) and mark all chunks as
// unpublished; they are at work beside the former.  4.0 us for one table of 2^11 states and 3 MB of results, 8 for 53 of 2^12
// and 35 MB; packing a set with build_tables_device before it, results allocated by the caller of the binding: 369 chunks of
// 65,536 symbols 98 -> 79 us, 144 of 16,384 43 -> 35, two layers of 11,792 symbols 64 -> 31; 300 layers of 300 symbols, 2^12 states, 256
// symbols in each 123 -> 80 (215 with all of the workgroups that sort on one die), 16 symbols 124 -> 37.
constexpr uint32_t kDirectSymbols = 128u;
constexpr uint32_t kClearUnits = 8u * kThreads;             // of 16 bytes, per workgroup
constexpr uint32_t kJobsPerLaunch = 64u;
constexpr uint32_t kFinishWords = 1u + kWave;               // EncParams::finish: a bit per chunk (chunks_per_group)
struct JobsArg { anszp_pack_job_t job[kJobsPerLaunch]; };
struct PrepareParams {
    anszp_pack_job_t* jobs;                                 // null: one layer, of `n_jobs` 0
    uint32_t* records;
    uint32_t n_jobs, first_job;                             // in this launch
    uint32_t shares, table_groups, clear;                   // workgroups per table, of all tables; whether the results are cleared
    uint64_t chunk_units, hdr_words, payload_words;         // sizes of what is cleared
};
struct PrepareLds {
    SpreadLds spread;
    __attribute__((aligned(16))) uint32_t list[ANSZP_ALPHABET];     // the symbols there are: frequency, first occurrence << 16
};

// `words` words from `to`, a multiple of 16 bytes, on; this workgroup's share: units of 16 bytes [first, end).
__device__ __forceinline__ void fill_words(uint32_t* to, uint64_t words, uint32_t value, uint64_t first, uint64_t end) {
    const spread_words4 v = {value, value, value, value};
    const uint64_t whole = words / 4u;
    for (uint64_t i = first + threadIdx.x; i < min(end, whole); i += kThreads) reinterpret_cast<spread_words4*>(to)[i] = v;
    if (first <= whole && whole < end && threadIdx.x < words % 4u) to[4u * whole + threadIdx.x] = value;
}

__device__ __forceinline__ void store_jobs(const PrepareParams& q, const JobsArg& jobs) {
    if (threadIdx.x < q.n_jobs) q.jobs[q.first_job + threadIdx.x] = jobs.job[threadIdx.x];
}

__global__ __launch_bounds__(kJobsPerLaunch) void encode_jobs(PrepareParams q, JobsArg jobs) { store_jobs(q, jobs); }

__global__ __launch_bounds__(kThreads, 4) void encode_prepare(EncParams p, PrepareParams q, JobsArg jobs) {
    __shared__ PrepareLds t;
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1u), wave = __builtin_amdgcn_readfirstlane(tid >> 6), L = 1u << p.table_log;
    if (blockIdx.x >= q.table_groups) {
        const uint64_t share = blockIdx.x - q.table_groups;
        if (share == 0u) {
            store_jobs(q, jobs);
            if (tid < kFinishWords) p.finish[tid] = 0u;
            if (q.clear && tid < 2u) p.status[tid] = 0u;
        }
        uint64_t first = share * kClearUnits, end = first + kClearUnits;        // among the units of all buffers, one behind the other
        if (q.clear) {
            const uint64_t payload_units = (q.payload_words + 3u) / 4u, hdr_units = (q.hdr_words + 3u) / 4u;
            fill_words(p.payload, q.payload_words, 0xFFFFFFFFu, first, end);
            if (end <= payload_units) return;
            first = first > payload_units ? first - payload_units : 0u;
            end -= payload_units;
            fill_words(p.stream_hdr, q.hdr_words, 0u, first, end);
            if (end <= hdr_units) return;
            first = first > hdr_units ? first - hdr_units : 0u;
            end -= hdr_units;
        }
        // (one layer of bad frequencies: nothing is written at all)
        const bool mark = p.jobs || one_layer_ok(p);
        end = min(end, (unsigned long long)q.chunk_units);
        for (uint64_t i = first + tid; i < end; i += kThreads) {
            uint32_t* const at = reinterpret_cast<uint32_t*>(p.chunks) + 4u * i;
            const uint32_t words = mark && (i & 1u) && i / 2u < p.n_chunks ? kUnknown : 0u;
            if (q.clear) *reinterpret_cast<spread_words4*>(at) = spread_words4{0u, 0u, words, 0u};
            else if (words) at[2] = words;
        }
        return;
    }
    static_assert(sizeof(anszp_chunk_t) == 32 && offsetof(anszp_chunk_t, payload_words) == 24, "two units a descriptor");
    // (share by share: a layer's first share may be the one that sorts, and consecutive workgroups go to the eight dies in turn)
    const uint32_t share = blockIdx.x / p.n_layers, layer = blockIdx.x - share * p.n_layers;
    const uint32_t* const freqs = p.freqs + size_t(layer) * ANSZP_ALPHABET;
    uint32_t* const record = q.records + size_t(layer) * record_words(p.table_log);
    uint16_t* const next = reinterpret_cast<uint16_t*>(record + kRecordNext);
    uint32_t fs = 0, upto = 0, place = 0;
    if (tid < ANSZP_ALPHABET) {
        fs = freqs[tid];
        const uint64_t there = __ballot(fs != 0u);
        upto = spread_wave_sum(min(fs, L + 1u));                // (as in spread_states)
        place = static_cast<uint32_t>(__popcll(there & ((1ull << lane) - 1ull)));
        if (lane == kWave - 1u) {
            t.spread.part[wave] = upto;
            t.spread.part[8u + wave] = static_cast<uint32_t>(__popcll(there));
        }
    }
    __syncthreads();
    uint32_t total = 0, symbols = 0;
#pragma unroll
    for (uint32_t w = 0; w < ANSZP_ALPHABET / kWave; ++w) {
        if (w == wave) {
            upto += total;
            place += symbols;
        }
        total += t.spread.part[w];
        symbols += t.spread.part[8u + w];
    }
    const bool ok = total == L;
    if (share == 0u) {
        if (tid == 0u) record[0] = ok ? 1u : 0u;
        if (ok && tid < ANSZP_ALPHABET) reinterpret_cast<uint2*>(record + kRecordInfo)[tid] = symbol_info(fs, upto - fs, p.table_log);
    }
    if (!ok) return;
    if (symbols > kDirectSymbols) {
        if (share) return;
        __syncthreads();                                        // (`part` has been read)
        spread_states<kThreads>(freqs, p.table_log, t.spread, [&](uint32_t g, uint32_t, uint32_t, uint32_t, uint32_t state) {
            next[g] = static_cast<uint16_t>(L + state);
        });
        return;
    }
    if (fs) t.list[place] = fs | (upto - fs) << 16;             // (fs <= 2^12, upto - fs < 2^12)
    if (tid >= symbols && tid < ((symbols + 3u) & ~3u)) t.list[tid] = 0u;       // up to a multiple of four: counted, and nothing
    __syncthreads();
    const uint32_t g = share * kThreads + tid;
    if (g >= L) return;
    uint32_t mine = 0;                                          // the last symbol whose first occurrence is not beyond g
    for (uint32_t step = 0x80000000u >> __builtin_clz(symbols); step; step >>= 1) {
        const uint32_t c = mine + step;
        if (c < symbols && (t.list[c] >> 16) <= g) mine = c;
    }
    const uint32_t f = t.list[mine] & 0xFFFFu, odd = 2u * (g - (t.list[mine] >> 16)) + 1u;
    // n / f for n < 2^25, n / f < 2^13 (odd < 2f): the quotient with the reciprocal, whose and whose product's errors of less than
    // 2^-22 are made to lie on one side, is right or one too small
    const float inverse = __builtin_amdgcn_rcpf(static_cast<float>(f)) * (1.0f - 0x1p-20f);
    uint32_t state = L;
    auto count = [&](uint32_t j, uint32_t entry) {
        const uint32_t n = __umul24(odd, entry & 0xFFFFu) - (j >= mine ? 1u : 0u);
        uint32_t q0 = static_cast<uint32_t>(static_cast<float>(n) * inverse);
        q0 += n - __umul24(q0, f) >= f ? 1u : 0u;
        state += (q0 + 1u) >> 1;
    };
    for (uint32_t j = 0; j < symbols; j += 4u) {
        const spread_words4 e = *reinterpret_cast<const spread_words4*>(&t.list[j]);
        count(j, e.x);
        if (e.y) count(j + 1u, e.y);                            // (uniform; behind the last symbol nothing)
        if (e.z) count(j + 2u, e.z);
        if (e.w) count(j + 3u, e.w);
    }
    next[g] = static_cast<uint16_t>(state);
}

// Words of the chunks before c (each a multiple of four), once all are published.  False for every thread when one of
// them was not by the `looks`-th look.
__device__ __forceinline__ bool words_before(const EncParams& p, uint64_t c, uint32_t looks, uint32_t& before, uint32_t& gave_up, uint64_t& out) {
    const uint32_t tid = threadIdx.x;
    if (tid == 0) { before = 0u; gave_up = 0u; }
    __syncthreads();
    uint32_t sum = 0;
    for (uint64_t i = tid; i < c; i += kThreads) {
        uint32_t v, n = 0;
        while ((v = __hip_atomic_load(&p.chunks[i].payload_words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == kUnknown) {
            if (n++ >= looks) { gave_up = 1u; v = 0u; break; }
            __builtin_amdgcn_s_sleep(8);
        }
        sum += (v + 3u) & ~3u;
    }
    if (sum) atomicAdd(&before, sum);
    __syncthreads();
    out = before;                                           // (at most 2^9 chunks of less than 2^22 words each)
    return gave_up == 0u;
}

// Chunk c.  FINISH: its descriptor and words are complete where this returns true; false: its words before are not known.
template <bool FINISH>
__device__ __forceinline__ bool encode_chunk(const EncParams& p, OnceLds& t, uint64_t c) {
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t N = p.n_streams, L = 1u << p.table_log;
    auto publish = [&](uint32_t words) { __hip_atomic_store(&p.chunks[c].payload_words, words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // FINISH: where the chunk's words begin; the last chunk knows the total
    auto settle = [&](uint64_t before, uint64_t padded) {
        if (tid != 0) return;
        p.chunks[c].payload_offset = p.payload_word_offset + before;
        if (c + 1u < p.n_chunks) return;
        *p.used = before + padded;
        if (before + padded > p.payload_cap_words) report(p.status, ANSZP_ST_NO_SPACE);
    };
    auto settle_empty = [&]() {
        uint64_t before = 0;
        const bool known = words_before(p, c, p.spin_limit, t.before, t.gave_up, before);
        if (known) settle(before, 0u);
        return known;
    };
    uint32_t layer;
    anszp_pack_job_t job;
    uint64_t local;
    if (!layer_of_chunk(p, c, layer, job, local)) {         // the jobs do not cover the chunks the caller counted
        if (tid == 0) {
            report(p.status, ANSZP_ST_BAD_DESC);
            anszp_chunk_t* const d = &p.chunks[c];
            d->layer_id = d->n_symbols = d->stream_offset = 0u;
            d->out_offset = FINISH ? 0u : kNotWritten;
            publish(0u);
        }
        if (tid < N) p.stream_hdr[c * N + tid] = 0u;
        return FINISH ? settle_empty() : true;
    }
    const bool ok = layer_tables(p, layer, t.tables, t.spread);
    const uint64_t out_offset = p.out_offset + job.first_symbol + local * job.chunk_size;
    auto describe = [&](uint32_t n_symbols, bool later) {
        anszp_chunk_t* const d = &p.chunks[c];
        d->layer_id = p.jobs ? layer : p.layer_id;
        d->n_symbols = n_symbols;
        d->out_offset = out_offset | (later && !FINISH ? kNotWritten : 0u);
        d->stream_offset = p.stream_offset + static_cast<uint32_t>(c) * N;
    };
    if (!ok) {
        if (tid == 0 && local == 0) report(p.status, ANSZP_ST_BAD_FREQ);
        if (!p.jobs) {                                      // (one layer: nothing is written)
            if (FINISH && tid == 0 && c + 1u == p.n_chunks) *p.used = 0ull;
            return true;
        }
        if (tid < N) p.stream_hdr[c * N + tid] = 0u;
        if (tid == 0) {
            describe(0u, true);
            publish(0u);
        }
        return FINISH ? settle_empty() : true;
    }
    const ChunkStreams s = streams_of(p, job, local, lane);
    if (tid == 0) t.bad = t.over = 0u;
    const uint32_t batches = (s.max_len + kRows - 1u) / kRows, skip = batches * kRows - s.max_len;   // the first batch's first `skip` places are empty
    // (the tables have been built: what they were built with makes room for the ring)
    __syncthreads();
    auto next_phase = [] { asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory"); };     // (loads from global memory stay under way)
    // Phase ph: batch ph is loaded, ph - 1 read by the walk, ph - 2 walked, ph - 3 packed.
    const uint32_t phases = batches + 3u;
    if (wave == 0u) {
        __builtin_amdgcn_s_setprio(3);
        uint32_t x = L;
        const uint8_t* const next = reinterpret_cast<const uint8_t*>(t.tables.next);
        // (the sum's upper half is the number of bits dropped, and as f_s << k ends in k zeros its lowest bits are the
        // state's: all that the packing wavefront needs)
        auto step = [&](const uint2 i, uint32_t& note) {
            const uint32_t sum = x + i.x;
            uint32_t kept;                                  // x >> (the count in the sum's upper half)
            asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD" : "=v"(kept) : "v"(sum), "v"(x));
            x = *reinterpret_cast<const uint16_t*>(next + (2u * kept + i.y));
            note = sum;
        };
        auto walk = [&](uint32_t b, const uint2 (&info)[kRows], uint2 (&then)[kRows]) {
            const uint2* const row = &t.ring[(b + 1u) & 1u][0][lane];           // (behind the last batch: read, and not used)
            uint32_t* const note = &t.sums[b & 1u][0][lane];
#pragma unroll
            for (uint32_t j = 0; j < kRows; ++j) {
                step(info[j], note[j * kWave]);
                then[j] = row[j * kWave];
            }
            next_phase();
        };
        uint2 info_a[kRows], info_b[kRows];
        next_phase();
#pragma unroll
        for (uint32_t j = 0; j < kRows; ++j) info_a[j] = t.ring[0][j][lane];
        next_phase();
#pragma unroll
        for (uint32_t j = 0; j < kRows; ++j) {              // the first batch: its first `skip` places are empty, in some lanes one more
            info_b[j] = t.ring[1][j][lane];
            uint32_t note = 0u;
            if (j > skip || (j == skip && s.has_last)) step(info_a[j], note);
            t.sums[0][j][lane] = note;
        }
        next_phase();
        for (uint32_t b = 1; b < batches; b += 2u) {
            walk(b, info_b, info_a);
            if (b + 1u >= batches) break;
            walk(b + 1u, info_a, info_b);
        }
        t.x[lane] = s.has_any ? x - L : 0u;
        next_phase();
        __builtin_amdgcn_s_setprio(0);
    } else if (wave == 1u) {
        __builtin_amdgcn_s_setprio(2);
        // A word is written to its place whenever bits have been added to it, whether it is full or not: no branch.
        uint32_t low = 0, count = 0, bits = 0;              // the bits of the word being filled, how many; of the stream
        uint32_t at = lds_offset(t.bits) + 4u * lane;
        const uint32_t last = at + 4u * kBitsStride * kBitRows;         // (a row for what finds no room)
        next_phase();
        next_phase();
        next_phase();
        for (uint32_t b = 0; b < batches; ++b) {
            const uint32_t* const note = &t.sums[b & 1u][0][lane];
            uint32_t sum[kRows];
#pragma unroll
            for (uint32_t j = 0; j < kRows; ++j) sum[j] = note[j * kWave];
#pragma unroll
            for (uint32_t j = 0; j < kRows; j += 2u) {      // at most 24 bits
                const uint32_t n0 = sum[j] >> 16, n1 = sum[j + 1u] >> 16, n = n0 + n1;
                const uint32_t two = __builtin_amdgcn_ubfe(sum[j + 1u], 0u, n1) << n0 | __builtin_amdgcn_ubfe(sum[j], 0u, n0);
                const uint32_t carry = (two >> 1) >> (~count & 31u);
                low |= two << count;
                *reinterpret_cast<lds_word_t*>(static_cast<uintptr_t>(at)) = low;
                count += n;
                bits += n;
                const bool full = count >= 32u;
                low = full ? carry : low;
                at = min(full ? at + 4u * kBitsStride : at, last);
                count &= 31u;
            }
            if (b + 1u < batches) next_phase();
        }
        *reinterpret_cast<lds_word_t*>(static_cast<uintptr_t>(at)) = low;
        if (!s.has_any) bits = 0u;
        uint32_t nw = (bits + 31u) >> 5;
        const bool too_long = nw > 0xFFFFu;
        nw = min(nw, 0xFFFFu);
        const bool over = __ballot(nw > kBitRows) != 0ull;
        const uint32_t upto = spread_wave_sum(nw), words = __builtin_amdgcn_readlane(upto, kWave - 1);
        const uint64_t fifth = __ballot((bits & 16u) != 0u);
        if (lane == 0) {
            describe(s.cn, over);
            publish(words);
            t.fifth = fifth;
            if (over) t.over = 1u;
        }
        if (__ballot(too_long) && lane == 0) report(p.status, ANSZP_ST_NO_SPACE);
        t.first[lane] = upto - nw;
        t.n_words[lane] = nw;
        t.pad[lane] = (32u - bits) & 31u;
        next_phase();
    } else {
        // loading wavefronts: 2, 3, 6 and 7 (the others share a SIMD with the wavefronts above, as SIMDs are dealt out)
        const bool loads = (wave & 2u) != 0u;
        const uint32_t from = ((wave & 1u) + (wave >> 2) * 2u) * kRowsPerLoader;
        uint32_t sym_a[kRowsPerLoader] = {}, sym_b[kRowsPerLoader] = {}, lowest = 0xFFFFFFFFu;
        auto fetch = [&](uint32_t b, uint32_t (&sym)[kRowsPerLoader]) {
            if (b >= batches) return;
#pragma unroll
            for (uint32_t j = 0; j < kRowsPerLoader; ++j) {
                const uint32_t place = max(b * kRows + from + j, skip);
                // (a lane without a symbol in the last row takes another one there, which is neither walked nor packed)
                const uint32_t row = s.max_len - 1u - (place - skip);
                global_uint8_t* const at = s.chunk + uint64_t(row) * N;
                sym[j] = place == skip && !s.has_last ? s.chunk[s.lane_off] : at[s.lane_off];
            }
        };
        auto prepare = [&](uint32_t b, uint32_t slot, const uint32_t (&sym)[kRowsPerLoader]) {
            if (b >= batches) return;
            uint2 info[kRowsPerLoader];
#pragma unroll
            for (uint32_t j = 0; j < kRowsPerLoader; ++j) info[j] = t.tables.info[sym[j]];
#pragma unroll
            for (uint32_t j = 0; j < kRowsPerLoader; ++j) {
                lowest = min(lowest, info[j].x);
                t.ring[slot][from + j][lane] = info[j];
            }
        };
        if (loads) { fetch(0u, sym_a); fetch(1u, sym_b); }
        for (uint32_t ph = 0; ph < phases; ph += 2u) {
            if (loads) {
                prepare(ph, 0u, sym_a);
                fetch(ph + 2u, sym_a);
            }
            next_phase();
            if (ph + 1u >= phases) break;
            if (loads) {
                prepare(ph + 1u, 1u, sym_b);
                fetch(ph + 3u, sym_b);
            }
            next_phase();
        }
        if (lowest == 0u) t.bad = 1u;
    }
    __syncthreads();
    if (tid == 0 && t.bad) report(p.status, ANSZP_ST_BAD_SYMBOL);
    const bool over = t.over != 0u;
    uint64_t before = 0;
    const bool known = (FINISH || !over) && words_before(p, c, p.spin_limit, t.before, t.gave_up, before);
    const uint32_t nw = t.n_words[lane], n_words = __builtin_amdgcn_readlane(t.first[lane] + nw, kWave - 1);
    const uint64_t padded = (uint64_t(n_words) + 3ull) & ~3ull;
    if (wave == 0u && lane < N)
        p.stream_hdr[c * N + lane] = t.x[lane] | (FINISH || known ? 0u : ((32u - t.pad[lane]) & 15u) << 12) | nw << 16;
    if constexpr (FINISH) {
        if (!known) return false;
        settle(before, padded);
    } else {
        if (!known) {
            if (tid == 0) {
                p.chunks[c].payload_offset = t.fifth;
                p.chunks[c].out_offset = out_offset | kNotWritten;
            }
            return true;
        }
        if (tid == 0) p.chunks[c].payload_offset = p.payload_word_offset + before;
    }
    if (before > p.payload_cap_words || padded > p.payload_cap_words - before) return true;    // no room: reported with the total
    uint32_t* const out = p.payload + before;
    // A wavefront takes a stream at a time, a lane every 64th word: the bits as laid down, moved up by the zero bits behind
    // the stream's last one, are whole words of the stream from its last to its first, bit-reversed.
    for (uint32_t k = wave; k < N; k += kWaves) {
        const uint32_t n = __builtin_amdgcn_readfirstlane(t.n_words[k]), pad = __builtin_amdgcn_readfirstlane(t.pad[k]);
        uint32_t* const words = out + __builtin_amdgcn_readfirstlane(t.first[k]);
        for (uint32_t m = lane; m < n; m += kWave) {
            const uint32_t hi = t.bits[m * kBitsStride + k], lo = m ? t.bits[(m - 1u) * kBitsStride + k] : 0u;
            words[n - 1u - m] = __brev(static_cast<uint32_t>(((uint64_t(hi) << 32 | lo) << pad) >> 32));
        }
    }
    if (tid < padded - n_words) out[n_words + tid] = 0u;        // up to three pad words
    return true;
}

// Without scratch memory: encode_rest behind it.
__global__ __launch_bounds__(kThreads, 4) void encode_once(EncParams p) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kOnceLds];
    encode_chunk<false>(p, *reinterpret_cast<OnceLds*>(lds), blockIdx.x);
}

// A stream's words symbol by symbol, nothing asked for ahead: for the few chunks the last workgroup writes, in little code.
__device__ __forceinline__ uint32_t walk_plain(const EncTables& t, const ChunkStreams& s, uint32_t N, uint32_t L, uint32_t* words, uint32_t n_words, uint32_t pad) {
    uint32_t x = L, bits = 0, cnt = pad, at = n_words;
    uint64_t acc = 0;
#pragma unroll 1
    for (uint32_t row = s.max_len; row-- > 0u;) {
        if (row + 1u == s.max_len && !s.has_last) continue;
        const uint2 i = t.info[(s.chunk + uint64_t(row) * N)[s.lane_off]];
        const uint32_t nb = (x + i.x) >> 16;
        acc |= uint64_t(__builtin_amdgcn_ubfe(x, 0u, nb)) << cnt;
        cnt += nb;
        bits += nb;
        if (cnt >= 32u) {
            if (at) words[--at] = __brev(static_cast<uint32_t>(acc));
            acc >>= 32;
            cnt -= 32u;
        }
        x = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(t.next) + (2u * (x >> nb) + i.y));
    }
    return bits;
}

// With it, and with streams that fit LDS whatever their symbols: the last workgroup to be done writes the chunks of those that
// gave up waiting (all chunks' words are published by then), and no launch is needed behind this one: 144 chunks of 16,384
// symbols with their tables 34.6 -> 32.8 us, three layers of 533,769 30.5 -> 29.8.  (Writing chunks that do not fit here too took
// the kernel 85 KB of code and registers to scratch memory: 69 us.)
__global__ __launch_bounds__(kThreads, 4) void encode_all(EncParams p) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kOnceLds];
    OnceLds& t = *reinterpret_cast<OnceLds*>(lds);
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1u);
    uint32_t* const left = p.finish + 1;
    const bool done = encode_chunk<true>(p, t, blockIdx.x);
    __syncthreads();
    if (tid == 0) {
        if (!done) {
            atomicOr(&left[blockIdx.x / 32u], 1u << blockIdx.x % 32u);
            __threadfence();                                // (before it is counted as done)
        }
        t.over = atomicAdd(&p.finish[0], 1u) + 1u == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (!t.over) return;
    __threadfence();
    const uint32_t marks = __hip_atomic_load(&left[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    static_assert(kFinishWords == 1u + kWave, "a lane a word");
    for (uint64_t c = 0; c < p.n_chunks; ++c) {             // (alike for every thread)
        const uint32_t word = __builtin_amdgcn_readlane(marks, uint32_t(c) / 32u);
        if (!word) c |= 31u;                                // none of the word's
        if (!(word >> c % 32u & 1u)) continue;
        __syncthreads();                                    // (what words_before and the tables use is free)
        uint64_t before = 0;
        const bool known = words_before(p, c, 1u << 16, t.before, t.gave_up, before);
        uint32_t layer, nw = 0, bits = 0;
        anszp_pack_job_t job;
        uint64_t local;
        const bool ok = layer_of_chunk(p, c, layer, job, local) && layer_tables(p, layer, t.tables, t.spread);
        if (tid >= kWave) continue;
        ChunkStreams s{};
        if (ok) {
            s = streams_of(p, job, local, lane);
            bits = s.has_any ? walk_plain(t.tables, s, p.n_streams, 1u << p.table_log, nullptr, 0u, 0u) : 0u;
            nw = (bits + 31u) >> 5;
        }
        const uint32_t upto = spread_wave_sum(nw), words = __builtin_amdgcn_readlane(upto, kWave - 1u);
        const uint64_t padded = (uint64_t(words) + 3ull) & ~3ull;
        const bool room = before <= p.payload_cap_words && padded <= p.payload_cap_words - before;
        if (tid == 0) {
            p.chunks[c].payload_offset = p.payload_word_offset + before;
            if (!known) report(p.status, ANSZP_ST_INTERNAL);
            if (c + 1u == p.n_chunks) {
                *p.used = before + padded;
                if (!room) report(p.status, ANSZP_ST_NO_SPACE);
            }
        }
        if (!ok || !known || !room) continue;
        walk_plain(t.tables, s, p.n_streams, 1u << p.table_log, p.payload + before + (upto - nw), nw, (32u - bits) & 31u);
        if (lane < padded - words) p.payload[before + words + lane] = 0u;       // up to three pad words
    }
}

// Behind it: the total, and the chunks that were not written.
__global__ __launch_bounds__(kThreads, 4) void encode_rest(EncParams p) {
    __shared__ EncLds t;
    __shared__ unsigned long long sum;
    const uint32_t tid = threadIdx.x;
    const uint64_t c = blockIdx.x;
    const bool last = c + 1u == p.n_chunks;
    if (!p.jobs && !one_layer_ok(p)) {
        if (last && tid == 0) *p.used = 0ull;
        return;
    }
    const anszp_chunk_t d = p.chunks[c];
    const bool written = !(d.out_offset & kNotWritten);
    if (!written || last) {                                     // words before this chunk
        if (tid == 0) sum = 0ull;
        __syncthreads();
        unsigned long long mine = 0;
        for (uint64_t i = tid; i < c; i += kThreads) mine += (uint64_t(p.chunks[i].payload_words) + 3ull) & ~3ull;
        if (mine) atomicAdd(&sum, mine);
        __syncthreads();
    }
    if (last && tid == 0) {
        const uint64_t used = sum + ((uint64_t(d.payload_words) + 3ull) & ~3ull);
        *p.used = used;
        if (used > p.payload_cap_words) report(p.status, ANSZP_ST_NO_SPACE);
    }
    uint32_t layer;
    anszp_pack_job_t job;
    uint64_t local;
    if (written) return;
    const bool has_layer = layer_of_chunk(p, c, layer, job, local);
    if (d.n_symbols == 0u) {                                    // no layer, or one of bad frequencies
        if (tid == 0) {
            p.chunks[c].out_offset = has_layer ? p.out_offset + job.first_symbol + local * job.chunk_size : 0u;
            p.chunks[c].payload_offset = p.payload_word_offset + sum;
        }
        return;
    }
    if (!layer_tables(p, layer, t, t.spread)) return;      // (they were there: the chunk has symbols)
    if (tid >= kWave) return;
    if (tid == 0) p.chunks[c].payload_offset = p.payload_word_offset + sum;
    write_chunk(p, t, job, local, c, d.payload_words, p.payload_word_offset + sum, d.payload_offset);
}

// Chunks per workgroup: one as long as every CU gets no more than two workgroups (a walk is a chain: the fewer wavefronts
// share a SIMD the better), then as many as keep it at two, so that a layer's tables are built by few workgroups and the
// grid stays small however many chunks there are.  (With no more chunks than a workgroup has wavefronts, every eight of
// 100,000 chunks of 2,048 symbols paid for tables of their own: 1,092 us, 438 with this; 20,000 chunks 233, 122;
// the 369 chunks of a ResNet-50-shaped set as before.)
uint32_t chunks_per_group(uint64_t n_chunks) {
    const uint64_t resident = std::min(2u * device_cus(), 32u * (kFinishWords - 1u));
    return uint32_t(std::max<uint64_t>(1u, (n_chunks + resident - 1u) / resident));
}

int launch(EncParams& p, hipStream_t s) {
    p.chunks_per_group = chunks_per_group(p.n_chunks);
    if (p.n_chunks && p.chunks_per_group == 1u) {
        // (a look at the others' words takes about 0.4 us: some 25 ms)
        const uint32_t looks = spin_limit_for_tests().load(std::memory_order_relaxed);
        p.spin_limit = looks ? looks - 1u : 1u << 16;
        const dim3 groups(uint32_t(p.n_chunks)), threads(kThreads);
        // (a symbol has at most table_log bits)
        const uint64_t rows = (uint64_t(p.longest_chunk) + p.n_streams - 1u) / p.n_streams;
        if (p.prepared && rows * p.table_log <= 32u * kBitRows) {
            hipLaunchKernelGGL(encode_all, groups, threads, 0, s, p);
            return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
        }
        if (!p.prepared) hipLaunchKernelGGL(encode_begin, dim3(1), threads, 0, s, p);
        hipLaunchKernelGGL(encode_once, groups, threads, 0, s, p);
        hipLaunchKernelGGL(encode_rest, groups, threads, 0, s, p);
        return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
    }
    const uint64_t groups = (p.n_chunks + p.chunks_per_group - 1u) / p.chunks_per_group;
    if (groups) hipLaunchKernelGGL(encode_sizes, dim3(uint32_t(groups)), dim3(kThreads), 0, s, p);
    else if (!p.jobs) hipLaunchKernelGGL(encode_nothing, dim3(1), dim3(kWave), 0, s, p);
    hipLaunchKernelGGL(encode_scan, dim3(1), dim3(kThreads), 0, s, p);
    if (groups) hipLaunchKernelGGL(encode_write, dim3(uint32_t(groups)), dim3(kThreads), 0, s, p);
    return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
}

}  // namespace

extern "C" uint64_t anszp_pack_scratch_bytes(uint32_t n_layers, int table_log) {
    if (table_log < 1 || table_log > ANSZP_MAX_TABLE_LOG) return 0;
    return uint64_t(n_layers) * (sizeof(anszp_pack_job_t) + 4u * record_words(uint32_t(table_log))) + (4u * kFinishWords + 15u) / 16u * 16u;
}

extern "C" int anszp_pack_set_device(const anszp_pack_set_t* a, void* stream) {
    if (!a || !a->payload_words_used || !a->status || !a->scratch || (a->n_layers && (!a->layer_symbols || !a->chunk_sizes || !a->freqs))) return ANSZP_E_NULL;
    if (a->table_log < 1 || a->table_log > ANSZP_MAX_TABLE_LOG || a->n_streams < 1 || a->n_streams > ANSZP_MAX_STREAMS || (a->payload_word_offset & 3) ||
        (a->single && a->n_layers != 1u) || a->n_layers >= (1u << 27) || a->scratch_bytes < anszp_pack_scratch_bytes(a->n_layers, int(a->table_log)) ||
        (reinterpret_cast<uintptr_t>(a->scratch) & 15) ||
        (a->clear && ((reinterpret_cast<uintptr_t>(a->chunks) | reinterpret_cast<uintptr_t>(a->stream_hdr) | reinterpret_cast<uintptr_t>(a->payload)) & 15)))
        return ANSZP_E_RANGE;
    uint64_t n_chunks = 0, n_symbols = 0, longest = 0;
    for (uint32_t l = 0; l < a->n_layers; ++l) {
        if (!a->chunk_sizes[l] || a->layer_symbols[l] >= (1ull << 63)) return ANSZP_E_RANGE;
        n_chunks += (a->layer_symbols[l] + a->chunk_sizes[l] - 1u) / a->chunk_sizes[l];
        n_symbols += a->layer_symbols[l];
        longest = std::max(longest, std::min<uint64_t>(a->layer_symbols[l], a->chunk_sizes[l]));
        if (n_chunks >= (1ull << 32) || n_symbols >= (1ull << 63)) return ANSZP_E_RANGE;
    }
    if (!a->single && (n_chunks >= (1ull << 31) || n_chunks * a->n_streams >= (1ull << 32))) return ANSZP_E_RANGE;
    if (n_chunks && (!a->symbols || !a->chunks || !a->stream_hdr)) return ANSZP_E_NULL;
    if (!a->payload && a->payload_cap_words) return ANSZP_E_NULL;
    if (a->clear && ((a->clear_chunks && !a->chunks) || (a->clear_stream_hdr && !a->stream_hdr) || (a->clear_payload_words && !a->payload))) return ANSZP_E_NULL;
    if (a->clear && a->clear_chunks < n_chunks) return ANSZP_E_RANGE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    EncParams p{};
    p.symbols = a->symbols; p.freqs = a->freqs; p.chunks = a->chunks; p.stream_hdr = a->stream_hdr; p.payload = a->payload;
    p.used = reinterpret_cast<unsigned long long*>(a->payload_words_used); p.status = a->status;
    p.n_chunks = n_chunks; p.payload_word_offset = a->payload_word_offset; p.payload_cap_words = a->payload_cap_words;
    p.out_offset = a->out_offset; p.n_layers = a->n_layers; p.table_log = a->table_log; p.n_streams = a->n_streams;
    p.layer_id = a->layer_id; p.stream_offset = a->stream_offset; p.longest_chunk = uint32_t(longest);
    if (!a->single && (a->layer_id || a->stream_offset || a->out_offset || a->payload_word_offset)) return ANSZP_E_RANGE;
    PrepareParams q{};
    JobsArg jobs;
    anszp_pack_job_t* const jobs_dev = static_cast<anszp_pack_job_t*>(a->scratch);
    q.records = reinterpret_cast<uint32_t*>(jobs_dev + a->n_layers);
    p.finish = q.records + size_t(a->n_layers) * record_words(p.table_log);
    if (!a->single) {
        p.jobs = q.jobs = jobs_dev;
    } else {
        p.one.n_symbols = a->layer_symbols[0]; p.one.chunk_size = a->chunk_sizes[0];
    }
    if (q.jobs) {                                           // by the kernels' arguments: no copy from host memory
        uint64_t symbol = 0, chunk = 0;
        for (uint32_t l = 0; l < a->n_layers; ++l) {
            if (q.n_jobs == kJobsPerLaunch) {
                hipLaunchKernelGGL(encode_jobs, dim3(1), dim3(kJobsPerLaunch), 0, s, q, jobs);
                q.first_job = l;
                q.n_jobs = 0;
            }
            jobs.job[q.n_jobs++] = anszp_pack_job_t{symbol, a->layer_symbols[l], a->chunk_sizes[l], uint32_t(chunk), {0u, 0u}};
            symbol += a->layer_symbols[l];
            chunk += (a->layer_symbols[l] + a->chunk_sizes[l] - 1u) / a->chunk_sizes[l];
        }
    }
    q.clear = a->clear ? 1u : 0u;
    q.shares = std::max(1u, (1u << p.table_log) / kThreads);
    q.table_groups = n_chunks ? a->n_layers * q.shares : 0u;    // (without chunks nobody reads them)
    q.chunk_units = 2u * (a->clear ? a->clear_chunks : n_chunks);
    q.hdr_words = a->clear_stream_hdr; q.payload_words = a->clear_payload_words;
    const uint64_t units = q.chunk_units + (a->clear ? (q.hdr_words + 3u) / 4u + (q.payload_words + 3u) / 4u : 0u);
    const uint64_t groups = q.table_groups + std::max<uint64_t>(1u, (units + kClearUnits - 1u) / kClearUnits);
    if (groups >= (1ull << 31)) return ANSZP_E_RANGE;
    hipLaunchKernelGGL(encode_prepare, dim3(uint32_t(groups)), dim3(kThreads), 0, s, p, q, jobs);
    p.prepared = n_chunks ? q.records : nullptr;
    return launch(p, s);
}

extern "C" int anszp_pack_layers_device(const uint8_t* symbols_dev, const anszp_pack_job_t* jobs_dev, uint32_t n_layers,
                                        uint64_t n_chunks, const uint32_t* freqs_dev, int table_log, int n_streams,
                                        anszp_chunk_t* chunks_dev, uint32_t* stream_hdr_dev, uint32_t* payload_dev,
                                        uint64_t payload_cap_words, uint64_t* payload_words_used_dev,
                                        uint32_t* status_dev, void* stream) {
    if (!payload_words_used_dev || !status_dev) return ANSZP_E_NULL;
    if (n_chunks && (!symbols_dev || !jobs_dev || !freqs_dev || !chunks_dev || !stream_hdr_dev)) return ANSZP_E_NULL;
    if (!payload_dev && payload_cap_words) return ANSZP_E_NULL;
    if (table_log < 1 || table_log > ANSZP_MAX_TABLE_LOG || n_streams < 1 || n_streams > ANSZP_MAX_STREAMS ||
        n_chunks >= (1ull << 31) || uint64_t(n_chunks) * uint64_t(n_streams) >= (1ull << 32) || (n_chunks && n_layers == 0))
        return ANSZP_E_RANGE;
    EncParams p{};
    p.symbols = symbols_dev; p.freqs = freqs_dev; p.chunks = chunks_dev; p.stream_hdr = stream_hdr_dev;
    p.payload = payload_dev; p.used = reinterpret_cast<unsigned long long*>(payload_words_used_dev); p.status = status_dev;
    p.n_chunks = n_chunks; p.payload_cap_words = payload_cap_words;
    p.table_log = uint32_t(table_log); p.n_streams = uint32_t(n_streams);
    p.jobs = jobs_dev; p.n_layers = n_layers;
    return launch(p, static_cast<hipStream_t>(stream));
}

extern "C" int anszp_pack_layer_device(const uint8_t* symbols_dev, uint64_t n_symbols, const uint32_t* freqs_dev,
                                       int table_log, int n_streams, uint32_t chunk_size, uint32_t layer_id,
                                       uint64_t out_offset, uint64_t payload_word_offset, uint32_t stream_offset,
                                       anszp_chunk_t* chunks_dev, uint32_t* stream_hdr_dev, uint32_t* payload_dev,
                                       uint64_t payload_cap_words, uint64_t* payload_words_used_dev,
                                       uint32_t* status_dev, void* stream) {
    if (!freqs_dev || !payload_words_used_dev || !status_dev) return ANSZP_E_NULL;
    if (n_symbols && (!symbols_dev || !chunks_dev || !stream_hdr_dev)) return ANSZP_E_NULL;
    if (!payload_dev && payload_cap_words) return ANSZP_E_NULL;
    if (table_log < 1 || table_log > ANSZP_MAX_TABLE_LOG || n_streams < 1 || n_streams > ANSZP_MAX_STREAMS ||
        chunk_size < 1 || (payload_word_offset & 3))
        return ANSZP_E_RANGE;
    EncParams p{};
    p.symbols = symbols_dev; p.freqs = freqs_dev; p.chunks = chunks_dev; p.stream_hdr = stream_hdr_dev;
    p.payload = payload_dev; p.used = reinterpret_cast<unsigned long long*>(payload_words_used_dev); p.status = status_dev;
    p.one.n_symbols = n_symbols; p.one.chunk_size = chunk_size;
    p.n_chunks = (n_symbols + chunk_size - 1) / chunk_size;
    p.out_offset = out_offset; p.payload_word_offset = payload_word_offset; p.payload_cap_words = payload_cap_words;
    p.n_layers = 1; p.table_log = uint32_t(table_log); p.n_streams = uint32_t(n_streams);
    p.layer_id = layer_id; p.stream_offset = stream_offset;
    if (p.n_chunks >= (1ull << 32)) return ANSZP_E_RANGE;
    return launch(p, static_cast<hipStream_t>(stream));
}
