// tANS encoder on the GPU: compresses layers whose symbols are in device memory into the container
// anszp_decode reads, word for word what the host packer (anszp_pack_layer) writes.
//
// Encoding (Sec. II-A) walks a stream's symbols backwards: to encode symbol s in state x (in
// [L, 2L)) the low bits of x are dropped, and written out, until x lies in [f_s, 2 f_s); the new
// state is the (x - f_s)-th state of s, counted in increasing order, plus L.  The decoder reads the
// bits of the first symbol first, so a stream's bits are laid down from its end: the walk is done
// once to learn the stream's length and once to write.
//
// Three launches, nothing allocated and no scratch memory: sizes (every stream's final state and
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
    uint64_t n_chunks, out_offset, payload_word_offset, payload_cap_words;
    uint32_t n_layers, table_log, n_streams, layer_id, stream_offset, chunks_per_group;
};

// A layer's encoding tables.  info[s]: what x + info.x has in its upper half is the number of bits symbol s drops
// in state x; 2 * (x >> that) + info.y is the byte of `next` that holds the new state plus L.  A symbol without a
// frequency has info.x = 0 (no other symbol has), drops nothing and leads to some state.
struct EncLds {
    SpreadLds spread;
    uint2 info[ANSZP_ALPHABET];
    uint16_t next[kSpreadStates];
};

__device__ __forceinline__ void report(uint32_t* status, uint32_t bits) {
    atomicOr(&status[0], bits);
    atomicAdd(&status[1], 1u);
}

// The workgroup's encoding tables.  False (for every thread) when the frequencies do not sum to L.
__device__ __forceinline__ bool build_tables(const uint32_t* freqs, uint32_t table_log, EncLds& t) {
    const uint32_t tid = threadIdx.x, L = 1u << table_log;
    const bool ok = spread_states<kThreads>(freqs, table_log, t.spread, [&](uint32_t g, uint32_t, uint32_t, uint32_t, uint32_t state) {
        t.next[g] = static_cast<uint16_t>(L + state);
    });
    if (!ok) return false;
    if (tid < ANSZP_ALPHABET) {
        const uint32_t f = t.spread.f[tid];
        // x in [L, 2L) drops k or k - 1 bits, k = table_log - floor(log2 f): k when x >= f << k
        const uint32_t k = f ? table_log - (31u - static_cast<uint32_t>(__clz(f))) : 0u;
        t.info[tid] = f ? make_uint2((k << 16) - (f << k), 2u * (t.spread.first[tid] - f)) : make_uint2(0u, 0u - 2u * L);
    }
    __syncthreads();
    return true;
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
__device__ __forceinline__ uint32_t walk_stream(const EncLds& t, const ChunkStreams& s, uint32_t N, uint32_t L, uint32_t* words, uint32_t n_words,
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

// The layer chunk c belongs to (jobs are in chunk order: the last one whose first_chunk is not beyond c) and the
// chunk's number within it.  False when c belongs to no layer.
__device__ bool layer_of_chunk(const EncParams& p, uint64_t c, uint32_t& layer, anszp_pack_job_t& job, uint64_t& local) {
    layer = 0;
    if (!p.jobs) {
        job = p.one;
    } else {
        uint32_t lo = 0, hi = p.n_layers;
        if (hi == 0 || p.jobs[0].first_chunk > c) return false;
        while (hi - lo > 1u) {
            const uint32_t mid = (lo + hi) >> 1;
            if (p.jobs[mid].first_chunk <= c) lo = mid; else hi = mid;
        }
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
        const bool ok = build_tables(p.freqs + size_t(layer) * ANSZP_ALPHABET, p.table_log, t);
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

__global__ __launch_bounds__(kThreads, 4) void encode_write(EncParams p) {
    __shared__ EncLds t;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t N = p.n_streams, L = 1u << p.table_log;
    for_each_chunk(p, t, [&](const anszp_pack_job_t& job, uint32_t, uint64_t local, uint64_t c, bool ok) {
        if (!ok) return;                                        // reported by the first pass
        const ChunkStreams s = streams_of(p, job, local, lane);
        const anszp_chunk_t d = p.chunks[c];
        const uint32_t hdr = lane < N ? p.stream_hdr[c * N + lane] : 0u;
        const uint32_t nw = hdr >> 16;
        const uint32_t beyond = ((hdr >> 12) & 15u) | ((d.out_offset >> lane) & 1u ? 16u : 0u);   // bits of the last word, 0: all
        if (lane < N) p.stream_hdr[c * N + lane] = hdr & 0xFFFF0FFFu;
        if (lane == 0) p.chunks[c].out_offset = p.out_offset + job.first_symbol + local * job.chunk_size;
        const uint64_t at = d.payload_offset - p.payload_word_offset;          // in the caller's payload region
        const uint64_t padded = (uint64_t(d.payload_words) + 3ull) & ~3ull;
        if (at > p.payload_cap_words || padded > p.payload_cap_words - at) return;     // no room: reported by the scan
        uint32_t* words = p.payload + at + (spread_wave_sum(nw) - nw);
        uint32_t x = L, room = nw;
        bool bad = false;
        if (__ballot(nw == 0xFFFFu) != 0ull) {                  // a stream too long for its header is not written
            const uint32_t bits = walk_stream<false>(t, s, N, L, nullptr, 0u, 0u, x, bad);
            if (((bits + 31u) >> 5) != nw) room = 0u;
        }
        if (!s.has_any) room = 0u;
        walk_stream<true>(t, s, N, L, words, room, (32u - beyond) & 31u, x, bad);
        if (lane < padded - d.payload_words) p.payload[at + d.payload_words + lane] = 0u;   // up to three pad words
    }, [&](uint64_t) {});                                       // reported by the first pass
}

// Chunks per workgroup: one as long as every CU gets no more than two workgroups (a walk is a chain: the fewer wavefronts
// share a SIMD the better), then as many as keep it at two, so that a layer's tables are built by few workgroups and the
// grid stays small however many chunks there are.  (With no more chunks than a workgroup has wavefronts, every eight of
// 100,000 chunks of 2,048 symbols paid for tables of their own: 1,092 us, 438 with this; 20,000 chunks 233, 122;
// the 369 chunks of a ResNet-50-shaped set as before.)
uint32_t chunks_per_group(uint64_t n_chunks) {
    const uint64_t resident = 2u * device_cus();
    return uint32_t(std::max<uint64_t>(1u, (n_chunks + resident - 1u) / resident));
}

int launch(EncParams& p, hipStream_t s) {
    p.chunks_per_group = chunks_per_group(p.n_chunks);
    const uint64_t groups = (p.n_chunks + p.chunks_per_group - 1u) / p.chunks_per_group;
    if (groups) hipLaunchKernelGGL(encode_sizes, dim3(uint32_t(groups)), dim3(kThreads), 0, s, p);
    else if (!p.jobs) hipLaunchKernelGGL(encode_nothing, dim3(1), dim3(kWave), 0, s, p);
    hipLaunchKernelGGL(encode_scan, dim3(1), dim3(kThreads), 0, s, p);
    if (groups) hipLaunchKernelGGL(encode_write, dim3(uint32_t(groups)), dim3(kThreads), 0, s, p);
    return hipGetLastError() == hipSuccess ? ANSZP_OK : ANSZP_E_HIP;
}

}  // namespace

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
