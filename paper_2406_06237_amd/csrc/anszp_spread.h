// The states of every symbol, worked out by a workgroup in LDS (internal to the library; shared by the
// decode-table builder and the encoder).
//
// This library's choice of spread (Sec. II-A says only that the rate depends on how the states are initialised):
// occurrence i of a symbol of frequency f sits at (2i + 1) / (2f); all occurrences of all symbols are sorted by that
// fraction, ties going to the smaller symbol, and an occurrence's rank is its state.
//
// The rank is found by a counting sort: occurrence -> one of L buckets by the integer part of L (2i + 1) / (2f)
// (equal fractions share a bucket and buckets are ordered as the fractions are), a prefix sum over the buckets, and an
// exact comparison with the other occurrences of the same bucket: one division per state, and as many comparisons as a
// bucket has members.  On most tables these are a few, compared by their products (below 2^26; all symbols of odd
// frequency meet in the middle, but one bucket of a dozen is soon done).  Where symbols share a frequency they share all
// fractions, and every bucket has as many members as there are such symbols: then a second division gives every
// occurrence a number that orders its bucket by itself.  With r / 2f the place in the bucket, that is the integer part of
// 2L r / 2f (different fractions, of frequencies f + g <= L, are 1 / 2fg >= 2 / L^2 apart, so 4 apart here), the symbol
// below it.
// Counting the occurrences of every other symbol before each occurrence takes a division per state and symbol instead: with
// 2^12 states a decode table took 57 us that way (16 symbols; 218 us with 256), 36 us (46 us) this way by one workgroup.
// Flat rows of 2^12 states by several workgroups, by products -> by numbers: 16 symbols 25 -> 16 us, 256 symbols
// 231 -> 60; tables with a crowded middle only as before.
#ifndef ANSZP_SPREAD_H
#define ANSZP_SPREAD_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "anszp.h"

constexpr uint32_t kSpreadStates = 1u << ANSZP_MAX_TABLE_LOG;
constexpr uint32_t kSpreadFew = 8, kSpreadMany = 24;      // crowded: that many lanes of a wavefront have an occurrence that is not
                                                          // among the first kSpreadFew of its bucket

struct SpreadLds {
    uint32_t f[ANSZP_ALPHABET];
    uint32_t first[ANSZP_ALPHABET];        // occurrences of smaller symbols: occurrence i of symbol s is number first[s] + i
    uint32_t bucket[kSpreadStates];        // members of each bucket, then where each bucket's members start
    uint32_t member[kSpreadStates];        // bucket after bucket: f - 1 | i << 12 | symbol << 24 (crowded: order in the bucket << 8 | symbol)
    uint32_t part[16];                     // a wavefront's share of a prefix sum
    uint32_t crowded;                      // many buckets have many members
};

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ uint32_t spread_wave_sum(uint32_t v) {
    int x = static_cast<int>(v);
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);      // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);      // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);      // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);      // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2 and 3
    return static_cast<uint32_t>(x);
}

// Called by all THREADS threads of the workgroup.  place(g, symbol, f, i, state): for every occurrence (g = first[symbol] + i)
// once, by some thread.  False (for every thread, nothing placed) when the frequencies do not sum to 2^table_log.
// Ends without a barrier behind the calls of place.
template <uint32_t THREADS, class PLACE>
__device__ __forceinline__ bool spread_states(const uint32_t* freqs, uint32_t table_log, SpreadLds& t, PLACE&& place) {
    static_assert(THREADS >= ANSZP_ALPHABET && THREADS <= 1024u && kSpreadStates % THREADS == 0, "a thread per symbol, sixteen shares");
    constexpr uint32_t kPerThread = kSpreadStates / THREADS;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t L = 1u << table_log;
    uint32_t fs = 0, upto = 0;
    if (tid < ANSZP_ALPHABET) {
        fs = freqs[tid];
        upto = spread_wave_sum(min(fs, L + 1u));               // (a frequency beyond L cannot wrap the sum around)
        if (lane == 63u) t.part[wave] = upto;
    }
    for (uint32_t b = tid; b < L; b += THREADS) t.bucket[b] = 0u;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (uint32_t w = 0; w < ANSZP_ALPHABET / 64u; ++w) {
        if (w == wave) upto += total;
        total += t.part[w];
    }
    if (total != L) return false;
    if (tid < ANSZP_ALPHABET) {
        t.f[tid] = fs;
        t.first[tid] = upto - fs;
        t.crowded = 0u;
    }
    __syncthreads();
    // occurrence g: its symbol, frequency, number among the symbol's, bucket
    auto occurrence = [&](uint32_t g, uint32_t& sy, uint32_t& f, uint32_t& i) {
        sy = 0;                                                // the largest symbol with first[sy] <= g (it has a frequency)
#pragma unroll
        for (uint32_t step = ANSZP_ALPHABET / 2u; step; step >>= 1)
            sy += t.first[sy + step] <= g ? step : 0u;
        f = t.f[sy];
        i = g - t.first[sy];
        return ((2u * i + 1u) << table_log) / (2u * f);        // below 2^26; i < f, so below L
    };
    uint32_t mine[kPerThread], at[kPerThread] = {};     // as in `member`; bucket | place within it << 16
    uint32_t places = 0;
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) {
        const uint32_t g = tid + u * THREADS;
        if (g < L) {
            uint32_t sy, f, i;
            const uint32_t b = occurrence(g, sy, f, i);
            mine[u] = (f - 1u) | i << 12 | sy << 24;
            at[u] = b | atomicAdd(&t.bucket[b], 1u) << 16;     // below 2^12 both
        }
        places |= at[u];
    }
    // (kSpreadFew is a power of two: a place beyond it has a bit that high)
    if (__builtin_expect(__popcll(__ballot((places >> 16) >= kSpreadFew)) >= kSpreadMany, 0)) t.crowded = 1u;
    __syncthreads();
    {                                                          // counts -> starts: neighbouring buckets per thread
        const uint32_t per = max(L / THREADS, 1u), b0 = tid * per;
        uint32_t n[kPerThread], sum = 0;
#pragma unroll
        for (uint32_t u = 0; u < kPerThread; ++u) {
            n[u] = u < per && b0 + u < L ? t.bucket[b0 + u] : 0u;
            sum += n[u];
        }
        const uint32_t incl = spread_wave_sum(sum);
        if (lane == 63u) t.part[wave] = incl;
        __syncthreads();
        uint32_t start = incl - sum;
        for (uint32_t w = 0; w < wave; ++w) start += t.part[w];
#pragma unroll
        for (uint32_t u = 0; u < kPerThread; ++u) {
            if (u < per && b0 + u < L) t.bucket[b0 + u] = start;
            start += n[u];
        }
    }
    __syncthreads();
    uint32_t starts[kPerThread];                               // (asked for together with `crowded`, not behind the branch)
    const uint32_t crowded = t.crowded;
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) starts[u] = t.bucket[at[u] & 0xFFFFu];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(crowded), 0)) {        // (uniform)
        // (loops that work everything out again: less code beside the other tables' than from registers)
        auto key_of = [&](uint32_t g, uint32_t& sy, uint32_t& f, uint32_t& i, uint32_t& b) {
            b = occurrence(g, sy, f, i);
            const uint32_t rest = ((2u * i + 1u) << table_log) - b * 2u * f;             // below 2 f
            return (rest << (table_log + 1u)) / (2u * f) << 8 | sy;                      // (the division below 2^26)
        };
        uint32_t sy, f, i, b;
#pragma unroll 1
        for (uint32_t g = tid; g < L; g += THREADS) {
            const uint32_t key = key_of(g, sy, f, i, b);
            t.member[atomicAdd(&t.bucket[b], 1u)] = key;       // (behind this loop every bucket's entry is its end)
        }
        __syncthreads();
#pragma unroll 1
        for (uint32_t g = tid; g < L; g += THREADS) {
            const uint32_t key = key_of(g, sy, f, i, b), begin = b ? t.bucket[b - 1u] : 0u, end = t.bucket[b];
            // (from another member in every lane: occurrences of one symbol are in buckets of like sizes, whose members
            // in one place would share an LDS bank)
            uint32_t state = begin, m = begin + lane % (end - begin);
#pragma unroll 8
            for (uint32_t n = end - begin; n; --n) {
                state += t.member[m] < key ? 1u : 0u;
                m = m + 1u < end ? m + 1u : begin;
            }
            place(g, sy, f, i, state);
        }
        return true;
    }
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u)
        if (tid + u * THREADS < L) t.member[starts[u] + (at[u] >> 16)] = mine[u];
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) {
        const uint32_t g = tid + u * THREADS;
        if (g < L) {
            const uint32_t b = at[u] & 0xFFFFu;
            const uint32_t begin = t.bucket[b], end = b + 1u < L ? t.bucket[b + 1u] : L;
            const uint32_t f = (mine[u] & 0xFFFu) + 1u, i = (mine[u] >> 12) & 0xFFFu, s = mine[u] >> 24;
            uint32_t state = begin;
#pragma unroll 4
            for (uint32_t m = begin; m < end; ++m) {
                const uint32_t o = t.member[m];
                const uint32_t fo = (o & 0xFFFu) + 1u, io = (o >> 12) & 0xFFFu, so = o >> 24;
                // (2 io + 1) / fo against (2 i + 1) / f, ties to the smaller symbol (an occurrence is not before itself)
                const uint32_t theirs = __umul24(2u * io + 1u, f), ours = __umul24(2u * i + 1u, fo);
                state += theirs < ours || (theirs == ours && so < s) ? 1u : 0u;
            }
            place(g, s, f, i, state);
        }
    }
    return true;
}

#endif
