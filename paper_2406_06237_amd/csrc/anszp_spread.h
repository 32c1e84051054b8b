// The states of every symbol, worked out by a workgroup in LDS (internal to the library; shared by the
// decode-table builder and the encoder).
//
// This library's choice of spread (Sec. II-A says only that the rate depends on how the states are initialised):
// occurrence i of a symbol of frequency f sits at (2i + 1) / (2f); all occurrences of all symbols are sorted by that
// fraction, ties going to the smaller symbol, and an occurrence's rank is its state.
//
// The rank is found by a counting sort with a key per occurrence, floor(L^2 (2i + 1) / (2f)) with the symbol below it: equal
// fractions have equal first parts, and different ones, of frequencies f + g <= L, are at least 1 / 2fg >= 2 / L^2 apart, so
// their first parts differ.  The key's upper log2 L bits are a bucket; a prefix sum over the buckets' sizes, and then every
// occurrence counts the smaller keys among its bucket's, four to an LDS read: a key of a bucket before or behind is smaller
// or larger by itself, so the reads need neither begin nor end where the bucket does.
// What bounds it is instructions (a workgroup's wavefronts share the four SIMDs): a quotient takes eight with a reciprocal
// that is a little too small, a comparison two, and wavefronts whose 64 occurrences are one symbol's search for nothing.
// A call that builds one table of 2^12 states (several workgroups) with the divisions and the members' products, or second
// divisions where buckets were large, that stood here before -> now: 16 symbols around a dominant one 12.5 -> 7.8 us (with the
// shorter chains of the look-ahead entries, which are a third of it), 16 symbols alike 16.3 -> 10.2, 64 alike 28.6 -> 20, 256
// alike 60 -> 37, 256 of random frequencies 40 -> 22; in the packer (a workgroup of 512 threads, two per CU) 11.2 -> 7.5 us.
#ifndef ANSZP_SPREAD_H
#define ANSZP_SPREAD_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "anszp.h"

constexpr uint32_t kSpreadStates = 1u << ANSZP_MAX_TABLE_LOG;

typedef __attribute__((ext_vector_type(4))) uint32_t spread_words4;
struct SpreadLds {
    uint32_t f[ANSZP_ALPHABET];
    // occurrences of smaller symbols: occurrence i of symbol s is number first[s] + i
    __attribute__((aligned(16))) uint32_t first[ANSZP_ALPHABET];
    spread_words4 member[kSpreadStates / 4u];       // keys, bucket after bucket
    uint32_t bucket[kSpreadStates];        // members of each bucket, then where each bucket's members start
    uint32_t part[16];                     // a wavefront's share of a prefix sum
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
    typedef spread_words4 words4;
    uint32_t* const members = reinterpret_cast<uint32_t*>(t.member);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t L = 1u << table_log;
    uint32_t fs = 0, upto = 0;
    if (tid < ANSZP_ALPHABET) {
        fs = freqs[tid];
        upto = spread_wave_sum(min(fs, L + 1u));               // (a frequency beyond L cannot wrap the sum around)
        if (lane == 63u) t.part[wave] = upto;
    }
    for (uint32_t b = tid; b < L; b += THREADS) t.bucket[b] = 0u;
    if (tid >= L && tid < 4u) members[tid] = 0xFFFFFFFFu;      // (read with the others when L < 4)
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
    }
    __syncthreads();
    // symbols whose first occurrence is not beyond g (g alike for all lanes)
    const words4 firsts = reinterpret_cast<const words4*>(t.first)[lane];
    auto symbols_upto = [&](uint32_t g) {
        return static_cast<uint32_t>(__popcll(__ballot(firsts.x <= g)) + __popcll(__ballot(firsts.y <= g)) +
                                     __popcll(__ballot(firsts.z <= g)) + __popcll(__ballot(firsts.w <= g)));
    };
    uint32_t sy[kPerThread], number[kPerThread], key[kPerThread], at[kPerThread];   // number: f - 1 | i << 12; at: place within the bucket
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) {
        const uint32_t g0 = wave * 64u + u * THREADS, g = g0 + lane;
        if (g0 >= L) break;                                    // (uniform)
        // the largest symbol with first[symbol] <= g (it has a frequency)
        uint32_t s = symbols_upto(g0) - 1u;
        const uint32_t most = symbols_upto(g0 + 63u) - 1u;
        if (s != most) {                                       // (uniform)
            for (uint32_t step = 0x80000000u >> __builtin_clz(most - s); step; step >>= 1) {
                const uint32_t c = min(s + step, most);
                s = t.first[c] <= g ? c : s;
            }
        }
        if (g >= L) break;                                     // (L < 64: one round)
        const uint32_t f = t.f[s], i = g - t.first[s];
        // n / 2f for n < 2^26, n / 2f < 2^12 (i < f): the quotient with the reciprocal, whose and whose product's errors of
        // less than 2^-22 are made to lie on one side, is right or one too small
        const float inverse = __builtin_amdgcn_rcpf(static_cast<float>(2u * f)) * (1.0f - 0x1p-20f);
        auto divide = [&](uint32_t n, uint32_t& rest) {
            const uint32_t q = static_cast<uint32_t>(static_cast<float>(n) * inverse);
            rest = n - __umul24(q, 2u * f);
            const bool more = rest >= 2u * f;
            rest = more ? rest - 2u * f : rest;
            return more ? q + 1u : q;
        };
        uint32_t rest;
        const uint32_t b = divide((2u * i + 1u) << table_log, rest);
        const uint32_t low = divide(rest << table_log, rest);
        sy[u] = s;
        number[u] = (f - 1u) | i << 12;
        key[u] = (b << table_log | low) << 8 | s;
        at[u] = atomicAdd(&t.bucket[b], 1u);
    }
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
    uint32_t starts[kPerThread];
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) {
        if (tid + u * THREADS < L) {
            starts[u] = t.bucket[key[u] >> (table_log + 8u)];
            members[starts[u] + at[u]] = key[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kPerThread; ++u) {
        const uint32_t g = tid + u * THREADS;
        if (g < L) {
            const uint32_t b = key[u] >> (table_log + 8u), end = b + 1u < L ? t.bucket[b + 1u] : L;
            const uint32_t first = starts[u] / 4u, behind = (end + 3u) / 4u;
            uint32_t state = 4u * first;
            auto count = [&](const words4 k) {
                state += (k.x < key[u] ? 1u : 0u) + (k.y < key[u] ? 1u : 0u) + (k.z < key[u] ? 1u : 0u) + (k.w < key[u] ? 1u : 0u);
            };
            count(t.member[first]);
            uint32_t left = behind - first - 1u;
            if (left) {
                // the bucket's other reads, from another one in every lane: where symbols share a frequency a wavefront's
                // buckets are of one size, and reads in one place of each would share an LDS bank
                uint32_t at = first + 1u + ((lane * 37u & 63u) * left >> 6);
#pragma unroll 1
                do {
                    const words4 k = t.member[at];
                    at = at + 1u < behind ? at + 1u : first + 1u;
                    count(k);
                } while (--left);
            }
            place(g, sy[u], (number[u] & 0xFFFu) + 1u, number[u] >> 12, state);
        }
    }
    return true;
}

#endif
