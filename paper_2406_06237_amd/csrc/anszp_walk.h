// Walking look-ahead entries through LDS, a stream per lane (internal to the library; included by the decode kernels'
// source, whose names it uses).
#ifndef ANSZP_WALK_H
#define ANSZP_WALK_H

// Two look-ahead entries as they come (anszp_layout.h) -> as walk_entries reads them from an LDS table at `table_at`.
__device__ __forceinline__ uint4 walk_entry_pair(const uint4& e, uint32_t table_at) {
    auto low = [](uint32_t w) {
        const uint32_t T = (w >> 24) & 15u, symbols = ((w >> 28) & 7u) + 1u;
        return (31u - T) | T << 8 | (w & 0xFF0000u) | symbols << 24;
    };
    return make_uint4(low(e.x), e.y + table_at, low(e.z), e.w + table_at);
}

// Look-ups of every lane from the entry at LDS address `at` with the stream at bit `q` on.  Entries as staged by
// walk_entry_pair: low word 31 - T | T << 8 | symbol << 16 | c << 24, high word the address of entry number `base`; T + 1 bits
// choose the next entry, c symbols are counted.  q is 31 more than the LDS bit address of the next bit (words first bit
// on top: then ~q is what v_alignbit shifts two words by to bring it to the top).  A lane stops before the first look-up
// at which q >= q_end (when it writes: n >= n_end) holds; every four look-ups the other bound is looked at too.  kWalkWrite: n is an
// address in LDS, and the entry's last symbol goes to n after c has been added to it; kWalkSpread: after c times `step`.
// Bound by one LDS round trip per look-up where a SIMD has one wavefront (two words serve two look-ups, and what does
// not stand between an entry's arrival and the next read is issued while that is under way: 8.5 vector instructions per
// look-up in all), by those instructions with four.  As the compiler had it, 20 instructions with the loads at the loop's
// head, a look-up took twice as long.
// ALONE: for a wavefront that has its SIMD to itself, or nearly.  There the words stand between the second look-up of a window and
// the next (they are asked for where that look-up's bits are known): 50 ns a look-up.  A window of two registers lasts for four,
// and the next one is asked for a look-up early and shifted by what that one reads: 45 ns, for one instruction and a half more a
// look-up, which four wavefronts on a SIMD would feel.
enum { kWalkCount, kWalkWrite, kWalkSpread };
template <int MODE, bool ALONE = false>
__device__ __forceinline__ void walk_entries(uint32_t& at, uint32_t& q, uint32_t& n, uint32_t q_end, uint32_t n_end, uint32_t step = 1u) {
#define ANSZP_WALK_ADD(TO, E, BYTE) "v_add_u32_sdwa " TO ", " TO ", " E " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:" BYTE "\n"
#define ANSZP_WALK_NEXT(ELO, EHI, FB)                                                                  \
        "v_lshrrev_b32 v46, " ELO ", v47\n"                                                             \
        "v_lshl_add_u32 %[at], v46, 3, " EHI "\n"                                                       \
        "ds_read_b64 " FB ", %[at]\n"                                                                   \
        ANSZP_WALK_ADD("%[q]", ELO, "BYTE_1")
#define ANSZP_WALK_WORDS                                                                               \
        "v_lshrrev_b32 v49, 3, %[q]\n"                                                                  \
        "v_and_b32 v49, 0x1ffffffc, v49\n"                                                              \
        "ds_read2_b32 v[44:45], v49 offset1:1\n"                                                        \
        "v_not_b32 v48, %[q]\n"
    // two look-ups from one window; the entry in v[40:41] at the start and the end
#define ANSZP_WALK_TWO(COUNT_A, COUNT_B, EMIT_A, EMIT_B, WAIT, STOP)                                                      \
        "v_alignbit_b32 v47, v44, v45, v48\n"                                                           \
        ANSZP_WALK_NEXT("v40", "v41", "v[42:43]")                                                      \
        COUNT_A                                                                                         \
        EMIT_A                                                                                          \
        "v_lshlrev_b32_sdwa v47, v40, v47 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n" \
        STOP                                                                                            \
        "s_waitcnt lgkmcnt(" WAIT ")\n"                                                                 \
        ANSZP_WALK_NEXT("v42", "v43", "v[40:41]")                                                      \
        ANSZP_WALK_WORDS                                                                               \
        COUNT_B                                                                                         \
        EMIT_B                                                                                          \
        STOP                                                                                            \
        "s_waitcnt lgkmcnt(" WAIT ")\n"
#define ANSZP_WALK_ALL(COUNT_A, COUNT_B, EMIT_A, EMIT_B, WAIT, STOP, BOUND)                                              \
    asm volatile(                                                                                       \
        "s_mov_b64 s[40:41], exec\n"                                                                    \
        "v_cmpx_gt_u32 vcc, %[qe], %[q]\n"                                                              \
        "v_cmpx_gt_u32 vcc, %[ne], %[n]\n"                                                              \
        "s_cbranch_execz 2f\n"                                                                          \
        "ds_read_b64 v[40:41], %[at]\n"                                                                 \
        ANSZP_WALK_WORDS                                                                               \
        "s_waitcnt lgkmcnt(0)\n"                                                                        \
        "1:\n"                                                                                          \
        ANSZP_WALK_TWO(COUNT_A, COUNT_B, EMIT_A, EMIT_B, WAIT, STOP)                                                     \
        ANSZP_WALK_TWO(COUNT_A, COUNT_B, EMIT_A, EMIT_B, WAIT, STOP)                                                     \
        BOUND                                                                                           \
        "s_cbranch_execnz 1b\n"                                                                         \
        "2:\n"                                                                                          \
        "s_mov_b64 exec, s[40:41]\n"                                                                    \
        "s_waitcnt lgkmcnt(0)\n"                                                                        \
        : [at] "+v"(at), [q] "+v"(q), [n] "+v"(n)                                                       \
        : [qe] "v"(q_end), [ne] "v"(n_end), [step] "v"(step)                                                              \
        : "memory", "vcc", "scc", "s40", "s41", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50")
#define ANSZP_WALK_STEPS(E)                                                                              \
        "v_mul_u32_u24_sdwa v50, %[step], " E " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3\n" \
        "v_add_u32 %[n], %[n], v50\n"
    // four look-ups from one window, in v[48:49] (its first bit on top); the entry in v[40:41] at the start and the end
#define ANSZP_WALK_LOOK(WAIT, ELO, EHI, FB)                                                             \
        "s_waitcnt lgkmcnt(" WAIT ")\n"                                                                \
        "v_lshrrev_b32 v47, " ELO ", v49\n"                                                            \
        "v_lshl_add_u32 %[at], v47, 3, " EHI "\n"                                                      \
        "ds_read_b64 " FB ", %[at]\n"                                                                  \
        ANSZP_WALK_ADD("%[q]", ELO, "BYTE_1")
#define ANSZP_WALK_SHIFT(ELO)                                                                           \
        "v_lshrrev_b32 v51, 8, " ELO "\n"                 /* (bits 0..5: T) */                          \
        "v_lshlrev_b64 v[48:49], v51, v[48:49]\n"
#define ANSZP_WALK_WINDOW                                                                               \
        "v_lshrrev_b32 v51, 3, %[q]\n"                                                                 \
        "v_and_b32 v51, 0x1ffffffc, v51\n"                                                             \
        "ds_read2_b32 v[44:45], v51 offset1:1\n"                                                       \
        "ds_read_b32 v46, v51 offset:8\n"                                                              \
        "v_not_b32 v52, %[q]\n"
#define ANSZP_WALK_ALIGN                                                                                \
        "v_alignbit_b32 v49, v44, v45, v52\n"                                                          \
        "v_alignbit_b32 v48, v45, v46, v52\n"
#define ANSZP_WALK_FOUR(COUNT_A, COUNT_B, EMIT_A, EMIT_B, WAIT, WAIT_4, WAIT_WORDS, STOP, BOUND)        \
    asm volatile(                                                                                       \
        "s_mov_b64 s[40:41], exec\n"                                                                   \
        "v_cmpx_gt_u32 vcc, %[qe], %[q]\n"                                                             \
        "v_cmpx_gt_u32 vcc, %[ne], %[n]\n"                                                             \
        "s_cbranch_execz 2f\n"                                                                         \
        "ds_read_b64 v[40:41], %[at]\n"                                                                \
        ANSZP_WALK_WINDOW                                                                               \
        "s_waitcnt lgkmcnt(0)\n"                                                                       \
        ANSZP_WALK_ALIGN                                                                                \
        "1:\n"                                                                                         \
        ANSZP_WALK_LOOK(WAIT, "v40", "v41", "v[42:43]")                                                 \
        ANSZP_WALK_SHIFT("v40") COUNT_A EMIT_A STOP                                                     \
        ANSZP_WALK_LOOK(WAIT, "v42", "v43", "v[40:41]")                                                 \
        ANSZP_WALK_SHIFT("v42") COUNT_B EMIT_B STOP                                                     \
        ANSZP_WALK_LOOK(WAIT, "v40", "v41", "v[42:43]")                                                 \
        ANSZP_WALK_SHIFT("v40")                                                                         \
        ANSZP_WALK_WINDOW                                  /* of the next four, as it is before this window's last */ \
        COUNT_A EMIT_A STOP                                                                             \
        ANSZP_WALK_LOOK(WAIT_4, "v42", "v43", "v[40:41]")                                               \
        "s_waitcnt lgkmcnt(" WAIT_WORDS ")\n"                                                          \
        ANSZP_WALK_ALIGN                                                                                \
        ANSZP_WALK_SHIFT("v42") COUNT_B EMIT_B STOP                                                     \
        BOUND                                                                                           \
        "s_cbranch_execnz 1b\n"                                                                        \
        "2:\n"                                                                                         \
        "s_mov_b64 exec, s[40:41]\n"                                                                   \
        "s_waitcnt lgkmcnt(0)\n"                                                                       \
        : [at] "+v"(at), [q] "+v"(q), [n] "+v"(n)                                                       \
        : [qe] "v"(q_end), [ne] "v"(n_end), [step] "v"(step)                                            \
        : "memory", "vcc", "scc", "s40", "s41", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51", "v52")
    static_assert(ANSZP_MAX_TABLE_LOG <= 12, "a window of 64 bits, shifted by up to 12, holds four look-ups: 3 * 12 + 13 bits");
    // (a write follows the entry's read and the words' read: with one access more in flight they have arrived)
    if constexpr (ALONE && MODE == kWalkCount)
        ANSZP_WALK_FOUR(ANSZP_WALK_ADD("%[n]", "v40", "BYTE_3"), ANSZP_WALK_ADD("%[n]", "v42", "BYTE_3"), "", "", "0", "2", "1",
                        "v_cmpx_gt_u32 vcc, %[qe], %[q]\n", "v_cmpx_gt_u32 vcc, %[ne], %[n]\n");
    else if constexpr (ALONE && MODE == kWalkWrite)
        ANSZP_WALK_FOUR(ANSZP_WALK_ADD("%[n]", "v40", "BYTE_3"), ANSZP_WALK_ADD("%[n]", "v42", "BYTE_3"),
                        "ds_write_b8_d16_hi %[n], v40\n", "ds_write_b8_d16_hi %[n], v42\n", "1", "3", "2",
                        "v_cmpx_gt_u32 vcc, %[ne], %[n]\n", "v_cmpx_gt_u32 vcc, %[qe], %[q]\n");
    else if constexpr (ALONE)
        ANSZP_WALK_FOUR(ANSZP_WALK_STEPS("v40"), ANSZP_WALK_STEPS("v42"),
                        "ds_write_b8_d16_hi %[n], v40\n", "ds_write_b8_d16_hi %[n], v42\n", "1", "3", "2",
                        "v_cmpx_gt_u32 vcc, %[ne], %[n]\n", "v_cmpx_gt_u32 vcc, %[qe], %[q]\n");
    else if constexpr (MODE == kWalkCount)
        ANSZP_WALK_ALL(ANSZP_WALK_ADD("%[n]", "v40", "BYTE_3"), ANSZP_WALK_ADD("%[n]", "v42", "BYTE_3"), "", "", "0",
                       "v_cmpx_gt_u32 vcc, %[qe], %[q]\n", "v_cmpx_gt_u32 vcc, %[ne], %[n]\n");
    else if constexpr (MODE == kWalkWrite)
        ANSZP_WALK_ALL(ANSZP_WALK_ADD("%[n]", "v40", "BYTE_3"), ANSZP_WALK_ADD("%[n]", "v42", "BYTE_3"),
                       "ds_write_b8_d16_hi %[n], v40\n", "ds_write_b8_d16_hi %[n], v42\n", "1",
                       "v_cmpx_gt_u32 vcc, %[ne], %[n]\n", "v_cmpx_gt_u32 vcc, %[qe], %[q]\n");
    else
        ANSZP_WALK_ALL(ANSZP_WALK_STEPS("v40"), ANSZP_WALK_STEPS("v42"),
                       "ds_write_b8_d16_hi %[n], v40\n", "ds_write_b8_d16_hi %[n], v42\n", "1",
                       "v_cmpx_gt_u32 vcc, %[ne], %[n]\n", "v_cmpx_gt_u32 vcc, %[qe], %[q]\n");
#undef ANSZP_WALK_FOUR
#undef ANSZP_WALK_ALIGN
#undef ANSZP_WALK_WINDOW
#undef ANSZP_WALK_SHIFT
#undef ANSZP_WALK_LOOK
#undef ANSZP_WALK_STEPS
#undef ANSZP_WALK_ALL
#undef ANSZP_WALK_TWO
#undef ANSZP_WALK_WORDS
#undef ANSZP_WALK_NEXT
#undef ANSZP_WALK_ADD
}

#endif
