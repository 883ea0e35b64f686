// split_stack.h -- the per-lane split recursion over a pruned stack of
// predecessors in registers (device code shared by the evaluation kernels;
// not part of the public ABI).
//
// Recursion and potential form as in split_dp.h: position j takes
//   m_j = min over admissible p < j of f_p,   f_j = m_j + c_j,
// and a predecessor p is admissible while L_p + Q >= L_j.  Thresholds grow
// with p, so once a newer predecessor has a potential no larger than an
// older one's, the older one can never be the minimum again.  The register
// ring of split_dp.h keeps and scans every position of the window; here a
// new potential first removes, from the top of the stack, every older entry
// that it dominates ON ALL LANES of the wave, and then takes that slot.
// Every lane's minimum is unchanged (each lane still has an entry that
// stands for each removed one, at least as cheap and admissible at least as
// long), and the wave scans only the entries some lane may still need:
// travel costs are common to the lanes, so they agree on most removals.  On
// random tours (n = 200, Q = 150) the 11.7 + 6.0 window cells (admitted by
// every lane + by some) become 4.1 + 1.4 entries, and windows of a hundred
// positions hold ten.  A tour in which little is dominated keeps most of its
// window; such tours go to the window scan (TourRec::smooth).
//
// The slot of the next entry is wave-uniform and lives in the program
// counter: the code is unrolled over the R slots, block u handles a position
// whose newest entry sits in slot u - 1, and a removal continues in the block
// of a lower slot.  A position therefore costs no copies and no indexing.
// The whole recursion is one asm block, so its blocks can jump to each other:
//   .Lw_u  the usual position, without a write of EXEC: cells 1 and 2 (newest
//          first) folded as they are, 3-6 through a compare and a select
//          each, one branch to .Lc_u if some lane rejects cell 2, some lane
//          admits cell 7 or the tour ends; then f_j into slot u, the compare
//          that decides on removals, the push (threshold, the load of the
//          next position, the demand and the table entry after it requested
//          a position ahead), and the branch to .Lp_u;
//   .Lp_u, .Lq_u, .Lr_u  one, two, three removals (a fourth can wait for the
//          next position: keeping a removable entry is exact);
//   .Lc_u  cells 1 and 2 selected too; from cell 7 on under EXEC narrowed by
//          v_cmpx, or in groups of four while every lane admits them.
// Slots above the top keep entries that were removed.  A scan meets them only
// past the oldest live entry, where they change nothing (a live entry is at
// least as cheap and admissible wherever they are).  The scan covers live
// entries without a gap, so a live entry about to be overwritten is one that
// some lane admits at cell R: that sets ov, ends the recursion, and the
// caller recomputes the tile.  Every memory operation is waited for inside
// the block.
//
// What bounds it: at one wave per SIMD the number of instructions (a wave
// issues one about every six cycles: 120 ns a position); with three or more
// waves its 23 VALU instructions per position (the ring: 32), most of them
// compares, selects and minima, which take four cycles where adds take two.
// Selecting cells 3-6 under EXEC instead takes two instructions less and
// measured slower (n = 200, S = 1e6: 190 against 184 us), as did marking
// vacated slots (195 us) and a first version with a check for every head
// group (211 us).  The ring scan took 244 us.  n = N = 1000, S = 2e4,
// Q = 300: 230 -> 164 us; 256 tours of 50..400, S = 1e4: 479 -> 370 us;
// n = 300, S = 2e4, windows of a hundred positions: 52 ms (exact fallback)
// -> 79 us.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "split_device.h"

namespace splitk {

// The evaluation variants (ring, kStackFirst, 4, 3) select this recursion.
template <int F> constexpr bool stack_variant() { return F == kStackFirst; }

// Physical registers of the block: v32.. (R potentials, then R thresholds),
// the rest of the vector registers are operands.
//   s[74:75] output row (value table)       s77 b_j (value table)
//   s78 byte selector of a streamed dword   s79 table offset past the tour
//   s[72:73] low half -1 at position n, else 0 (a pair: a write of vcc_lo
//            alone leaves VCCZ, which the branch reads, as it was)
//   s[80:81] active lanes                   s83 table offset
//   s[88:89] table entry of j + 2
//   s90, s91 c_j, c_{j+1}                   s[92:93] address (streamed)
//   s[84:87], s[94:99] lane masks (a VALU instruction reads a mask that
//            another wrote no sooner than the third after it)

#define SPLIT_STACK_CELL(D)                                                                      \
    "v_cmpx_le_i32_e32 vcc, %[L], v[.LQ%=+((\\u-" #D ")&.LM%=)]\n"
#define SPLIT_STACK_MIN(D)                                                                       \
    "v_min_i32_e32 %[m], %[m], v[.LF%=+((\\u-" #D ")&.LM%=)]\n"
// s[84:85] = lanes that reject one of the cells D..G (each is looked at: past
// the oldest live entry a removed, newer one can follow an expired one)
#define SPLIT_STACK_CHECK4(D, E, F, G)                                                           \
    "v_min3_i32 %[va], v[.LQ%=+((\\u-" #D ")&.LM%=)], v[.LQ%=+((\\u-" #E ")&.LM%=)], "           \
    "v[.LQ%=+((\\u-" #F ")&.LM%=)]\n"                                                            \
    "v_min_i32_e32 %[va], %[va], v[.LQ%=+((\\u-" #G ")&.LM%=)]\n"                                \
    "v_cmp_gt_i32_e64 s[84:85], %[L], %[va]\n"
#define SPLIT_STACK_FOLD2(D, E)                                                                  \
    "v_min3_i32 %[m], %[m], v[.LF%=+((\\u-" #D ")&.LM%=)], v[.LF%=+((\\u-" #E ")&.LM%=)]\n"
// cells D..G = D + 3, entered at .Lt<D> with every cell before D admitted
#define SPLIT_STACK_TAIL4(D, E, F, G)                                                            \
    ".Lt" #D "_%=_\\u:\n" SPLIT_STACK_CELL(D) SPLIT_STACK_MIN(D) SPLIT_STACK_CELL(E)             \
    "s_cbranch_execz .Le_%=_\\u\n" SPLIT_STACK_MIN(E) SPLIT_STACK_CELL(F) SPLIT_STACK_MIN(F)     \
    SPLIT_STACK_CELL(G) "s_cbranch_execz .Le_%=_\\u\n" SPLIT_STACK_MIN(G)
// cells D..D+3 admitted by every lane; the next group is checked meanwhile
#define SPLIT_STACK_HEAD4(D, E, F, G, H, I, J, K)                                                \
    SPLIT_STACK_CHECK4(H, I, J, K) SPLIT_STACK_FOLD2(D, E) SPLIT_STACK_FOLD2(F, G)               \
    "s_cmp_lg_u64 s[84:85], 0\n"                                                                 \
    "s_cbranch_scc1 .Lt" #H "_%=_\\u\n"

#define SPLIT_STACK_HEADS_32                                                                     \
    SPLIT_STACK_HEAD4(8, 9, 10, 11, 12, 13, 14, 15)                                              \
    SPLIT_STACK_HEAD4(12, 13, 14, 15, 16, 17, 18, 19)                                            \
    SPLIT_STACK_FOLD2(16, 17) SPLIT_STACK_FOLD2(18, 19) "s_branch .Lt20_%=_\\u\n"
#define SPLIT_STACK_TAILS_32                                                                     \
    SPLIT_STACK_TAIL4(8, 9, 10, 11)                                                              \
    SPLIT_STACK_TAIL4(12, 13, 14, 15)                                                            \
    SPLIT_STACK_TAIL4(16, 17, 18, 19)                                                            \
    SPLIT_STACK_TAIL4(20, 21, 22, 23)                                                            \
    SPLIT_STACK_TAIL4(24, 25, 26, 27)                                                            \
    SPLIT_STACK_TAIL4(28, 29, 30, 31)                                                            \
    SPLIT_STACK_CELL(32) "s_cbranch_execz .Le_%=_\\u\n"

#define SPLIT_STACK_HEADS_64                                                                     \
    SPLIT_STACK_HEAD4(8, 9, 10, 11, 12, 13, 14, 15)                                              \
    SPLIT_STACK_HEAD4(12, 13, 14, 15, 16, 17, 18, 19)                                            \
    SPLIT_STACK_HEAD4(16, 17, 18, 19, 20, 21, 22, 23)                                            \
    SPLIT_STACK_HEAD4(20, 21, 22, 23, 24, 25, 26, 27)                                            \
    SPLIT_STACK_HEAD4(24, 25, 26, 27, 28, 29, 30, 31)                                            \
    SPLIT_STACK_HEAD4(28, 29, 30, 31, 32, 33, 34, 35)                                            \
    SPLIT_STACK_HEAD4(32, 33, 34, 35, 36, 37, 38, 39)                                            \
    SPLIT_STACK_FOLD2(36, 37) SPLIT_STACK_FOLD2(38, 39) "s_branch .Lt40_%=_\\u\n"
#define SPLIT_STACK_TAILS_64                                                                     \
    SPLIT_STACK_TAIL4(8, 9, 10, 11)                                                              \
    SPLIT_STACK_TAIL4(12, 13, 14, 15)                                                            \
    SPLIT_STACK_TAIL4(16, 17, 18, 19)                                                            \
    SPLIT_STACK_TAIL4(20, 21, 22, 23)                                                            \
    SPLIT_STACK_TAIL4(24, 25, 26, 27)                                                            \
    SPLIT_STACK_TAIL4(28, 29, 30, 31)                                                            \
    SPLIT_STACK_TAIL4(32, 33, 34, 35)                                                            \
    SPLIT_STACK_TAIL4(36, 37, 38, 39)                                                            \
    SPLIT_STACK_TAIL4(40, 41, 42, 43)                                                            \
    SPLIT_STACK_TAIL4(44, 45, 46, 47)                                                            \
    SPLIT_STACK_TAIL4(48, 49, 50, 51)                                                            \
    SPLIT_STACK_TAIL4(52, 53, 54, 55)                                                            \
    SPLIT_STACK_TAIL4(56, 57, 58, 59)                                                            \
    SPLIT_STACK_TAIL4(60, 61, 62, 63)                                                            \
    SPLIT_STACK_CELL(64) "s_cbranch_execz .Le_%=_\\u\n"

// ---- demand sources: START reads positions 1 and 2, STEP (at the push of
// position j) folds the demand of j + 1 into L and requests that of j + 2
#define SPLIT_STACK_START_LDS                                                                    \
    "v_add_u32_e32 %[va], s84, %[row]\n"                                                         \
    "ds_read_u8 %[L], %[va]\n"                                                                   \
    "v_add_u32_e32 %[va], s86, %[row]\n"                                                         \
    "ds_read_u8 %[vq], %[va]\n"                                                                  \
    "s_mov_b32 s90, s85\n"                                                                       \
    "s_mov_b32 s91, s87\n"                                                                       \
    "s_waitcnt lgkmcnt(0)\n"
#define SPLIT_STACK_STEP_LDS                                                                     \
    "s_waitcnt lgkmcnt(0)\n"                                                                     \
    "v_add_u32_e32 %[L], %[L], %[vq]\n"                                                          \
    "v_add_u32_e32 %[va], s88, %[row]\n"                                                         \
    "ds_read_u8 %[vq], %[va]\n"
#define SPLIT_STACK_START_LDS16                                                                  \
    "v_lshl_add_u32 %[va], s84, 1, %[row]\n"                                                     \
    "ds_read_i16 %[L], %[va]\n"                                                                  \
    "v_lshl_add_u32 %[va], s86, 1, %[row]\n"                                                     \
    "ds_read_i16 %[vq], %[va]\n"                                                                 \
    "s_mov_b32 s90, s85\n"                                                                       \
    "s_mov_b32 s91, s87\n"                                                                       \
    "s_waitcnt lgkmcnt(0)\n"
#define SPLIT_STACK_STEP_LDS16                                                                   \
    "s_waitcnt lgkmcnt(0)\n"                                                                     \
    "v_add_u32_e32 %[L], %[L], %[vq]\n"                                                          \
    "v_lshl_add_u32 %[va], s88, 1, %[row]\n"                                                     \
    "ds_read_i16 %[vq], %[va]\n"
#define SPLIT_STACK_COLD_LDS16                                                                   \
    ""
#define SPLIT_STACK_START_STREAM                                                                 \
    "s_mov_b32 s92, %[base]\n"                                                                   \
    "s_mov_b32 s93, %[baseh]\n"                                                                  \
    "global_load_dword %[vq], %[row], s[92:93]\n"                                                \
    "global_load_dword %[vn], %[row], s[92:93] offset:256\n"                                     \
    "s_add_u32 s92, s92, 0x200\n"                                                                \
    "s_addc_u32 s93, s93, 0\n"                                                                   \
    "s_movk_i32 s78, 0x100\n"                                                                    \
    "s_mov_b32 s90, s85\n"                                                                       \
    "s_mov_b32 s91, s87\n"                                                                       \
    "s_waitcnt vmcnt(0)\n"                                                                       \
    "v_and_b32_e32 %[L], 0xff, %[vq]\n"
#define SPLIT_STACK_STEP_STREAM                                                                  \
    "s_waitcnt lgkmcnt(0)\n"                                                                     \
    "v_dot4_u32_u8 %[L], %[vq], s78, %[L]\n"                                                     \
    "s_lshl_b32 s78, s78, 8\n"                                                                   \
    "s_cbranch_scc0 .Lf_%=_\\u\n"                                                                \
    ".Lg_%=_\\u:\n"
#define SPLIT_STACK_COLD_LDS                                                                     \
    ""
#define SPLIT_STACK_COLD_STREAM                                                                  \
    ".Lf_%=_\\u:\n"                                                                              \
    "s_waitcnt vmcnt(0)\n"                                                                       \
    "v_mov_b32_e32 %[vq], %[vn]\n"                                                               \
    "global_load_dword %[vn], %[row], s[92:93]\n"                                                \
    "s_add_u32 s92, s92, 0x100\n"                                                                \
    "s_addc_u32 s93, s93, 0\n"                                                                   \
    "s_mov_b32 s78, 1\n"                                                                         \
    "s_branch .Lg_%=_\\u\n"

// ---- outputs besides m_n: BEGIN before the first position, PUT where m_j is
// final (not at position n), NEXT at the push
#define SPLIT_STACK_BEGIN_NONE ""
#define SPLIT_STACK_PUT_NONE ""
#define SPLIT_STACK_NEXT_NONE ""
// V(j) = m_j + b_j to the lane's column, one row of the table per position
#define SPLIT_STACK_BEGIN_VALUES                                                                 \
    "s_mov_b32 s74, %[out]\n"                                                                    \
    "s_mov_b32 s75, %[outh]\n"                                                                   \
    "s_load_dword s77, %[ab], 0x18\n"
#define SPLIT_STACK_PUT_VALUES                                                                   \
    "s_waitcnt lgkmcnt(0)\n"                                                                     \
    "v_add_u32_e32 %[ta], s77, %[m]\n"                                                           \
    "global_store_dword %[col], %[ta], s[74:75] nt\n"                                            \
    "s_add_u32 s74, s74, %[step]\n"                                                              \
    "s_addc_u32 s75, s75, %[steph]\n"
#define SPLIT_STACK_NEXT_VALUES                                                                  \
    "s_load_dword s77, %[ab], s83\n"

// The compiler counts the lines of an asm text to place its own branches; the
// macros hide most of this one's, so the size of the code (at most this many
// bytes) stands in a directive that it counts and the assembler skips.
#define SPLIT_STACK_BYTES_32 "32768"
#define SPLIT_STACK_BYTES_64 "106496"

// macro NAME for every slot u: the slot, and the two below it
#define SPLIT_STACK_SLOTS(R, NAME)                                                               \
    ".altmacro\n"                                                                                \
    ".set .LI%=, 0\n"                                                                            \
    ".rept " #R "\n" NAME "%= %%(.LI%=), %%((.LI%=-1)&.LM%=), %%((.LI%=-2)&.LM%=)\n"              \
    ".set .LI%=, .LI%=+1\n"                                                                      \
    ".endr\n"                                                                                    \
    ".noaltmacro\n"

#define SPLIT_STACK_ASM(R, START, STEP, COLD, BEGIN, PUT, NEXT)                                  \
    ".if 0\n"                                                                                    \
    ".space " SPLIT_STACK_BYTES_##R "\n"                                                         \
    ".endif\n"                                                                                   \
    ".set .LF%=, 32\n"                                                                           \
    ".set .LQ%=, 32+" #R "\n"                                                                    \
    ".set .LM%=, " #R "-1\n"                                                                     \
    ".macro hot%= u, p, o\n"                                                                     \
    ".Lw_%=_\\u:\n"                                                                              \
    "v_cmp_le_i32_e32 vcc, %[L], v[.LQ%=+((\\u-7)&.LM%=)]\n"                                     \
    "v_cmp_gt_i32_e64 s[84:85], %[L], v[.LQ%=+\\o]\n"                                            \
    "v_cmp_le_i32_e64 s[86:87], %[L], v[.LQ%=+((\\u-3)&.LM%=)]\n"                                \
    "v_cmp_le_i32_e64 s[94:95], %[L], v[.LQ%=+((\\u-4)&.LM%=)]\n"                                \
    "v_cmp_le_i32_e64 s[96:97], %[L], v[.LQ%=+((\\u-5)&.LM%=)]\n"                                \
    "v_cmp_le_i32_e64 s[98:99], %[L], v[.LQ%=+((\\u-6)&.LM%=)]\n"                                \
    "v_min_i32_e32 %[m], v[.LF%=+\\p], v[.LF%=+\\o]\n"                                           \
    "s_or_b64 vcc, vcc, s[84:85]\n"                                                              \
    "v_cndmask_b32_e64 %[va], 2.0, v[.LF%=+((\\u-3)&.LM%=)], s[86:87]\n"                         \
    "v_cndmask_b32_e64 %[ta], 2.0, v[.LF%=+((\\u-4)&.LM%=)], s[94:95]\n"                         \
    "s_or_b64 vcc, vcc, s[72:73]\n"                                                              \
    "v_cndmask_b32_e64 %[tb], 2.0, v[.LF%=+((\\u-5)&.LM%=)], s[96:97]\n"                         \
    "v_cndmask_b32_e64 %[tc], 2.0, v[.LF%=+((\\u-6)&.LM%=)], s[98:99]\n"                         \
    "v_min3_i32 %[m], %[m], %[va], %[ta]\n"                                                      \
    "v_min3_i32 %[m], %[m], %[tb], %[tc]\n"                                                      \
    "s_cbranch_vccnz .Lc_%=_\\u\n"                                                               \
    ".Ld_%=_\\u:\n"                                                                              \
    PUT                                                                                         \
    "v_add_u32_e32 v[.LF%=+\\u], s90, %[m]\n"                                                    \
    "v_cmp_gt_i32_e32 vcc, v[.LF%=+\\u], v[.LF%=+\\p]\n"                                         \
    "v_add_u32_e32 v[.LQ%=+\\u], %[vQ], %[L]\n"                                                  \
    STEP                                                                                         \
    "s_mov_b32 s90, s91\n"                                                                       \
    "s_mov_b32 s91, s89\n"                                                                       \
    "s_load_dwordx2 s[88:89], %[tab], s83\n"                                                     \
    NEXT                                                                                        \
    "s_add_u32 s83, s83, 8\n"                                                                    \
    "s_sub_u32 s72, s79, s83\n"                                                                  \
    "s_ashr_i32 s72, s72, 31\n"                                                                  \
    "s_cbranch_vccz .Lp_%=_\\u\n"                                                                \
    ".endm\n"                                                                                    \
    ".macro pop%= u, p, o\n"                                                                     \
    ".Lp_%=_\\u:\n"                                                                              \
    "v_cmp_gt_i32_e32 vcc, v[.LF%=+\\u], v[.LF%=+\\o]\n"                                         \
    "s_cbranch_vccz .Lq_%=_\\u\n"                                                                \
    "v_mov_b32_e32 v[.LF%=+\\p], v[.LF%=+\\u]\n"                                                 \
    "v_mov_b32_e32 v[.LQ%=+\\p], v[.LQ%=+\\u]\n"                                                 \
    "s_branch .Lw_%=_\\u\n"                                                                      \
    ".Lq_%=_\\u:\n"                                                                              \
    "v_cmp_gt_i32_e32 vcc, v[.LF%=+\\u], v[.LF%=+((\\u-3)&.LM%=)]\n"                             \
    "s_cbranch_vccz .Lr_%=_\\u\n"                                                                \
    "v_mov_b32_e32 v[.LF%=+\\o], v[.LF%=+\\u]\n"                                                 \
    "v_mov_b32_e32 v[.LQ%=+\\o], v[.LQ%=+\\u]\n"                                                 \
    "s_branch .Lw_%=_\\p\n"                                                                      \
    ".Lr_%=_\\u:\n"                                                                              \
    "v_mov_b32_e32 v[.LF%=+((\\u-3)&.LM%=)], v[.LF%=+\\u]\n"                                     \
    "v_mov_b32_e32 v[.LQ%=+((\\u-3)&.LM%=)], v[.LQ%=+\\u]\n"                                     \
    "s_branch .Lw_%=_\\o\n"                                                                      \
    ".endm\n"                                                                                    \
    ".macro cold%= u, p, o\n"                                                                    \
    COLD                                                                                         \
    ".Lc_%=_\\u:\n"                                                                              \
    "v_cmp_le_i32_e32 vcc, %[L], v[.LQ%=+((\\u-7)&.LM%=)]\n"                                     \
    "s_cmp_eq_u64 s[84:85], 0\n"                                                                 \
    "s_cbranch_scc1 .Lb_%=_\\u\n"                                                                \
    "v_cmp_le_i32_e64 s[84:85], %[L], v[.LQ%=+\\p]\n"                                            \
    "v_cmp_le_i32_e64 s[86:87], %[L], v[.LQ%=+\\o]\n"                                            \
    "v_min3_i32 %[ta], %[ta], %[tb], %[tc]\n"                                                    \
    "v_min_i32_e32 %[va], %[va], %[ta]\n"                                                        \
    "v_cndmask_b32_e64 %[m], 2.0, v[.LF%=+\\p], s[84:85]\n"                                      \
    "v_cndmask_b32_e64 %[tb], 2.0, v[.LF%=+\\o], s[86:87]\n"                                     \
    "v_min3_i32 %[m], %[m], %[va], %[tb]\n"                                                      \
    ".Lb_%=_\\u:\n"                                                                              \
    "s_cbranch_vccz .Lz_%=_\\u\n"                                                                \
    "s_cmp_eq_u64 vcc, s[80:81]\n"                                                               \
    "s_cbranch_scc1 .Lh_%=_\\u\n"                                                                \
    "s_mov_b64 exec, vcc\n"                                                                      \
    SPLIT_STACK_MIN(7)                                                                           \
    SPLIT_STACK_TAILS_##R                                                                        \
    "v_mov_b32_e32 %[ov], 1\n"                                                                   \
    "s_branch .Lx_%=\n"                                                                          \
    ".Lh_%=_\\u:\n"                                                                              \
    SPLIT_STACK_CHECK4(8, 9, 10, 11)                                                             \
    SPLIT_STACK_MIN(7)                                                                           \
    "s_cmp_lg_u64 s[84:85], 0\n"                                                                 \
    "s_cbranch_scc1 .Lt8_%=_\\u\n"                                                               \
    SPLIT_STACK_HEADS_##R                                                                        \
    ".Le_%=_\\u:\n"                                                                              \
    "s_mov_b64 exec, s[80:81]\n"                                                                 \
    ".Lz_%=_\\u:\n"                                                                              \
    "s_cmp_eq_u32 s72, 0\n"                                                                      \
    "s_cbranch_scc1 .Ld_%=_\\u\n"                                                                \
    "s_branch .Lx_%=\n"                                                                          \
    ".endm\n"                                                                                    \
    "s_mov_b64 s[80:81], exec\n"                                                                 \
    "s_load_dwordx4 s[84:87], %[tab], 0x8\n"                                                     \
    "s_load_dwordx2 s[88:89], %[tab], 0x18\n"                                                    \
    BEGIN                                                                                       \
    "v_mov_b32_e32 %[ov], 0\n"                                                                   \
    ".set .LI%=, 0\n"                                                                            \
    ".rept " #R "\n"                                                                             \
    "v_mov_b32_e32 v[.LF%=+.LI%=], -2.0\n"                                                       \
    "v_mov_b32_e32 v[.LQ%=+.LI%=], -2.0\n"                                                       \
    ".set .LI%=, .LI%=+1\n"                                                                      \
    ".endr\n"                                                                                    \
    "v_mov_b32_e32 v[.LF%=], %[f0]\n"                                                            \
    "v_mov_b32_e32 %[vQ], %[Q]\n"                                                                \
    "v_mov_b32_e32 v[.LQ%=], %[Q]\n"                                                             \
    "s_lshl_b32 s79, %[n], 3\n"                                                                  \
    "s_add_u32 s79, s79, 0x10\n"                                                                 \
    "s_sub_u32 s72, s79, 0x20\n"                                                                 \
    "s_ashr_i32 s72, s72, 31\n"                                                                  \
    "s_mov_b32 s73, 0\n"                                                                         \
    "s_movk_i32 s83, 0x20\n"                                                                     \
    "s_waitcnt lgkmcnt(0)\n"                                                                     \
    START                                                                                        \
    "s_branch .Lw_%=_1\n"                                                                        \
    ".p2align 8\n"                                                                               \
    SPLIT_STACK_SLOTS(R, "hot")                                                                  \
    "s_branch .Lw_%=_0\n"                                                                        \
    SPLIT_STACK_SLOTS(R, "pop")                                                                  \
    SPLIT_STACK_SLOTS(R, "cold")                                                                 \
    ".Lx_%=:\n"                                                                                  \
    "s_mov_b64 exec, s[80:81]\n"                                                                 \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n"                                                            \
    ".purgem hot%=\n.purgem pop%=\n"                                                             \
    ".purgem cold%=\n"

#define SPLIT_STACK_CLOBBER_32                                                                   \
    "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41",                        \
    "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51",                        \
    "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", "v60", "v61",                        \
    "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71",                        \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81",                        \
    "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91",                        \
    "v92", "v93", "v94", "v95"
#define SPLIT_STACK_CLOBBER_64                                                                   \
    "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41",                        \
    "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51",                        \
    "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", "v60", "v61",                        \
    "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71",                        \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81",                        \
    "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91",                        \
    "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v100", "v101",                      \
    "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111",              \
    "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121",              \
    "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131",              \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141",              \
    "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151",              \
    "v152", "v153", "v154", "v155", "v156", "v157", "v158", "v159"

#define SPLIT_STACK_RUN(R, SRC, OUT, ...)                                                             \
    asm volatile(SPLIT_STACK_ASM(R, SPLIT_STACK_START_##SRC, SPLIT_STACK_STEP_##SRC,                \
                                 SPLIT_STACK_COLD_##SRC, SPLIT_STACK_BEGIN_##OUT,                \
                                 SPLIT_STACK_PUT_##OUT, SPLIT_STACK_NEXT_##OUT)                  \
                 : [m] "=&v"(m), [ov] "=&v"(ov), [L] "=&v"(L), [vq] "=&v"(vq), [va] "=&v"(va),   \
                   [ta] "=&v"(ta), [tb] "=&v"(tb), [tc] "=&v"(tc), [vQ] "=&v"(vQ),               \
                   [vn] "=&v"(vn)                                                                \
                 : [row] "v"(row), [tab] "s"(tab), [n] "s"(n), [f0] "s"(f0), [Q] "s"(Q),         \
                   ##__VA_ARGS__                                                                 \
                 : "memory", "vcc", "scc", "s72", "s73", "s74", "s75", "s77", "s78", "s79",      \
                   "s80", "s81", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90",         \
                   "s91", "s92", "s93", "s94", "s95", "s96", "s97", "s98", "s99",                \
                   SPLIT_STACK_CLOBBER_##R)

// m_n of the lane's scenario, its demand bytes in LDS at byte offset `row`,
// indexed by the table's customer; ovf is set when a window held more than R
// entries (m_n is then meaningless).  n >= 1; the table has three entries
// after position n.
template <int R>
__device__ __forceinline__ int stack_lane(uint32_t row, CInt *tab, int n, int f0, int Q, bool &ovf)
{
    int m, ov, L, vq, va, ta, tb, tc, vQ, vn;
    if constexpr (R == 32)
        SPLIT_STACK_RUN(32, LDS, NONE);
    else
        SPLIT_STACK_RUN(64, LDS, NONE);
    ovf = ov != 0;
    return m;
}

// The same with 16-bit demands (not negative) at byte offset `row`.
template <int R>
__device__ __forceinline__ int stack_lane_wide(uint32_t row, CInt *tab, int n, int f0, int Q,
                                               bool &ovf)
{
    int m, ov, L, vq, va, ta, tb, tc, vQ, vn;
    if constexpr (R == 32)
        SPLIT_STACK_RUN(32, LDS16, NONE);
    else
        SPLIT_STACK_RUN(64, LDS16, NONE);
    ovf = ov != 0;
    return m;
}

// Where a run that writes the value table puts it: V(j) of the lane's
// scenario at out + (j - 1) * step + col, from b_j = ab[j - 1].y.
struct StackTable {
    int32_t *out;  // the tile's first column of row 1 (wave-uniform)
    uint64_t step; // bytes between rows
    uint32_t col;  // the lane's byte offset
    const int2 *ab;
};

// stack_lane and stack_lane_wide (WIDE) that also write V(1) .. V(n - 1),
// 2^30 or more where no split exists.
template <int R, bool WIDE>
__device__ __forceinline__ int stack_lane_values(uint32_t row, CInt *tab, int n, int f0, int Q,
                                                 const StackTable &table, bool &ovf)
{
    int m, ov, L, vq, va, ta, tb, tc, vQ, vn;
    const uint32_t out = (uint32_t)(uintptr_t)table.out;
    const uint32_t outh = (uint32_t)((uintptr_t)table.out >> 32);
    const uint32_t step = (uint32_t)table.step, steph = (uint32_t)(table.step >> 32);
    const uint32_t col = table.col;
    // the push of position j reads b_{j+1} at the table offset of j + 3
    const char *ab = reinterpret_cast<const char *>(table.ab) - 20;
#define SPLIT_STACK_TABLE                                                                        \
    [out] "s"(out), [outh] "s"(outh), [step] "s"(step), [steph] "s"(steph), [col] "v"(col),      \
        [ab] "s"(ab)
    if constexpr (R == 32 && WIDE)
        SPLIT_STACK_RUN(32, LDS16, VALUES, SPLIT_STACK_TABLE);
    else if constexpr (R == 32)
        SPLIT_STACK_RUN(32, LDS, VALUES, SPLIT_STACK_TABLE);
    else if constexpr (WIDE)
        SPLIT_STACK_RUN(64, LDS16, VALUES, SPLIT_STACK_TABLE);
    else
        SPLIT_STACK_RUN(64, LDS, VALUES, SPLIT_STACK_TABLE);
#undef SPLIT_STACK_TABLE
    ovf = ov != 0;
    return m;
}

// The same with the tile's demands in tour order in global memory, four
// positions to a dword and the lanes' dwords side by side: byte (j - 1) & 3
// of the dword at base + 256 * ((j - 1) / 4) + row (row = 4 * lane) is
// position j.  Readable up to dword (n - 1) / 4 + 2.
template <int R>
__device__ __forceinline__ int stack_lane_ordered(const uint8_t *base, uint32_t row, CInt *tab,
                                                  int n, int f0, int Q, bool &ovf)
{
    int m, ov, L, vq, va, ta, tb, tc, vQ, vn;
    const uint32_t base_lo = (uint32_t)(uintptr_t)base;
    const uint32_t base_hi = (uint32_t)((uintptr_t)base >> 32);
    if constexpr (R == 32)
        SPLIT_STACK_RUN(32, STREAM, NONE, [base] "s"(base_lo), [baseh] "s"(base_hi));
    else
        SPLIT_STACK_RUN(64, STREAM, NONE, [base] "s"(base_lo), [baseh] "s"(base_hi));
    ovf = ov != 0;
    return m;
}

} // namespace splitk
