// The walk of a plan's records (int4, cover.h): shared by the full evaluations of images
// (k_cover.hip) and of volumes (k_cover3.hip).
//
// Written in assembly: the running product and the two saved ones stay in one set of registers
// each (the compiler copied all R of them wherever a record's branches joined, 16 to 80 moves
// beside a record's 50 useful operations), and the next record's LDS reads are issued as soon as
// the current product is formed, so that they return under its popcounts and wave sum.
//
// (Records read 16 at a time into a vector register, one batch ahead, and taken out with readlane
// were 10 % slower than scalar loads one record ahead.)
//
// A lane has Q rows of P words.
//
//   M  start pixels of the lane's words (what a restore of level 1 gives), from v28 on
//   v24 ..  LDS byte address of each row's first word in array 0
//   slots   LDS byte address of the group's count slots
//
// Registers: from v28 on M, A (product), S1, S2 (saved) of K >= Q P each, D0 (the P + 1 dwords of
// each row for step 0, PD dwords apart in KD, an odd number: register pairs start even), T, D1 (step 1), N.  s72..75 the record, s76..79 the next
// one, s80.. the current record's fields once the next one has moved up; s88, s89: byte offsets of
// the record after it and of the end.  LDS reads are issued only for records of the piece; records
// are read up to two past it.  A wave sum of at most 64 lanes x 512 start pixels; all 64 lanes are
// active throughout.
#pragma once

#define LPF_WALK_TEXT(TWO, ONE, COUNT, ADD)                                                                              \
  ".set cvA, 28 + %[K]\n"                                                                         \
  ".set cvS1, cvA + %[K]\n"                                                                       \
  ".set cvS2, cvS1 + %[K]\n"                                                                      \
  ".set cvD0, cvS2 + %[K]\n"                                                                      \
  ".set cvT, cvD0 + %[KD]\n"                                                                      \
  ".set cvD1, cvT + 1\n"                                                                          \
  ".set cvN, cvD1 + %[KD]\n"                                                                      \
  ".set cvN2, cvN + 1\n"                                                                          \
  "s_lshl_b32 s88, %[r0], 4\n"                                                                    \
  "s_lshl_b32 s89, %[r1], 4\n"                                                                    \
  "Lcv_load%=:\n" /* record at s88 and the one after it, nothing in flight for them yet */        \
  "s_add_u32 s90, s88, 16\n"                                                                      \
  "s_load_dwordx4 s[72:75], %[recs], s88\n"                                                       \
  "s_load_dwordx4 s[76:79], %[recs], s90\n"                                                       \
  "s_waitcnt lgkmcnt(0)\n"                                                                        \
  LPF_WALK_READ("0")                                                                              \
  "s_waitcnt lgkmcnt(0)\n"                                                                        \
  "Lcv_top%=:\n" /* the record's dwords are in D0, D1 */                                          \
  "s_bfe_u32 s84, s72, 0x20016\n"                                                                 \
  "s_cmp_eq_u32 s84, 0\n"                                                                         \
  "s_cbranch_scc1 Lcv_and%=\n"                                                                    \
  "s_cmp_eq_u32 s84, 1\n"                                                                         \
  "s_cbranch_scc0 Lcv_r2%=\n"                                                                     \
  LPF_WALK_MOV("cvA", "28")                                                                       \
  "s_branch Lcv_and%=\n"                                                                          \
  "Lcv_r2%=:\n"                                                                                   \
  "s_cmp_eq_u32 s84, 2\n"                                                                         \
  "s_cbranch_scc0 Lcv_r3%=\n"                                                                     \
  LPF_WALK_MOV("cvA", "cvS1")                                                                     \
  "s_branch Lcv_and%=\n"                                                                          \
  "Lcv_r3%=:\n"                                                                                   \
  LPF_WALK_MOV("cvA", "cvS2")                                                                     \
  "Lcv_and%=:\n"                                                                                  \
  "s_lshr_b32 s85, s72, 16\n" /* a funnel shift takes the low five bits */                        \
  "s_bitcmp1_b32 s72, 21\n"                                                                       \
  "s_cbranch_scc0 Lcv_one%=\n"                                                                    \
  "s_lshr_b32 s86, s73, 16\n"                                                                     \
  TWO                                                                                             \
  "s_branch Lcv_next%=\n"                                                                         \
  "Lcv_one%=:\n"                                                                                  \
  ONE                                                                                             \
  "Lcv_next%=:\n" /* the next record moves up; its reads, and the record after it */              \
  "s_mov_b32 s80, s72\n"                                                                          \
  "s_mov_b64 s[82:83], s[74:75]\n"                                                                \
  "s_add_u32 s88, s88, 16\n"                                                                      \
  "s_cmp_ge_u32 s88, s89\n"                                                                       \
  "s_cbranch_scc1 Lcv_issued%=\n"                                                                 \
  "s_mov_b64 s[72:73], s[76:77]\n"                                                                \
  "s_mov_b64 s[74:75], s[78:79]\n"                                                                \
  "s_add_u32 s90, s88, 16\n"                                                                      \
  "s_load_dwordx4 s[76:79], %[recs], s90\n"                                                       \
  LPF_WALK_READ("1")                                                                              \
  "Lcv_issued%=:\n"                                                                               \
  "s_bfe_u32 s84, s80, 0x20018\n"                                                                 \
  "s_cmp_eq_u32 s84, 0\n"                                                                         \
  "s_cbranch_scc1 Lcv_count%=\n"                                                                  \
  "s_cmp_eq_u32 s84, 1\n"                                                                         \
  "s_cbranch_scc0 Lcv_s2%=\n"                                                                     \
  LPF_WALK_MOV("cvS1", "cvA")                                                                     \
  "s_branch Lcv_count%=\n"                                                                        \
  "Lcv_s2%=:\n"                                                                                   \
  LPF_WALK_MOV("cvS2", "cvA")                                                                     \
  "Lcv_count%=:\n"                                                                                \
  "s_bitcmp1_b32 s80, 26\n"                                                                       \
  "s_cbranch_scc0 Lcv_wait%=\n"                                                                   \
  COUNT                                                                                           \
  "s_lshl_b32 s82, s82, 2\n"                                                                      \
  "s_add_u32 s82, s82, %[slots]\n"                                                                \
  "v_cmp_ne_u32_e32 vcc, 0, v[cvN]\n"                                                             \
  "s_cbranch_vccz Lcv_zero%=\n"                                                                   \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"         \
  "s_nop 1\n"                                                                                     \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"         \
  "s_nop 1\n"                                                                                     \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] row_half_mirror row_mask:0xf bank_mask:0xf\n"             \
  "s_nop 1\n"                                                                                     \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] row_mirror row_mask:0xf bank_mask:0xf\n"                  \
  "s_nop 1\n"                                                                                     \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] row_bcast:15 row_mask:0xa bank_mask:0xf\n"                \
  "s_nop 1\n"                                                                                     \
  "v_add_u32_dpp v[cvN], v[cvN], v[cvN] row_bcast:31 row_mask:0xc bank_mask:0xf\n"                \
  "s_waitcnt lgkmcnt(0)\n" /* the reads, before the add: it need not be waited for */             \
  "v_mov_b32 v[cvT], s82\n"                                                                       \
  "s_brev_b64 exec, 1\n" /* lane 63 holds the sum */                                              \
  ADD                                                                                             \
  "s_mov_b64 exec, -1\n"                                                                          \
  "s_cmp_lt_u32 s88, s89\n"                                                                       \
  "s_cbranch_scc1 Lcv_top%=\n"                                                                    \
  "s_branch Lcv_end%=\n"                                                                          \
  "Lcv_zero%=:\n" /* nothing that extends this path counts here: on at the jump target */         \
  "s_waitcnt lgkmcnt(0)\n"                                                                        \
  "s_lshl_b32 s83, s83, 4\n"                                                                      \
  "s_cmp_eq_u32 s83, s88\n" /* the record already under way */                                    \
  "s_mov_b32 s88, s83\n"                                                                          \
  "s_cbranch_scc1 Lcv_more%=\n"                                                                   \
  "s_cmp_lt_u32 s88, s89\n"                                                                       \
  "s_cbranch_scc1 Lcv_load%=\n"                                                                   \
  "s_branch Lcv_end%=\n"                                                                          \
  "Lcv_wait%=:\n"                                                                                 \
  "s_waitcnt lgkmcnt(0)\n"                                                                        \
  "Lcv_more%=:\n"                                                                                 \
  "s_cmp_lt_u32 s88, s89\n"                                                                       \
  "s_cbranch_scc1 Lcv_top%=\n"                                                                    \
  "Lcv_end%=:\n"                                                                                  \
  "s_waitcnt lgkmcnt(0)\n"
// LDS reads of the record in s72, s73 into D0 and, for two steps, D1 (P + 1 dwords a row).
#define LPF_WALK_READ(id)                                                                         \
  "s_and_b32 s84, s72, 0xffff\n"                                                                  \
  LPF_WALK_READ1("cvD0")                                                                          \
  "s_bitcmp1_b32 s72, 21\n"                                                                       \
  "s_cbranch_scc0 Lcv_read" id "_%=\n"                                                            \
  "s_and_b32 s84, s73, 0xffff\n"                                                                  \
  LPF_WALK_READ1("cvD1")                                                                          \
  "Lcv_read" id "_%=:\n"
#define LPF_WALK_READ1(d)                                                                         \
  ".set cvq, 0\n"                                                                                 \
  ".rept %[Q]\n"                                                                                  \
  "v_lshl_add_u32 v[cvT], s84, 2, v[24+cvq]\n"                                                    \
  ".set cvd, " d "+cvq*%[PD]\n"                                                                   \
  ".set cvi, 0\n"                                                                                 \
  ".rept (%[P]+1)/2\n"                                                                            \
  "ds_read2_b32 v[cvd+cvi:cvd+cvi+1], v[cvT] offset0:cvi offset1:cvi+1\n"                         \
  ".set cvi, cvi+2\n"                                                                             \
  ".endr\n"                                                                                       \
  ".if ((%[P]+1) & 1)\n"                                                                          \
  "ds_read_b32 v[cvd+%[P]], v[cvT] offset:4*%[P]\n"                                               \
  ".endif\n"                                                                                      \
  ".set cvq, cvq+1\n"                                                                             \
  ".endr\n"
// The lane's words: cvi counts them, cvd their dwords in D0 and D1.
#define LPF_WALK_ROWS(body)                                                                       \
  ".set cvi, 0\n"                                                                                 \
  ".set cvd, 0\n"                                                                                 \
  ".rept %[Q]\n"                                                                                  \
  ".rept %[P]\n"                                                                                  \
  body                                                                                            \
  ".set cvi, cvi+1\n"                                                                             \
  ".set cvd, cvd+1\n"                                                                             \
  ".endr\n"                                                                                       \
  ".set cvd, cvd+%[PD]-%[P]\n"                                                                    \
  ".endr\n"
#define LPF_WALK_MOV(dst, src)                                                                    \
  ".set cvi, 0\n"                                                                                 \
  ".rept %[MV]\n"                                                                                 \
  "v_mov_b32 v[" dst "+cvi], v[" src "+cvi]\n"                                                    \
  ".set cvi, cvi+1\n"                                                                             \
  ".endr\n"

// One product, of pixels in the phase (the array is complemented for phase 0).
#define LPF_WALK_ASM                                                                              \
  LPF_WALK_TEXT(LPF_WALK_TWO1, LPF_WALK_ONE1, LPF_WALK_COUNT1, "ds_add_u32 v[cvT], v[cvN]\n")
#define LPF_WALK_TWO1                                                                             \
  LPF_WALK_ROWS(                                                                                  \
      "v_alignbit_b32 v[cvD0+cvd], v[cvD0+cvd+1], v[cvD0+cvd], s85\n"                             \
      "v_alignbit_b32 v[cvD1+cvd], v[cvD1+cvd+1], v[cvD1+cvd], s86\n"                             \
      "v_bitop3_b32 v[cvA+cvi], v[cvA+cvi], v[cvD0+cvd], v[cvD1+cvd] bitop3:0x80\n")
#define LPF_WALK_ONE1                                                                             \
  LPF_WALK_ROWS(                                                                                  \
      "v_alignbit_b32 v[cvD0+cvd], v[cvD0+cvd+1], v[cvD0+cvd], s85\n"                             \
      "v_and_b32 v[cvA+cvi], v[cvA+cvi], v[cvD0+cvd]\n")
#define LPF_WALK_COUNT1                                                                           \
  "v_bcnt_u32_b32 v[cvN], v[cvA], 0\n"                                                            \
  ".set cvi, 1\n"                                                                                 \
  ".rept %[R]-1\n"                                                                                \
  "v_bcnt_u32_b32 v[cvN], v[cvA+cvi], v[cvN]\n"                                                   \
  ".set cvi, cvi+1\n"                                                                             \
  ".endr\n"

// Both products at once, each step's words read and shifted once: R words of the product of pixels
// in phase 1, then R words of the product of pixels in phase 0.  The two counts of a lane share a
// register for the wave sum (16 bits each: at most 64 x 256), and go to slots `slots0` bytes
// apart.  Zero: both.
#define LPF_WALK_BOTH(slots0)                                                                     \
  LPF_WALK_TEXT(LPF_WALK_TWO2, LPF_WALK_ONE2, LPF_WALK_COUNT2, LPF_WALK_ADD2(slots0))
#define LPF_WALK_TWO2                                                                             \
  LPF_WALK_ROWS(                                                                                  \
      "v_alignbit_b32 v[cvD0+cvd], v[cvD0+cvd+1], v[cvD0+cvd], s85\n"                             \
      "v_alignbit_b32 v[cvD1+cvd], v[cvD1+cvd+1], v[cvD1+cvd], s86\n"                             \
      "v_bitop3_b32 v[cvA+cvi], v[cvA+cvi], v[cvD0+cvd], v[cvD1+cvd] bitop3:0x80\n"               \
      "v_bitop3_b32 v[cvA+%[R]+cvi], v[cvA+%[R]+cvi], v[cvD0+cvd], v[cvD1+cvd] bitop3:0x10\n")
#define LPF_WALK_ONE2                                                                             \
  LPF_WALK_ROWS(                                                                                  \
      "v_alignbit_b32 v[cvD0+cvd], v[cvD0+cvd+1], v[cvD0+cvd], s85\n"                             \
      "v_and_b32 v[cvA+cvi], v[cvA+cvi], v[cvD0+cvd]\n"                                           \
      "v_bitop3_b32 v[cvA+%[R]+cvi], v[cvA+%[R]+cvi], v[cvD0+cvd], v[cvD0+cvd] bitop3:0x30\n")
#define LPF_WALK_COUNT2                                                                           \
  "v_bcnt_u32_b32 v[cvN], v[cvA], 0\n"                                                            \
  "v_bcnt_u32_b32 v[cvN2], v[cvA+%[R]], 0\n"                                                      \
  ".set cvi, 1\n"                                                                                 \
  ".rept %[R]-1\n"                                                                                \
  "v_bcnt_u32_b32 v[cvN], v[cvA+cvi], v[cvN]\n"                                                   \
  "v_bcnt_u32_b32 v[cvN2], v[cvA+%[R]+cvi], v[cvN2]\n"                                            \
  ".set cvi, cvi+1\n"                                                                             \
  ".endr\n"                                                                                       \
  "v_lshl_or_b32 v[cvN], v[cvN2], 16, v[cvN]\n"
#define LPF_WALK_ADD2(slots0)                                                                     \
  "v_lshrrev_b32 v[cvN2], 16, v[cvN]\n"                                                           \
  "v_and_b32 v[cvN], 0xffff, v[cvN]\n"                                                            \
  "ds_add_u32 v[cvT], v[cvN]\n"                                                                   \
  "ds_add_u32 v[cvT], v[cvN2] offset:" slots0 "\n"
