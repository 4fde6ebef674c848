// svf_event_loop.h -- the event loop of the known-length path in gfx950
// assembly: one wave simulates one instance under one policy, with the
// finish-ordered list (ListProf) and the rank bitmap (bits_in, bits_out).
//
// What bounds it.  The loop is almost all uniform control flow with a few
// wave-wide operations on 64 list entries, so its time is the number of
// instructions issued where many waves share a CU (heavy traffic: 8 waves per
// SIMD), and the chain of dependent steps where one wave has a CU to itself.
// Compiled from C++ the same steps took 154 scalar and 115 vector
// instructions per admission: half of them copies of loop state, lane-mask
// handling and conditions rebuilt from flags, because the loop has many exits
// and more live scalars than the register budget of eight waves.  Written out,
// every condition is a branch on SCC or VCC and no value is copied.
//
// Registers.  Loop state is in named operands (%[..], the compiler places
// them); temporaries and tuples whose halves are needed are fixed registers,
// named by the .set lines below.  Every memory load is waited for inside the
// block.
//
// Wait states kept by hand (gfx940 and later): 2 between a VALU write of a
// scalar register or VCC and a VALU read of it, 1 between a VALU write of a
// vector register and a lane read, 2 before a DPP read, 4 between a VALU
// write of a scalar register and its use as a lane number, 5 to its use as an
// address.  The s_nop at the start covers what the compiler, which does not
// look into the block, may have written right before it.
//
// The steps (t: current step, rank: priority position, lower first):
//   visit    every request admitted and finished: done; t at the limit: leave
//   arrivals lanes of the 64-request window with a <= t set their rank bits;
//            the best of those above the blocked head is the candidate
//   begin    newly finished entries: their peak; 32 of them: the list moves down
//   fit      entries with t < F < te: largest G, number p; at te itself
//            ve = G_a - (F_a - te)(c + 1), a the entry at p, c the entries
//            from it on; any of them above lim = M - s + t: does not fit
//   insert   lanes before p: G += F + c_h; lanes from p on move up by one
//   next     the lowest bit left in the open word, else in the bitmap
//   fail     blocked head and the step t_f before which it cannot fit
//   advance  the next arrival ranked above the head, or t_f
#pragma once

// clang-format off

#define EV_NAMES                                                              \
    ".set eQ, 44\n\t"         /* 44..47 record: index, size, planned length, length */\
    ".set eCb, 48\n\t"        /* 48..49 the open bitmap word */               \
    ".set eX, 50\n\t"         /* 50..51 scratch */                            \
    ".set eM1, 52\n\t"        /* 52..53 lanes that arrive now */              \
    ".set eIn, 54\n\t"        /* 54..55 lanes with t < F < te */              \
    ".set eMk, 56\n\t"        /* 56..57 scratch mask */                       \
    ".set eR, 58\n\t"         /* candidate rank */                            \
    ".set eI, 59\n\t"         /* lane number */                               \
    ".set eW, 60\n\t"         /* word number of an arrival; end of an LDS group */\
    ".set eP, 61\n\t"         /* entries before te */                         \
    ".set eTe, 62\n\t"        /* t + planned length */                        \
    ".set eU, 63\n\t"         /* scratch */                                   \
    ".set eFa, 64\n\t"        /* entry a: F */                                \
    ".set eGa, 65\n\t"        /* entry a: G */                                \
    ".set eV, 65\n\t"         /* scratch */                                   \
    ".set eC1, 66\n\t"        /* c + 1 */                                     \
    ".set eVe, 67\n\t"        /* D(te) + te, then the candidate's G */        \
    ".set eLim, 68\n\t"       /* M - s + t */                                 \
    ".set eCh, 68\n\t"        /* s - t */                                     \
    ".set eT1, 69\n\t"        /* t + 1 */                                     \
    ".set eMt, 70\n\t"        /* M + t */                                     \
    ".set eCw, 71\n\t"        /* number of the open word */                   \
    ".set vX, 30\n\t"         /* 30..31 (F, G) of an LDS group; shifted entries */\
    ".set vY, 31\n\t"                                                         \
    ".set vZ, 32\n\t"         /* 32..33 scratch */                            \
    ".set vW, 33\n\t"                                                         \
    ".set vM, 34\n\t"         /* largest G of a check */                      \
    ".set vAd, 35\n\t"        /* LDS address, offsets */                      \
    ".set vAq, 36\n\t"        /* 36..39 records of the arrival window */      \
    ".set vNa, 40\n\t"        /* next window: arrivals */                     \
    ".set vNr, 41\n\t"        /* next window: ranks */                        \
    ".set vPd, 42\n\t"        /* 42..43 progress counter as last read */      \
    ".set vA, 44\n\t"         /* window: arrivals */                          \
    ".set vRk, 45\n\t"        /* window: ranks */                             \
    ".set vM0, 46\n\t"        /* the compiler's m0 */

#define EV_CLOBBER                                                            \
    "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53",     \
    "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63",     \
    "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71",                   \
    "v30", "v31", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39",     \
    "v40", "v41", "v42", "v43", "v44", "v45", "v46", "vcc", "scc", "memory"

// wave-wide maximum or minimum of v[r], in every lane of the last row
#define EV_REDUCE(op, r)                                                      \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"   \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"   \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] row_half_mirror row_mask:0xf bank_mask:0xf\n\t"       \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] row_mirror row_mask:0xf bank_mask:0xf\n\t"            \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"          \
    "s_nop 1\n\t" op " v[" r "], v[" r "], v[" r "] row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"          \
    "s_nop 1\n\t"

// ---- the rank bitmap: up to 4096 ranks in one register pair, up to 8192 in
// two, else both levels in LDS.  SET: the ranks in the lanes eM1 of v[reg];
// OPEN: word eCw into eCb; CLOSE: eCb back; EMPTY: the open word has no bit
// left; SCAN: the lowest non-empty word into eCw, eCb (to ev_none if there is
// none).  l: a suffix for the labels.

#define EV_SET_LOOP(reg, l, body)                                             \
    "s_mov_b64 s[eX:eX+1], s[eM1:eM1+1]\n"                                    \
    ".Lev_bit" l "_%=:\n\t"                                                   \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "v_readlane_b32 s[eU], v[" reg "], s[eI]\n\t"                             \
    "s_bitset0_b64 s[eX:eX+1], s[eI]\n\t"                                     \
    "s_lshr_b32 s[eW], s[eU], 6\n\t"                                          \
    "s_mov_b32 m0, s[eW]\n\t"                                                 \
    body                                                                      \
    "s_cmp_lg_u64 s[eX:eX+1], 0\n\t"                                          \
    "s_cbranch_scc1 .Lev_bit" l "_%=\n\t"

#define EV_SET_PAIR(lo, hi)                                                   \
    "v_readlane_b32 s[eMk], " lo ", s[eW]\n\t"                                \
    "v_readlane_b32 s[eMk+1], " hi ", s[eW]\n\t"                              \
    "s_bitset1_b64 s[eMk:eMk+1], s[eU]\n\t"                                   \
    "v_writelane_b32 " lo ", s[eMk], m0\n\t"                                  \
    "v_writelane_b32 " hi ", s[eMk+1], m0\n\t"

#define EV_GET_PAIR(lo, hi)                                                   \
    "v_readlane_b32 s[eCb], " lo ", s[eCw]\n\t"                               \
    "v_readlane_b32 s[eCb+1], " hi ", s[eCw]\n\t"

#define EV_PUT_PAIR(lo, hi)                                                   \
    "v_writelane_b32 " lo ", s[eCb], m0\n\t"                                  \
    "v_writelane_b32 " hi ", s[eCb+1], m0\n\t"

#define EV_SET_1(reg, l) EV_SET_LOOP(reg, l, EV_SET_PAIR("%[b0l]", "%[b0h]"))
#define EV_OPEN_1(l) EV_GET_PAIR("%[b0l]", "%[b0h]")
#define EV_CLOSE_1(l) "s_mov_b32 m0, s[eCw]\n\t" EV_PUT_PAIR("%[b0l]", "%[b0h]")
#define EV_EMPTY_1 EV_CLOSE_1("")
#define EV_SCAN_1(l)                                                          \
    "v_or_b32 v[vX], %[b0l], %[b0h]\n\t"                                      \
    "v_cmp_ne_u32 vcc, 0, v[vX]\n\t"                                          \
    "s_cbranch_vccz .Lev_none_%=\n\t"                                         \
    "s_ff1_i32_b64 s[eCw], vcc\n\t" EV_OPEN_1(l)

#define EV_SET_2(reg, l)                                                      \
    EV_SET_LOOP(reg, l,                                                       \
                "s_cmp_lt_u32 s[eW], 64\n\t"                                  \
                "s_cbranch_scc0 .Lev_bit1" l "_%=\n\t"                        \
                EV_SET_PAIR("%[b0l]", "%[b0h]")                               \
                "s_branch .Lev_bit2" l "_%=\n"                                \
                ".Lev_bit1" l "_%=:\n\t"                                      \
                EV_SET_PAIR("%[b1l]", "%[b1h]")                               \
                ".Lev_bit2" l "_%=:\n\t")
#define EV_OPEN_2(l)                                                          \
    "s_cmp_lt_u32 s[eCw], 64\n\t"                                             \
    "s_cbranch_scc0 .Lev_get" l "_%=\n\t"                                     \
    EV_GET_PAIR("%[b0l]", "%[b0h]")                                           \
    "s_branch .Lev_got" l "_%=\n"                                             \
    ".Lev_get" l "_%=:\n\t"                                                   \
    EV_GET_PAIR("%[b1l]", "%[b1h]")                                           \
    ".Lev_got" l "_%=:\n\t"
#define EV_CLOSE_2(l)                                                         \
    "s_mov_b32 m0, s[eCw]\n\t"                                                \
    "s_cmp_lt_u32 s[eCw], 64\n\t"                                             \
    "s_cbranch_scc0 .Lev_put" l "_%=\n\t"                                     \
    EV_PUT_PAIR("%[b0l]", "%[b0h]")                                           \
    "s_branch .Lev_pot" l "_%=\n"                                             \
    ".Lev_put" l "_%=:\n\t"                                                   \
    EV_PUT_PAIR("%[b1l]", "%[b1h]")                                           \
    ".Lev_pot" l "_%=:\n\t"
#define EV_EMPTY_2 EV_CLOSE_2("f")
#define EV_SCAN_2(l)                                                          \
    "v_or_b32 v[vX], %[b0l], %[b0h]\n\t"                                      \
    "v_cmp_ne_u32 vcc, 0, v[vX]\n\t"                                          \
    "s_cbranch_vccz .Lev_find1" l "_%=\n\t"                                   \
    "s_ff1_i32_b64 s[eCw], vcc\n\t"                                           \
    EV_GET_PAIR("%[b0l]", "%[b0h]")                                           \
    "s_branch .Lev_found" l "_%=\n"                                           \
    ".Lev_find1" l "_%=:\n\t"                                                 \
    "v_or_b32 v[vX], %[b1l], %[b1h]\n\t"                                      \
    "v_cmp_ne_u32 vcc, 0, v[vX]\n\t"                                          \
    "s_cbranch_vccz .Lev_none_%=\n\t"                                         \
    "s_ff1_i32_b64 s[eCw], vcc\n\t"                                           \
    "s_add_i32 s[eCw], s[eCw], 64\n\t"                                        \
    EV_GET_PAIR("%[b1l]", "%[b1h]")                                           \
    ".Lev_found" l "_%=:\n\t"

/* LDS: word w at %[bb] + 8 w, its level above at %[sb] + 8 (w >> 6), %[w1]
   words of it */
#define EV_SET_0(reg, l)                                                      \
    "s_mov_b64 exec, s[eM1:eM1+1]\n\t"                                        \
    "v_lshrrev_b32 v[vAd], 6, v[" reg "]\n\t"                                 \
    "v_lshlrev_b64 v[vX:vX+1], v[" reg "], 1\n\t"                             \
    "v_lshlrev_b64 v[vZ:vZ+1], v[vAd], 1\n\t"                                 \
    "v_lshlrev_b32 v[vAd], 3, v[vAd]\n\t"                                     \
    "v_add_u32 v[vAd], %[bb], v[vAd]\n\t"                                     \
    "ds_or_b64 v[vAd], v[vX:vX+1]\n\t"                                        \
    "v_lshrrev_b32 v[vAd], 12, v[" reg "]\n\t"                                \
    "v_lshlrev_b32 v[vAd], 3, v[vAd]\n\t"                                     \
    "v_add_u32 v[vAd], %[sb], v[vAd]\n\t"                                     \
    "ds_or_b64 v[vAd], v[vZ:vZ+1]\n\t"                                        \
    "s_mov_b64 exec, -1\n\t"
#define EV_OPEN_0(l)                                                          \
    "s_lshl3_add_u32 s[eU], s[eCw], %[bb]\n\t"                                \
    "v_mov_b32 v[vAd], s[eU]\n\t"                                             \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_readfirstlane_b32 s[eCb], v[vX]\n\t"                                   \
    "v_readfirstlane_b32 s[eCb+1], v[vY]\n\t"
/* (every lane stores the same word) */
#define EV_CLOSE_0(l)                                                         \
    "s_lshl3_add_u32 s[eU], s[eCw], %[bb]\n\t"                                \
    "v_mov_b32 v[vAd], s[eU]\n\t"                                             \
    "v_mov_b32 v[vX], s[eCb]\n\t"                                             \
    "v_mov_b32 v[vY], s[eCb+1]\n\t"                                           \
    "ds_write_b64 v[vAd], v[vX:vX+1]\n\t"
#define EV_EMPTY_0                                                            \
    EV_CLOSE_0("")                                                            \
    "s_lshr_b32 s[eU], s[eCw], 6\n\t"                                         \
    "s_lshl3_add_u32 s[eU], s[eU], %[sb]\n\t"                                 \
    "v_mov_b32 v[vAd], s[eU]\n\t"                                             \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_readfirstlane_b32 s[eCb], v[vX]\n\t"                                   \
    "v_readfirstlane_b32 s[eCb+1], v[vY]\n\t"                                 \
    "s_bitset0_b64 s[eCb:eCb+1], s[eCw]\n\t"                                  \
    "v_mov_b32 v[vX], s[eCb]\n\t"                                             \
    "v_mov_b32 v[vY], s[eCb+1]\n\t"                                           \
    "ds_write_b64 v[vAd], v[vX:vX+1]\n\t"
#define EV_SCAN_0(l)                                                          \
    "s_mov_b32 s[eW], 0\n"                                                    \
    ".Lev_find" l "_%=:\n\t"                                                  \
    "s_lshl3_add_u32 s[eU], s[eW], %[sb]\n\t"                                 \
    "v_lshlrev_b32 v[vAd], 3, %[lane]\n\t"                                    \
    "v_add_u32 v[vAd], s[eU], v[vAd]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_sub_i32 s[eU], %[w1], s[eW]\n\t"                                       \
    "v_cmp_gt_i32 s[eMk:eMk+1], s[eU], %[lane]\n\t"                           \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_cmp_ne_u64 vcc, 0, v[vX:vX+1]\n\t"                                     \
    "s_and_b64 vcc, vcc, s[eMk:eMk+1]\n\t"                                    \
    "s_cbranch_scc1 .Lev_found" l "_%=\n\t"                                   \
    "s_add_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_cmp_lt_i32 s[eW], %[w1]\n\t"                                           \
    "s_cbranch_scc1 .Lev_find" l "_%=\n\t"                                    \
    "s_branch .Lev_none_%=\n"                                                 \
    ".Lev_found" l "_%=:\n\t"                                                 \
    "s_ff1_i32_b64 s[eI], vcc\n\t"                                            \
    "v_readlane_b32 s[eX], v[vX], s[eI]\n\t"                                  \
    "v_readlane_b32 s[eX+1], v[vY], s[eI]\n\t"                                \
    "s_add_i32 s[eI], s[eI], s[eW]\n\t"                                       \
    "s_ff1_i32_b64 s[eCw], s[eX:eX+1]\n\t"                                    \
    "s_lshl_b32 s[eI], s[eI], 6\n\t"                                          \
    "s_add_i32 s[eCw], s[eCw], s[eI]\n\t"                                     \
    EV_OPEN_0(l)

// the next 64 requests: arrivals and ranks were loaded one window ahead
#define EV_RELOAD                                                             \
    "s_add_i32 %[wb], %[wb], 64\n\t"                                          \
    "s_mov_b64 %[pend], -1\n\t"                                               \
    "v_add_u32 v[vAd], %[wb], %[lane]\n\t"                                    \
    "v_cmp_ge_i32 vcc, %[n1], v[vAd]\n\t"                                     \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_min_u32 v[vNr], %[n1], v[vNr]\n\t"                                     \
    "v_cndmask_b32 v[vA], %[vmax], v[vNa], vcc\n\t"                           \
    "v_cndmask_b32 v[vRk], %[vmax], v[vNr], vcc\n\t"                          \
    "v_lshlrev_b32 v[vZ], 4, v[vNr]\n\t"                                      \
    "global_load_dwordx4 v[vAq:vAq+3], v[vZ], %[rec]\n\t"                     \
    "v_add_u32 v[vAd], 64, v[vAd]\n\t"                                        \
    "v_min_i32 v[vAd], %[n1], v[vAd]\n\t"                                     \
    "v_lshlrev_b32 v[vAd], 2, v[vAd]\n\t"                                     \
    "global_load_dword v[vNa], v[vAd], %[arr]\n\t"                            \
    "global_load_dword v[vNr], v[vAd], %[rank]\n\t"

// The check of a candidate (size eQ+1, planned length eQ+2) started at t and,
// when it fits, its place in the list: entries with t < F < te, their largest
// G (vM) and number (eP); then, past the limit and the room, the insertion.  A full
// register group first pushes lane 63's entry.
#define EV_FIT                                                                \
    "v_subrev_u32 v[vX], s[eT1], %[F]\n\t"                                    \
    "s_add_i32 s[eU], s[eQ+2], -1\n\t"                                        \
    "v_cmp_gt_u32 s[eIn:eIn+1], s[eU], v[vX]\n\t"                             \
    "s_add_i32 s[eTe], %[t], s[eQ+2]\n\t"                                     \
    "s_bcnt1_i32_b64 s[eP], s[eIn:eIn+1]\n\t"                                 \
    "s_add_i32 s[eP], s[eP], %[dead]\n\t"                                     \
    "v_cndmask_b32 v[vM], %[vmin], %[G], s[eIn:eIn+1]\n\t"                    \
    "s_cmp_gt_u32 s[eP], 63\n\t"                                              \
    "s_cbranch_scc1 .Lev_deep_%=\n\t"                                         \
    "v_readlane_b32 s[eFa], %[F], s[eP]\n\t"                                  \
    "v_readlane_b32 s[eGa], %[G], s[eP]\n\t"                                  \
    "s_sub_i32 s[eC1], %[ln1], s[eP]\n\t"                                     \
    "s_sub_i32 s[eFa], s[eFa], s[eTe]\n\t"                                    \
    "s_mul_i32 s[eFa], s[eFa], s[eC1]\n\t"                                    \
    "s_sub_i32 s[eVe], s[eGa], s[eFa]\n\t"                                    \
    "s_sub_i32 s[eLim], s[eMt], s[eQ+1]\n\t"                                  \
    "v_max_i32 v[vM], s[eVe], v[vM]\n\t"                                      \
    "v_cmp_lt_i32 vcc, s[eLim], v[vM]\n\t"                                    \
    "s_cbranch_vccnz .Lev_fail_%=\n\t"                                        \
    "s_cmp_gt_i32 %[ln1], %[cap]\n\t"                                         \
    "s_cbranch_scc1 .Lev_full_%=\n\t"                                         \
                                                                              \
    /* insert; a full register group first pushes lane 63's entry */          \
    "s_sub_i32 s[eCh], s[eQ+1], %[t]\n\t"                                     \
    "s_add_i32 s[eVe], s[eVe], s[eTe]\n\t"                                    \
    "s_add_i32 s[eVe], s[eVe], s[eCh]\n\t"                                    \
    "s_cmp_gt_i32 %[ln1], 64\n\t"                                             \
    "s_cbranch_scc0 .Lev_nopush_%=\n\t"                                       \
    "s_lshl3_add_u32 s[eU], %[ln1], %[pushb]\n\t"                             \
    "s_brev_b32 exec_hi, 1\n\t"                                               \
    "s_mov_b32 exec_lo, 0\n\t"                                                \
    "v_mov_b32 v[vAd], s[eU]\n\t"                                             \
    "ds_write2_b32 v[vAd], %[F], %[G] offset1:1\n\t"                          \
    "s_mov_b64 exec, -1\n"                                                    \
    ".Lev_nopush_%=:\n\t"                                                     \
    "v_mov_b32_dpp v[vX], %[F] wave_shr:1 row_mask:0xf bank_mask:0xf\n\t"     \
    "v_mov_b32_dpp v[vY], %[G] wave_shr:1 row_mask:0xf bank_mask:0xf\n\t"     \
    "s_lshl_b64 s[eMk:eMk+1], -1, s[eP]\n\t"                                  \
    "v_add3_u32 v[vM], %[F], %[G], s[eCh]\n\t"                                \
    "s_mov_b32 m0, s[eP]\n\t"                                                 \
    "v_writelane_b32 v[vX], s[eTe], m0\n\t"                                   \
    "v_writelane_b32 v[vY], s[eVe], m0\n\t"                                   \
    "v_cndmask_b32 %[F], %[F], v[vX], s[eMk:eMk+1]\n\t"                       \
    "v_cndmask_b32 %[G], v[vM], v[vY], s[eMk:eMk+1]\n"

// It does not fit: t_f = max over the violating steps of min(tau, D + tau - X).
#define EV_REL                                                                \
    "s_sub_i32 s[eU], %[M], s[eQ+1]\n\t"                                      \
    "v_subrev_u32 v[vX], s[eU], %[G]\n\t"                                     \
    "v_min_i32 v[vX], v[vX], %[F]\n\t"                                        \
    "v_cndmask_b32 v[vX], %[vmin], v[vX], s[eIn:eIn+1]\n"                     \
    ".Lev_rel_%=:\n\t"                                                        \
    EV_REDUCE("v_max_i32_dpp", "vX")                                          \
    "v_readlane_b32 %[tf], v[vX], 63\n\t"                                     \
    "s_sub_i32 s[eV], s[eVe], s[eU]\n\t"                                      \
    "s_min_i32 s[eV], s[eV], s[eTe]\n\t"                                      \
    "s_max_i32 %[tf], %[tf], s[eV]\n\t"

// The first eU entries leave: lane i takes entry i + eU, from the stack past
// lane 63.
#define EV_DROP                                                               \
    "v_add_u32 v[vX], s[eU], %[lane]\n\t"                                     \
    "v_lshlrev_b32 v[vY], 2, v[vX]\n\t"                                       \
    "v_and_b32 v[vY], 0xfc, v[vY]\n\t"                                        \
    "ds_bpermute_b32 v[vZ], v[vY], %[F]\n\t"                                  \
    "ds_bpermute_b32 v[vW], v[vY], %[G]\n\t"                                  \
    "s_sub_i32 s[eV], 64, s[eU]\n\t"                                          \
    "s_bfm_b64 s[eMk:eMk+1], s[eV], 0\n\t"                                    \
    "s_add_i32 s[eV], %[ln1], -2\n\t"                                         \
    "v_sub_u32 v[vX], s[eV], v[vX]\n\t"                                       \
    "v_max_i32 v[vX], -1, v[vX]\n\t"                                          \
    "v_cndmask_b32 v[vX], v[vX], -1, s[eMk:eMk+1]\n\t"                        \
    "v_lshlrev_b32 v[vX], 3, v[vX]\n\t"                                       \
    "v_add_u32 v[vX], 0x208, v[vX]\n\t"                                       \
    "v_add_u32 v[vAd], %[pushb], v[vX]\n\t"                                   \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_sub_i32 %[ln1], %[ln1], s[eU]\n\t"                                     \
    "s_mov_b32 %[dead], 0\n\t"                                                \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_cndmask_b32 %[F], v[vX], v[vZ], s[eMk:eMk+1]\n\t"                      \
    "v_cndmask_b32 %[G], v[vY], v[vW], s[eMk:eMk+1]\n\t"

// The check past the registers: groups of the stack from its end, eW one past
// the group's entries.
#define EV_DEEP                                                               \
    ".Lev_deep_%=:\n\t"                                                       \
    "s_add_i32 s[eW], %[ln1], -65\n"                                          \
    ".Lev_deepg_%=:\n\t"                                                      \
    "s_lshl_b32 s[eU], s[eW], 3\n\t"                                          \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_cmp_gt_i32 vcc, s[eTe], v[vX]\n\t"                                     \
    "s_bcnt1_i32_b64 s[eP], vcc\n\t"                                          \
    "s_cmp_gt_u32 s[eP], 63\n\t"                                              \
    "v_cndmask_b32 v[vZ], %[vmin], v[vY], vcc\n\t"                            \
    "v_max_i32 v[vM], v[vM], v[vZ]\n\t"                                       \
    "s_cbranch_scc0 .Lev_deepe_%=\n\t"                                        \
    "s_sub_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_branch .Lev_deepg_%=\n"                                                \
    ".Lev_deepe_%=:\n\t"                                                      \
    "v_readlane_b32 s[eFa], v[vX], s[eP]\n\t"                                 \
    "v_readlane_b32 s[eGa], v[vY], s[eP]\n\t"                                 \
    "s_sub_i32 s[eC1], s[eW], s[eP]\n\t"                                      \
    "s_add_i32 s[eC1], s[eC1], 1\n\t"                                         \
    "s_sub_i32 s[eFa], s[eFa], s[eTe]\n\t"                                    \
    "s_mul_i32 s[eFa], s[eFa], s[eC1]\n\t"                                    \
    "s_sub_i32 s[eVe], s[eGa], s[eFa]\n\t"                                    \
    "s_sub_i32 s[eLim], s[eMt], s[eQ+1]\n\t"                                  \
    "v_max_i32 v[vM], s[eVe], v[vM]\n\t"                                      \
    "v_cmp_lt_i32 vcc, s[eLim], v[vM]\n\t"                                    \
    "s_add_i32 s[eC1], %[ln1], -65\n\t"                                       \
    "s_cbranch_vccnz .Lev_deepfail_%=\n\t"                                    \
    "s_cmp_gt_i32 %[ln1], %[cap]\n\t"                                         \
    "s_cbranch_scc1 .Lev_full_%=\n\t"                                         \
    /* insert: the registers and whole groups before te move up unchanged in  \
       order; in the last group lanes before p move up and lane p stores the  \
       candidate above its own entry */                                       \
    "s_sub_i32 s[eCh], s[eQ+1], %[t]\n\t"                                     \
    "s_add_i32 s[eVe], s[eVe], s[eTe]\n\t"                                    \
    "s_add_i32 s[eVe], s[eVe], s[eCh]\n\t"                                    \
    "v_add3_u32 %[G], %[F], %[G], s[eCh]\n"                                   \
    ".Lev_deepi_%=:\n\t"                                                      \
    "s_cmp_eq_u32 s[eC1], s[eW]\n\t"                                          \
    "s_cbranch_scc1 .Lev_deepl_%=\n\t"                                        \
    "s_lshl_b32 s[eU], s[eC1], 3\n\t"                                         \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "ds_read_b64 v[vZ:vZ+1], v[vAd]\n\t"                                      \
    "s_sub_i32 s[eC1], s[eC1], 64\n\t"                                        \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_add3_u32 v[vW], v[vZ], v[vW], s[eCh]\n\t"                              \
    "ds_write_b64 v[vAd], v[vZ:vZ+1] offset:8\n\t"                            \
    "s_branch .Lev_deepi_%=\n"                                                \
    ".Lev_deepl_%=:\n\t"                                                      \
    "s_lshl_b32 s[eU], s[eW], 3\n\t"                                          \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "v_add3_u32 v[vY], v[vX], v[vY], s[eCh]\n\t"                              \
    "s_mov_b32 m0, s[eP]\n\t"                                                 \
    "v_writelane_b32 v[vX], s[eTe], m0\n\t"                                   \
    "v_writelane_b32 v[vY], s[eVe], m0\n\t"                                   \
    "s_lshl_b64 exec, -2, s[eP]\n\t"                                          \
    "s_not_b64 exec, exec\n\t"                                                \
    "ds_write_b64 v[vAd], v[vX:vX+1] offset:8\n\t"                            \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_branch .Lev_adm_%=\n"                                                  \
    /* fail past the registers: the same groups again */                      \
    ".Lev_deepfail_%=:\n\t"                                                   \
    "s_sub_i32 s[eU], %[M], s[eQ+1]\n\t"                                      \
    "v_subrev_u32 v[vM], s[eU], %[G]\n\t"                                     \
    "v_min_i32 v[vM], v[vM], %[F]\n\t"                                        \
    "v_cndmask_b32 v[vM], %[vmin], v[vM], s[eIn:eIn+1]\n"                     \
    ".Lev_deepr_%=:\n\t"                                                      \
    "s_lshl_b32 s[eV], s[eC1], 3\n\t"                                         \
    "v_add_u32 v[vAd], s[eV], %[rev]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_cmp_gt_i32 vcc, s[eTe], v[vX]\n\t"                                     \
    "v_subrev_u32 v[vY], s[eU], v[vY]\n\t"                                    \
    "v_min_i32 v[vY], v[vY], v[vX]\n\t"                                       \
    "v_cndmask_b32 v[vY], %[vmin], v[vY], vcc\n\t"                            \
    "v_max_i32 v[vM], v[vM], v[vY]\n\t"                                       \
    "s_sub_i32 s[eC1], s[eC1], 64\n\t"                                        \
    "s_cmp_ge_i32 s[eC1], s[eW]\n\t"                                          \
    "s_cbranch_scc1 .Lev_deepr_%=\n\t"                                        \
    "v_mov_b32 v[vX], v[vM]\n\t"                                              \
    "s_branch .Lev_rel_%=\n"

// The issue priority by the remaining work, n - done requests; the progress
// since the last update into the launch's counter.
#define EV_PRIO(done)                                                         \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_readfirstlane_b32 s[eU], v[vPd]\n\t"                                   \
    "v_readfirstlane_b32 s[eV], v[vPd+1]\n\t"                                 \
    "s_sub_i32 s[eFa], %[n1], " done "\n\t"                                   \
    "s_add_i32 s[eFa], s[eFa], 1\n\t"                                         \
    "s_lshr_b32 s[eC1], s[eV], 8\n\t"          /* waves in the count */       \
    "s_and_b32 s[eV], s[eV], 0xff\n\t"                                        \
    "s_mul_i32 s[eX], s[eFa], s[eC1]\n\t"                                     \
    "s_mul_hi_u32 s[eX+1], s[eFa], s[eC1]\n\t"                                \
    "s_sub_u32 s[eX], s[eX], s[eU]\n\t"        /* d: (mine - mean) * waves */ \
    "s_subb_u32 s[eX+1], s[eX+1], s[eV]\n\t"                                  \
    "s_mul_i32 s[eMk], %[th], s[eC1]\n\t"      /* s: the level step * waves */\
    "s_mul_hi_u32 s[eMk+1], %[th], s[eC1]\n\t"                                \
    "s_sub_u32 s[eU], s[eMk], s[eX]\n\t"                                      \
    "s_subb_u32 s[eU], s[eMk+1], s[eX+1]\n\t"                                 \
    "s_cmp_lt_i32 s[eU], 0\n\t"                /* d > s */                    \
    "s_cbranch_scc1 .Lev_prio3_%=\n\t"                                        \
    "s_sub_u32 s[eU], 0, s[eX]\n\t"                                           \
    "s_subb_u32 s[eU], 0, s[eX+1]\n\t"                                        \
    "s_cmp_lt_i32 s[eU], 0\n\t"                /* d > 0 */                    \
    "s_cbranch_scc1 .Lev_prio2_%=\n\t"                                        \
    "s_add_u32 s[eU], s[eX], s[eMk]\n\t"                                      \
    "s_addc_u32 s[eU], s[eX+1], s[eMk+1]\n\t"                                 \
    "s_cmp_lt_i32 s[eU], 0\n\t"                /* d < -s */                   \
    "s_cbranch_scc1 .Lev_prio0_%=\n\t"                                        \
    "s_setprio 1\n\t"                                                         \
    "s_branch .Lev_prio_%=\n"                                                 \
    ".Lev_prio0_%=:\n\t"                                                      \
    "s_setprio 0\n\t"                                                         \
    "s_branch .Lev_prio_%=\n"                                                 \
    ".Lev_prio2_%=:\n\t"                                                      \
    "s_setprio 2\n\t"                                                         \
    "s_branch .Lev_prio_%=\n"                                                 \
    ".Lev_prio3_%=:\n\t"                                                      \
    "s_setprio 3\n"                                                           \
    ".Lev_prio_%=:\n\t"                                                       \
    "s_sub_i32 s[eU], %[last], " done "\n\t"                                  \
    "s_ashr_i32 s[eV], s[eU], 31\n\t"                                         \
    "s_mov_b32 %[last], " done "\n\t"                                         \
    "v_mov_b32 v[vZ], s[eU]\n\t"                                              \
    "v_mov_b32 v[vW], s[eV]\n\t"                                              \
    "v_mov_b32 v[vM], 0\n\t"                                                  \
    "s_mov_b64 exec, 1\n\t"                                                   \
    "global_atomic_add_x2 v[vPd:vPd+1], v[vM], v[vZ:vZ+1], %[ctr] sc0\n\t"    \
    "s_mov_b64 exec, -1\n"

// ---- the loop

#define EV_LOOP(SET, OPEN, CLOSE, EMPTY, SCAN)                                \
    EV_NAMES                                                                  \
    "s_nop 4\n\t"                                                             \
    "v_mov_b32 v[vM0], m0\n\t"                                                \
    /* the first window's arrivals and ranks; the progress counter */         \
    "v_add_u32 v[vAd], %[wb], %[lane]\n\t"                                    \
    "v_min_i32 v[vAd], %[n1], v[vAd]\n\t"                                     \
    "v_lshlrev_b32 v[vAd], 2, v[vAd]\n\t"                                     \
    "global_load_dword v[vNa], v[vAd], %[arr]\n\t"                            \
    "global_load_dword v[vNr], v[vAd], %[rank]\n\t"                           \
    "s_cmp_lg_u64 %[ctr], 0\n\t"                                              \
    "s_cbranch_scc0 .Lev_noctr_%=\n\t"                                        \
    "v_mov_b32 v[vZ], 0\n\t"                                                  \
    "global_load_dwordx2 v[vPd:vPd+1], v[vZ], %[ctr]\n"                       \
    ".Lev_noctr_%=:\n\t"                                                      \
    "s_sub_i32 %[wb], %[wb], 64\n\t"                                          \
    EV_RELOAD                                                                 \
                                                                              \
    /* visit (at the start of a cache line: 4 bytes further on the loop took  \
       1.66 in place of 1.62 ms on 3 x 4096 x 1000, 0.59 for 0.57 on 512) */  \
    ".p2align 6\n"                                                            \
    ".Lev_visit_%=:\n\t"                                                      \
    "s_add_i32 s[eU], %[seq], %[nstg]\n\t"                                    \
    "s_cmp_gt_i32 s[eU], %[n1]\n\t"                                           \
    "s_cbranch_scc1 .Lev_alladm_%=\n"                                         \
    ".Lev_visit1_%=:\n\t"                                                     \
    "s_cmp_ge_i32 %[t], %[tstop]\n\t"                                         \
    "s_cbranch_scc1 .Lev_exit_%=\n\t"                                         \
    "s_mov_b32 s[eR], %[head]\n"                                              \
                                                                              \
    /* arrivals */                                                            \
    ".Lev_arr_%=:\n\t"                                                        \
    "v_cmp_ge_i32 vcc, %[t], v[vA]\n\t"                                       \
    "s_and_b64 s[eM1:eM1+1], vcc, %[pend]\n\t"                                \
    "s_cbranch_scc0 .Lev_noarr_%=\n\t"                                        \
    "s_andn2_b64 %[pend], %[pend], s[eM1:eM1+1]\n\t"                          \
    SET("vRk", "")                                                            \
    "v_cmp_gt_i32 vcc, s[eR], v[vRk]\n\t"                                     \
    "s_and_b64 s[eX:eX+1], vcc, s[eM1:eM1+1]\n\t"                             \
    "s_cbranch_scc0 .Lev_arrdone_%=\n\t"                                      \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "s_bcnt1_i32_b64 s[eU], s[eX:eX+1]\n\t"                                   \
    "s_cmp_eq_u32 s[eU], 1\n\t"                                               \
    "s_cbranch_scc1 .Lev_one_%=\n\t"                                          \
    "v_cndmask_b32 v[vX], %[vmax], v[vRk], s[eX:eX+1]\n\t"                    \
    EV_REDUCE("v_min_i32_dpp", "vX")                                          \
    "v_readlane_b32 s[eU], v[vX], 63\n\t"                                     \
    "s_nop 1\n\t"                                                             \
    "v_cmp_eq_u32 vcc, s[eU], v[vRk]\n\t"                                     \
    "s_and_b64 s[eX:eX+1], vcc, s[eX:eX+1]\n\t"                               \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n"                                       \
    ".Lev_one_%=:\n\t"                                                        \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_readlane_b32 s[eR], v[vRk], s[eI]\n\t"                                 \
    "v_readlane_b32 s[eQ], v[vAq], s[eI]\n\t"                                 \
    "v_readlane_b32 s[eQ+1], v[vAq+1], s[eI]\n\t"                             \
    "v_readlane_b32 s[eQ+2], v[vAq+2], s[eI]\n"                               \
    ".Lev_arrdone_%=:\n\t"                                                    \
    "s_cmp_eq_u64 %[pend], 0\n\t"                                             \
    "s_cbranch_scc1 .Lev_reload_%=\n"                                         \
    ".Lev_noarr_%=:\n\t"                                                      \
    "s_cmp_lt_i32 s[eR], %[head]\n\t"                                         \
    "s_cbranch_scc1 .Lev_cand_%=\n\t"                                         \
    "s_cmp_ge_i32 %[t], %[tf]\n\t"                                            \
    "s_cbranch_scc0 .Lev_adv_%=\n\t"                                          \
    "s_mov_b32 s[eQ], %[h0]\n\t"                                              \
    "s_mov_b32 s[eQ+1], %[h1]\n\t"                                            \
    "s_mov_b32 s[eQ+2], %[h2]\n"                                              \
                                                                              \
    /* begin */                                                               \
    ".Lev_cand_%=:\n\t"                                                       \
    "v_cmp_ge_i32 vcc, %[t], %[F]\n\t"                                        \
    "s_bcnt1_i32_b64 s[eU], vcc\n\t"                                          \
    "s_add_i32 s[eT1], %[t], 1\n\t"                                           \
    "s_add_i32 s[eMt], %[t], %[M]\n\t"                                        \
    "s_cmp_lg_u32 s[eU], %[dead]\n\t"                                         \
    "s_cbranch_scc1 .Lev_begin_%=\n"                                          \
    ".Lev_begun_%=:\n\t"                                                      \
    "s_mov_b32 %[tprev], %[t]\n\t"                                            \
    "s_lshr_b32 s[eCw], s[eR], 6\n\t"                                         \
    OPEN("o")                                                                 \
                                                                              \
    /* fit */                                                                 \
    ".Lev_fit_%=:\n\t"                                                        \
    EV_FIT                                                                    \
    /* admitted */                                                            \
    ".Lev_adm_%=:\n\t"                                                        \
    "s_add_i32 %[ln1], %[ln1], 1\n\t"                                         \
    "s_mov_b32 m0, %[nstg]\n\t"                                               \
    "v_writelane_b32 %[sgi], s[eQ], m0\n\t"                                   \
    "v_writelane_b32 %[sgt], %[t], m0\n\t"                                    \
    "s_max_i32 %[mf], %[mf], s[eTe]\n\t"                                      \
    "s_bitset0_b64 s[eCb:eCb+1], s[eR]\n\t"                                   \
    "s_add_i32 %[nstg], %[nstg], 1\n\t"                                       \
    "s_cmp_eq_u32 %[nstg], 64\n\t"                                            \
    "s_cbranch_scc1 .Lev_flush_%=\n"                                          \
    ".Lev_next_%=:\n\t"                                                       \
    "s_cmp_eq_u64 s[eCb:eCb+1], 0\n\t"                                        \
    "s_cbranch_scc1 .Lev_word_%=\n"                                           \
    ".Lev_pick_%=:\n\t"                                                       \
    "s_ff1_i32_b64 s[eR], s[eCb:eCb+1]\n\t"                                   \
    "s_lshl_b32 s[eU], s[eCw], 6\n\t"                                         \
    "s_add_i32 s[eR], s[eR], s[eU]\n\t"                                       \
    "s_cmp_eq_u32 s[eR], %[head]\n\t"                                         \
    "s_cbranch_scc1 .Lev_oldhead_%=\n"                                        \
    ".Lev_rec_%=:\n\t"                                                        \
    "s_lshl_b32 s[eU], s[eR], 4\n\t"                                          \
    "s_load_dwordx4 s[eQ:eQ+3], %[rec], s[eU]\n\t"                            \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "s_branch .Lev_fit_%=\n"                                                  \
    /* the old head: before t_f it still does not fit (the profile has only   \
       grown since t_f was computed) */                                       \
    ".Lev_oldhead_%=:\n\t"                                                    \
    "s_cmp_ge_i32 %[t], %[tf]\n\t"                                            \
    "s_cbranch_scc1 .Lev_rec_%=\n\t"                                          \
    "s_branch .Lev_close_%=\n"                                                \
    ".Lev_word_%=:\n\t"                                                       \
    EMPTY                                                                     \
    SCAN("")                                                                  \
    "s_branch .Lev_pick_%=\n"                                                 \
    ".Lev_none_%=:\n\t"                                                       \
    "s_brev_b32 %[head], -2\n\t"                                              \
    "s_brev_b32 %[tf], -2\n\t"                                                \
    "s_branch .Lev_adv_%=\n"                                                  \
                                                                              \
    /* fail: t_f = max over the violating steps of min(tau, D + tau - X) */   \
    ".Lev_fail_%=:\n\t"                                                       \
    EV_REL                                                                    \
    "s_mov_b32 %[head], s[eR]\n\t"                                            \
    "s_mov_b32 %[h0], s[eQ]\n\t"                                              \
    "s_mov_b32 %[h1], s[eQ+1]\n\t"                                            \
    "s_mov_b32 %[h2], s[eQ+2]\n"                                              \
    ".Lev_close_%=:\n\t"                                                      \
    CLOSE("c")                                                                \
                                                                              \
    /* advance */                                                             \
    ".Lev_adv_%=:\n\t"                                                        \
    "v_cmp_gt_i32 vcc, %[head], v[vRk]\n\t"                                   \
    "s_and_b64 s[eX:eX+1], vcc, %[pend]\n\t"                                  \
    "s_cbranch_scc0 .Lev_advnone_%=\n\t"                                      \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "v_readlane_b32 s[eV], v[vA], s[eI]\n\t"                                  \
    "s_min_i32 s[eV], s[eV], %[tf]\n"                                         \
    ".Lev_advto_%=:\n\t"                                                      \
    "s_add_i32 s[eU], %[t], 1\n\t"                                            \
    "s_min_i32 s[eV], s[eV], %[tstop]\n\t"                                    \
    "s_max_i32 %[t], s[eV], s[eU]\n\t"                                        \
    "s_branch .Lev_visit_%=\n"                                                \
    /* none in the window: its end, or (no more to come) the head's release   \
       or the last finish */                                                  \
    ".Lev_advnone_%=:\n\t"                                                    \
    "s_add_i32 s[eU], %[wb], 63\n\t"                                          \
    "s_mov_b32 s[eV], %[tf]\n\t"                                              \
    "s_cmp_lt_i32 s[eU], %[n1]\n\t"                                           \
    "s_cbranch_scc0 .Lev_advlast_%=\n\t"                                      \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_readfirstlane_b32 s[eV], v[vNa]\n\t"                                   \
    "s_min_i32 s[eV], s[eV], %[tf]\n\t"                                       \
    "s_branch .Lev_advto_%=\n"                                                \
    ".Lev_advlast_%=:\n\t"                                                    \
    "s_add_i32 s[eU], %[mf], 1\n\t"                                           \
    "s_cmp_eq_u32 %[head], 0x7fffffff\n\t"                                    \
    "s_cselect_b32 s[eV], s[eU], s[eV]\n\t"                                   \
    "s_branch .Lev_advto_%=\n"                                                \
                                                                              \
    ".Lev_reload_%=:\n\t"                                                     \
    EV_RELOAD                                                                 \
    "s_branch .Lev_arr_%=\n"                                                  \
                                                                              \
    /* begin: the memory at the finish steps of the newly finished entries,   \
       tprev < F <= t; they stay in front until 32 have gathered */           \
    ".Lev_begin_%=:\n\t"                                                      \
    "s_add_i32 s[eV], %[tprev], 1\n\t"                                        \
    "v_subrev_u32 v[vX], s[eV], %[F]\n\t"                                     \
    "s_sub_i32 s[eV], %[t], %[tprev]\n\t"                                     \
    "v_cmp_gt_u32 s[eMk:eMk+1], s[eV], v[vX]\n\t"                             \
    "v_sub_u32 v[vY], %[G], %[F]\n\t"                                         \
    "s_mov_b32 %[dead], s[eU]\n\t"                                            \
    "s_nop 0\n\t"                                                             \
    "v_cndmask_b32 v[vY], 0, v[vY], s[eMk:eMk+1]\n\t"                         \
    "v_max_i32 %[peak], %[peak], v[vY]\n\t"                                   \
    "s_cmp_lt_u32 s[eU], 32\n\t"                                              \
    "s_cbranch_scc1 .Lev_begun_%=\n\t"                                        \
    EV_DROP                                                                   \
    "v_cmp_ge_i32 vcc, %[t], %[F]\n\t"                                        \
    "s_bcnt1_i32_b64 s[eU], vcc\n\t"                                          \
    "s_cmp_lg_u32 s[eU], 0\n\t"                                               \
    "s_cbranch_scc1 .Lev_begin_%=\n\t"                                        \
    "s_branch .Lev_begun_%=\n"                                                \
                                                                              \
    EV_DEEP                                                                   \
                                                                              \
    /* 64 staged admissions out; the issue priority by the remaining work */  \
    ".Lev_flush_%=:\n\t"                                                      \
    "v_lshlrev_b32 v[vAd], 2, %[sgi]\n\t"                                     \
    "v_add_u32 v[vX], %[seq], %[lane]\n\t"                                    \
    "s_add_i32 %[seq], %[seq], 64\n\t"                                        \
    "s_mov_b32 %[nstg], 0\n\t"                                                \
    "s_cmp_eq_u64 %[ctr], 0\n\t"                                              \
    "s_cbranch_scc1 .Lev_noprio_%=\n\t"                                       \
    EV_PRIO("%[seq]")                                                         \
    ".Lev_noprio_%=:\n\t"                                                     \
    "global_store_dword v[vAd], %[sgt], %[start]\n\t"                         \
    "global_store_dword v[vAd], v[vX], %[adm]\n\t"                            \
    "s_branch .Lev_next_%=\n"                                                 \
                                                                              \
    /* a full list: the candidate is the head, checked again at t when the    \
       segment resumes */                                                     \
    ".Lev_full_%=:\n\t"                                                       \
    "s_mov_b32 %[head], s[eR]\n\t"                                            \
    "s_mov_b32 %[tf], -1\n\t"                                                 \
    CLOSE("g")                                                                \
    "s_branch .Lev_exit_%=\n"                                                 \
    ".Lev_alladm_%=:\n\t"                                                     \
    "s_cmp_lt_i32 %[mf], %[t]\n\t"                                            \
    "s_cbranch_scc0 .Lev_visit1_%=\n"                                         \
    ".Lev_exit_%=:\n\t"                                                       \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t"                                       \
    "v_readfirstlane_b32 s[eU], v[vM0]\n\t"                                   \
    "s_mov_b32 m0, s[eU]\n\t"

#define EV_LOOP_1 EV_LOOP(EV_SET_1, EV_OPEN_1, EV_CLOSE_1, EV_EMPTY_1, EV_SCAN_1)
#define EV_LOOP_2 EV_LOOP(EV_SET_2, EV_OPEN_2, EV_CLOSE_2, EV_EMPTY_2, EV_SCAN_2)
#define EV_LOOP_0 EV_LOOP(EV_SET_0, EV_OPEN_0, EV_CLOSE_0, EV_EMPTY_0, EV_SCAN_0)

#define EV_STATE                                                              \
    [t] "+&s"(t), [head] "+&s"(head), [tf] "+&s"(t_f), [h0] "+&s"(hq.x),          \
    [h1] "+&s"(hq.y), [h2] "+&s"(hq.z), [mf] "+&s"(max_fin), [seq] "+&s"(seq),    \
    [nstg] "+&s"(nstg), [wb] "+&s"(wb), [pend] "+&s"(pend), [ln1] "+&s"(ln1),     \
    [dead] "+&s"(L.dead), [tprev] "+&s"(L.tprev), [last] "+&s"(prio.last),       \
    [F] "+&v"(L.F), [G] "+&v"(L.G), [peak] "+&v"(L.peak_lane),                   \
    [sgi] "+&v"(stg_idx), [sgt] "+&v"(stg_t)

#define EV_INPUT                                                              \
    [tstop] "s"(t_stop), [n1] "s"(n - 1), [M] "s"(P.M), [cap] "s"(L.cap),     \
    [pushb] "s"(stk - 65 * 8), [rec] "s"(sg.rec),             \
    [rank] "s"(sg.rank), [arr] "s"(sg.a), [start] "s"(sg.start),              \
    [adm] "s"(sg.admit_seq), [ctr] "s"(prio.ctr), [th] "s"(prio.th),          \
    [lane] "v"(lane), [vmin] "v"(INT32_MIN), [vmax] "v"(INT32_MAX),           \
    [rev] "v"(stk - 8 - 8 * lane)

// clang-format on
