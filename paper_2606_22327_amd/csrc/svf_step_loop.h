// svf_step_loop.h -- the loop of the per-step path in gfx950 assembly: requests
// that may finish before or after their planned length (1-bit SVF, predicted
// lengths), overflow of the true memory with eviction, next-step admission.
//
// What bounds it.  Compiled from C++ with the running requests in global memory
// the waves waited for half of their cycles: each finish and each eviction
// scanned the whole running list through L2, at four waves per SIMD.  Here the
// running requests are in registers, 64 E places of {F, 2c, T, rank and index}
// (F planned finish, T true finish, c = s - k), any free place taking the next
// admission: a finish is a compare per group, an eviction a 24-bit product per
// group and one wave-wide maximum.  What needs no step is not visited: the
// memory held at t + 1 is C + n (t + 1) over all running requests, so a
// request that passes its planned length changes nothing but the planned
// profile, whose entries end by themselves.  With next-step admission there is
// no planned profile at all.  Measured, simulation per launch before and now:
// predicted lengths 8,192 x 5,000: 113 -> 40 ms; 1-bit SVF beside three known
// policies 4,096 x 1,000: 9.2 -> 3.4 ms; next-step admission 2,048 x 1,000 x 2:
// 9.9 -> 2.4 ms; predicted lengths, 1,531 ragged queues x 2: 23.2 -> 7.7 ms.
// E = 6: at most 231 requests run at once in those and 376 at twice their
// budget; 24 registers still leave six waves per SIMD.  E = 4 (eight
// waves) took 2 to 6 % less on the three smaller ones and a third more on
// predicted lengths 8,192 x 5,000 (56.9 against 42.4 ms a pass).
//
// The planned profile is the finish-ordered list of the event path
// (svf_event_loop.h: EV_FIT, EV_DEEP), with removal of entries whose request
// finishes early or is evicted.  A segment that needs more than 64 E places or
// a longer list leaves inside the admissions of its step; a launch with E = 10
// (five waves per SIMD) continues it there, and one with E = 32 and room for the
// bound what outgrows that.  Registers and wait states as in
// svf_event_loop.h.
#pragma once

#include "svf_event_loop.h"

// clang-format off

#define ST_NAMES                                                              \
    ".set eQ, 60\n\t"         /* 60..63 record: index, size, planned length, length */\
    ".set eCb, 64\n\t"        /* 64..65 the open bitmap word */               \
    ".set eX, 66\n\t"         /* 66..67 scratch */                            \
    ".set eM1, 68\n\t"        /* 68..69 lanes of a SET */                     \
    ".set eIn, 70\n\t"        /* 70..71 lanes with t < F < te; lanes that finish */\
    ".set eMk, 72\n\t"        /* 72..73 scratch mask */                       \
    ".set eR, 74\n\t"         /* candidate rank */                            \
    ".set eI, 75\n\t"         /* lane number */                               \
    ".set eW, 76\n\t"         /* word number; end of an LDS group */          \
    ".set eP, 77\n\t"         /* entries before te */                         \
    ".set eTe, 78\n\t"        /* t + planned length */                        \
    ".set eU, 79\n\t"         /* scratch */                                   \
    ".set eFa, 80\n\t"        /* entry a: F */                                \
    ".set eGa, 81\n\t"        /* entry a: G */                                \
    ".set eV, 81\n\t"         /* scratch */                                   \
    ".set eC1, 82\n\t"        /* c + 1 */                                     \
    ".set eVe, 83\n\t"        /* D(te) + te, then the candidate's G */        \
    ".set eLim, 84\n\t"       /* M - s + t */                                 \
    ".set eCh, 84\n\t"        /* s - t */                                     \
    ".set eT1, 85\n\t"        /* t + 1 */                                     \
    ".set eMt, 86\n\t"        /* M + t */                                     \
    ".set eCw, 87\n\t"        /* number of the open word */                   \
    ".set eNm, 88\n\t"        /* memory at t + 1 with the candidate */        \
    ".set eMem, 89\n\t"       /* memory at t + 1 */                           \
    ".set eRet, 90\n\t"       /* 90..91 return address */                     \
    ".set eRet2, 92\n\t"      /* 92..93 return address */                     \
    ".set vX, 20\n\t"         /* 20..21 (F, G) of an LDS group; shifted entries */\
    ".set vY, 21\n\t"                                                         \
    ".set vZ, 22\n\t"         /* 22..23 scratch */                            \
    ".set vW, 23\n\t"                                                         \
    ".set vM, 24\n\t"         /* largest G of a check; wave reductions */     \
    ".set vAd, 25\n\t"        /* LDS address, offsets */                      \
    ".set vNa, 26\n\t"        /* next window: arrivals */                     \
    ".set vNr, 27\n\t"        /* next window: ranks */                        \
    ".set vPd, 28\n\t"        /* 28..29 progress counter as last read */      \
    ".set vA, 30\n\t"         /* window: arrivals */                          \
    ".set vRk, 31\n\t"        /* window: ranks */                             \
    ".set vM0, 32\n\t"        /* the compiler's m0 */                         \
    ".set vEv, 33\n\t"        /* ranks evicted at t */                        \
    ".set vCF, 34\n\t"        /* finishing entries: F */                      \
    ".set vCC, 35\n\t"        /*   2 (s - k) */                               \
    ".set vCI, 36\n\t"        /*   rank and index */                          \
    ".set uR, 38\n\t"         /* E registers: a b of the group's requests */

#define ST_PLACES_6           ".set uU, 44\n\t"   /* 4 E registers: the running requests */
#define ST_PLACES_10           ".set uU, 48\n\t"   /* 4 E registers: the running requests */
#define ST_PLACES_32          ".set uU, 70\n\t"   /* 4 E registers: the running requests */

#define ST_CLOBBER_6                                                          \
    "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69",     \
    "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79",     \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89",     \
    "s90", "s91", "s92", "s93", "v20", "v21", "v22", "v23", "v24", "v25",     \
    "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35",     \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45",     \
    "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55",     \
    "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65",     \
    "v66", "v67", "vcc", "scc", "memory"

#define ST_CLOBBER_10                                                         \
    "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69",     \
    "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79",     \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89",     \
    "s90", "s91", "s92", "s93", "v20", "v21", "v22", "v23", "v24", "v25",     \
    "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35",     \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45",     \
    "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55",     \
    "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65",     \
    "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", "v74", "v75",     \
    "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85",     \
    "v86", "v87", "vcc", "scc", "memory"

#define ST_CLOBBER_32                                                         \
    "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69",     \
    "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79",     \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89",     \
    "s90", "s91", "s92", "s93", "v20", "v21", "v22", "v23", "v24", "v25",     \
    "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35",     \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45",     \
    "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55",     \
    "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65",     \
    "v66", "v67", "v68", "v69", "v70", "v71", "v72", "v73", "v74", "v75",     \
    "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85",     \
    "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95",     \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104",       \
    "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113",   \
    "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122",   \
    "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131",   \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140",   \
    "v141", "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149",   \
    "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", "v158",   \
    "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167",   \
    "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", "v176",   \
    "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185",   \
    "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", "v194",   \
    "v195", "v196", "v197", "vcc", "scc", "memory"

#define ST_REP_6(M)                                                           \
    M(0) M(1) M(2) M(3) M(4) M(5)

#define ST_REP_10(M)                                                          \
    M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9)

#define ST_REP_32(M)                                                          \
    M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7)                                   \
    M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15)                             \
    M(16) M(17) M(18) M(19) M(20) M(21) M(22) M(23)                           \
    M(24) M(25) M(26) M(27) M(28) M(29) M(30) M(31)

// the running requests: {F, 2 (s - k), true finish T, rank << 16 | index}; T = INT32_MAX: a free place
#define ST_LOADU(u)                                                           \
    "v_add_u32 v[vX], 64*" #u ", %[lane]\n\t"                                 \
    "v_cmp_gt_i32 vcc, %[nA], v[vX]\n\t"                                      \
    "v_mov_b32 v[uU+4*" #u "], 0\n\t"                                         \
    "v_mov_b32 v[uU+4*" #u "+1], 0\n\t"                                       \
    "v_mov_b32 v[uU+4*" #u "+2], %[vmax]\n\t"                                 \
    "v_mov_b32 v[uU+4*" #u "+3], 0\n\t"                                       \
    "v_lshlrev_b32 v[vX], 4, v[vX]\n\t"                                       \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "global_load_dwordx4 v[uU+4*" #u ":uU+4*" #u "+3], v[vX], %[act]\n\t"     \
    "s_mov_b64 exec, -1\n\t"

#define ST_STOREU(u)                                                          \
    "v_cmp_ne_u32 vcc, %[vmax], v[uU+4*" #u "+2]\n\t"                         \
    "s_cbranch_vccz .Lst_su" #u "_%=\n\t"                                     \
    "s_bcnt1_i32_b64 s[eU], vcc\n\t"                                          \
    "s_nop 0\n\t"                                                             \
    "v_mbcnt_lo_u32_b32 v[vX], vcc_lo, 0\n\t"                                 \
    "v_mbcnt_hi_u32_b32 v[vX], vcc_hi, v[vX]\n\t"                             \
    "v_add_u32 v[vX], s[eP], v[vX]\n\t"                                       \
    "v_lshlrev_b32 v[vX], 4, v[vX]\n\t"                                       \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "global_store_dwordx4 v[vX], v[uU+4*" #u ":uU+4*" #u "+3], %[act]\n\t"    \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_add_i32 s[eP], s[eP], s[eU]\n\t"                                       \
    ".Lst_su" #u "_%=:\n"

// the first free place takes the candidate
#define ST_FREE(u)                                                            \
    "v_cmp_eq_u32 vcc, %[vmax], v[uU+4*" #u "+2]\n\t"                         \
    "s_cbranch_vccz .Lst_fr" #u "_%=\n\t"                                     \
    "s_ff1_i32_b64 s[eI], vcc\n\t"                                            \
    "s_mov_b32 m0, s[eI]\n\t"                                                 \
    "v_writelane_b32 v[uU+4*" #u "], s[eTe], m0\n\t"                          \
    "v_writelane_b32 v[uU+4*" #u "+1], s[eV], m0\n\t"                         \
    "v_writelane_b32 v[uU+4*" #u "+2], s[eU], m0\n\t"                         \
    "v_writelane_b32 v[uU+4*" #u "+3], s[eW], m0\n\t"                         \
    "s_branch .Lst_put_%=\n\t"                                                \
    ".Lst_fr" #u "_%=:\n"

#define ST_EVENT(u)                                                           \
    "v_cmp_eq_u32 vcc, %[t], v[uU+4*" #u "+2]\n\t"                            \
    "s_cbranch_vccz .Lst_ne" #u "_%=\n\t"                                     \
    "s_mov_b64 s[eIn:eIn+1], vcc\n\t"                                         \
    "v_mov_b32 v[vCF], v[uU+4*" #u "]\n\t"                                    \
    "v_mov_b32 v[vCC], v[uU+4*" #u "+1]\n\t"                                  \
    "v_mov_b32 v[vCI], v[uU+4*" #u "+3]\n\t"                                  \
    "s_call_b64 s[eRet:eRet+1], .Lst_fin_%=\n\t"                              \
    "v_cndmask_b32 v[uU+4*" #u "+2], v[uU+4*" #u "+2], %[vmax], s[eIn:eIn+1]\n\t"\
    ".Lst_ne" #u "_%=:\n"                                                     \
    "v_min_i32 v[vM], v[vM], v[uU+4*" #u "+2]\n\t"

// twice the remaining volume (the host checks that it stays below 2^32, its factors below 2^24)
#define ST_VOLUME(u)                                                          \
    "v_cmp_ne_u32 vcc, %[vmax], v[uU+4*" #u "+2]\n\t"                         \
    "v_mov_b32 v[uR+" #u "], 0\n\t"                                           \
    "s_cbranch_vccz .Lst_nv" #u "_%=\n\t"                                     \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "v_max_i32 v[vX], s[eT1], v[uU+4*" #u "]\n\t"                             \
    "v_add3_u32 v[vY], v[uU+4*" #u "+1], v[vX], s[eT1]\n\t"                   \
    "v_subrev_u32 v[vX], %[t], v[vX]\n\t"                                     \
    "v_mul_u32_u24 v[uR+" #u "], v[vX], v[vY]\n\t"                            \
    "s_mov_b64 exec, -1\n\t"                                                  \
    ".Lst_nv" #u "_%=:\n"

#define ST_LARGEST(u)                                                         \
    "v_max_u32 v[vM], v[vM], v[uR+" #u "]\n\t"

// the latest index among the largest: its lane eC1, group eVe, index eP, F eTe, 2c eCh, rank and index eR
#define ST_VICTIM(u)                                                          \
    "v_cmp_eq_u32 vcc, s[eFa], v[uR+" #u "]\n\t"                              \
    "s_cbranch_vccz .Lst_nt" #u "_%=\n\t"                                     \
    "s_mov_b64 s[eX:eX+1], vcc\n\t"                                           \
    ".Lst_tl" #u "_%=:\n"                                                     \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "s_bitset0_b64 s[eX:eX+1], s[eI]\n\t"                                     \
    "v_readlane_b32 s[eU], v[uU+4*" #u "+3], s[eI]\n\t"                       \
    "s_and_b32 s[eV], s[eU], 0xffff\n\t"                                      \
    "s_cmp_gt_i32 s[eV], s[eP]\n\t"                                           \
    "s_cbranch_scc0 .Lst_tn" #u "_%=\n\t"                                     \
    "s_mov_b32 s[eP], s[eV]\n\t"                                              \
    "s_mov_b32 s[eR], s[eU]\n\t"                                              \
    "s_mov_b32 s[eC1], s[eI]\n\t"                                             \
    "s_mov_b32 s[eVe], " #u "\n\t"                                            \
    "v_readlane_b32 s[eTe], v[uU+4*" #u "], s[eI]\n\t"                        \
    "v_readlane_b32 s[eCh], v[uU+4*" #u "+1], s[eI]\n\t"                      \
    ".Lst_tn" #u "_%=:\n"                                                     \
    "s_cmp_lg_u64 s[eX:eX+1], 0\n\t"                                          \
    "s_cbranch_scc1 .Lst_tl" #u "_%=\n\t"                                     \
    ".Lst_nt" #u "_%=:\n"

#define ST_REMOVE(u)                                                          \
    "s_cmp_eq_u32 s[eVe], " #u "\n\t"                                         \
    "s_cbranch_scc0 .Lst_nd" #u "_%=\n\t"                                     \
    "s_mov_b32 m0, s[eC1]\n\t"                                                \
    "s_brev_b32 s[eU], -2\n\t"                                                \
    "v_writelane_b32 v[uU+4*" #u "+2], s[eU], m0\n\t"                         \
    "v_writelane_b32 v[uR+" #u "], 0, m0\n\t"                                 \
    "s_branch .Lst_gone_%=\n\t"                                               \
    ".Lst_nd" #u "_%=:\n"

// the next 64 requests: arrivals and ranks were loaded one window ahead
#define ST_RELOAD                                                             \
    "s_add_i32 %[wb], %[wb], 64\n\t"                                          \
    "s_mov_b64 %[pend], -1\n\t"                                               \
    "v_add_u32 v[vAd], %[wb], %[lane]\n\t"                                    \
    "v_cmp_ge_i32 vcc, %[n1], v[vAd]\n\t"                                     \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_min_u32 v[vNr], %[n1], v[vNr]\n\t"                                     \
    "v_cndmask_b32 v[vA], %[vmax], v[vNa], vcc\n\t"                           \
    "v_cndmask_b32 v[vRk], %[vmax], v[vNr], vcc\n\t"                          \
    "v_add_u32 v[vAd], 64, v[vAd]\n\t"                                        \
    "v_min_i32 v[vAd], %[n1], v[vAd]\n\t"                                     \
    "v_lshlrev_b32 v[vAd], 2, v[vAd]\n\t"                                     \
    "global_load_dword v[vNa], v[vAd], %[arr]\n\t"                            \
    "global_load_dword v[vNr], v[vAd], %[rank]\n\t"

// what a partial sum of the list is held at or above, -2^30
#define ST_FLOOR "0xc0000000"

// ---- the loop

#define ST_LOOP(REP, PLACES, SET, CLOSE, EMPTY, SCAN)                         \
    ST_NAMES                                                                  \
    PLACES                                                                    \
    "s_nop 4\n\t"                                                             \
    "v_mov_b32 v[vM0], m0\n\t"                                                \
    /* the running requests of the launch before */                           \
    REP(ST_LOADU)                                                             \
    /* the first window's arrivals and ranks; the progress counter */         \
    "v_add_u32 v[vAd], %[wb], %[lane]\n\t"                                    \
    "v_min_i32 v[vAd], %[n1], v[vAd]\n\t"                                     \
    "v_lshlrev_b32 v[vAd], 2, v[vAd]\n\t"                                     \
    "global_load_dword v[vNa], v[vAd], %[arr]\n\t"                            \
    "global_load_dword v[vNr], v[vAd], %[rank]\n\t"                           \
    "s_cmp_lg_u64 %[ctr], 0\n\t"                                              \
    "s_cbranch_scc0 .Lst_noctr_%=\n\t"                                        \
    "v_mov_b32 v[vZ], 0\n\t"                                                  \
    "global_load_dwordx2 v[vPd:vPd+1], v[vZ], %[ctr]\n\t"                     \
    ".Lst_noctr_%=:\n"                                                        \
    "s_sub_i32 %[wb], %[wb], 64\n\t"                                          \
    ST_RELOAD                                                                 \
    /* continued inside the admissions of step t: the ranks evicted there */  \
    "s_cmp_lt_i32 %[nev], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_visit_%=\n\t"                                        \
    "v_lshlrev_b32 v[vAd], 2, %[lane]\n\t"                                    \
    "v_cmp_gt_i32 vcc, %[nev], %[lane]\n\t"                                   \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "global_load_dword v[vEv], v[vAd], %[evl]\n\t"                            \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "s_add_i32 s[eT1], %[t], 1\n\t"                                           \
    "s_add_i32 s[eMt], %[t], %[M]\n\t"                                        \
    "s_mul_i32 s[eMem], %[nA], s[eT1]\n\t"                                    \
    "s_add_i32 s[eMem], s[eMem], %[C]\n\t"                                    \
    "s_branch .Lst_admit_%=\n\t"                                              \
                                                                              \
    /* visit */                                                               \
    ".Lst_visit_%=:\n"                                                        \
    "s_cmp_gt_i32 %[nfin], %[n1]\n\t"                                         \
    "s_cbranch_scc1 .Lst_exit_%=\n\t"                                         \
    "s_cmp_ge_i32 %[t], %[tstop]\n\t"                                         \
    "s_cbranch_scc1 .Lst_exit_%=\n\t"                                         \
    "s_mov_b32 %[nev], 0\n\t"                                                 \
    "s_add_i32 s[eT1], %[t], 1\n\t"                                           \
    "s_add_i32 s[eMt], %[t], %[M]\n\t"                                        \
                                                                              \
    /* arrivals; one ranked above the blocked head ends its wait */           \
    ".Lst_arr_%=:\n"                                                          \
    "v_cmp_ge_i32 vcc, %[t], v[vA]\n\t"                                       \
    "s_and_b64 s[eM1:eM1+1], vcc, %[pend]\n\t"                                \
    "s_cbranch_scc0 .Lst_noarr_%=\n\t"                                        \
    "s_andn2_b64 %[pend], %[pend], s[eM1:eM1+1]\n\t"                          \
    SET("vRk", "")                                                            \
    "v_cmp_gt_i32 vcc, %[head], v[vRk]\n\t"                                   \
    "s_and_b64 s[eX:eX+1], vcc, s[eM1:eM1+1]\n\t"                             \
    "s_cselect_b32 %[tf], 0, %[tf]\n\t"                                       \
    "s_cmp_eq_u64 %[pend], 0\n\t"                                             \
    "s_cbranch_scc1 .Lst_reload_%=\n\t"                                       \
    ".Lst_noarr_%=:\n"                                                        \
    "s_cmp_ge_i32 %[t], %[nextev]\n\t"                                        \
    "s_cbranch_scc1 .Lst_events_%=\n\t"                                       \
                                                                              \
    /* planned entries that ended stay in front of the list until 32 have gathered */\
    ".Lst_evdone_%=:\n"                                                       \
    "v_cmp_ge_i32 vcc, %[t], %[F]\n\t"                                        \
    "s_bcnt1_i32_b64 %[dead], vcc\n\t"                                        \
    "s_cmp_gt_u32 %[dead], 31\n\t"                                            \
    "s_cbranch_scc1 .Lst_drop_%=\n\t"                                         \
    "s_mul_i32 s[eMem], %[nA], s[eT1]\n\t"                                    \
    "s_add_i32 s[eMem], s[eMem], %[C]\n\t"                                    \
    "s_cmp_gt_i32 s[eMem], %[M]\n\t"                                          \
    "s_cbranch_scc1 .Lst_evict_%=\n\t"                                        \
    ".Lst_evicted_%=:\n"                                                      \
    "s_cmp_gt_i32 %[tf], %[t]\n\t"                                            \
    "s_cbranch_scc1 .Lst_after_%=\n\t"                                        \
                                                                              \
    /* admissions */                                                          \
    ".Lst_admit_%=:\n"                                                        \
    SCAN("s")                                                                 \
    ".Lst_pick_%=:\n"                                                         \
    "s_ff1_i32_b64 s[eR], s[eCb:eCb+1]\n\t"                                   \
    "s_lshl_b32 s[eU], s[eCw], 6\n\t"                                         \
    "s_add_i32 s[eR], s[eR], s[eU]\n\t"                                       \
    "s_lshl_b32 s[eU], s[eR], 4\n\t"                                          \
    "s_load_dwordx4 s[eQ:eQ+3], %[rec], s[eU]\n\t"                            \
    "s_cmp_ge_u32 %[nA], %[places]\n\t"                                       \
    "s_cbranch_scc1 .Lev_full_%=\n\t"                                         \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    /* over at t + 1 with its first token: blocked until something is released */\
    "s_add_i32 s[eNm], s[eMem], s[eQ+1]\n\t"                                  \
    "s_cmp_ge_i32 s[eNm], %[M]\n\t"                                           \
    "s_cbranch_scc1 .Lst_fail1_%=\n\t"                                        \
    "s_cmp_lg_u32 %[cur], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_current_%=\n\t"                                      \
    EV_FIT                                                                    \
                                                                              \
    ".Lev_adm_%=:\n"                                                          \
    "s_add_i32 %[ln1], %[ln1], 1\n\t"                                         \
    ".Lst_run_%=:\n"                                                          \
    "s_sub_i32 s[eCh], s[eQ+1], %[t]\n\t"                                     \
    "s_lshl_b32 s[eV], s[eCh], 1\n\t"                                         \
    "s_lshl_b32 s[eW], s[eR], 16\n\t"                                         \
    "s_or_b32 s[eW], s[eW], s[eQ]\n\t"                                        \
    "s_add_i32 s[eU], %[t], s[eQ+3]\n\t"                                      \
    REP(ST_FREE)                                                              \
    ".Lst_put_%=:\n"                                                          \
    "s_min_i32 %[nextev], %[nextev], s[eU]\n\t"                               \
    "s_add_i32 %[C], %[C], s[eCh]\n\t"                                        \
    "s_add_i32 %[nA], %[nA], 1\n\t"                                           \
    "s_add_i32 s[eMem], s[eNm], 1\n\t"                                        \
    "s_mov_b32 m0, %[nstg]\n\t"                                               \
    "v_writelane_b32 %[sgi], s[eQ], m0\n\t"                                   \
    "v_writelane_b32 %[sgt], %[t], m0\n\t"                                    \
    "s_bitset0_b64 s[eCb:eCb+1], s[eR]\n\t"                                   \
    "s_add_i32 %[nstg], %[nstg], 1\n\t"                                       \
    "s_cmp_eq_u32 %[nstg], 64\n\t"                                            \
    "s_cbranch_scc1 .Lst_flush_%=\n\t"                                        \
    ".Lst_next_%=:\n"                                                         \
    "s_cmp_lg_u64 s[eCb:eCb+1], 0\n\t"                                        \
    "s_cbranch_scc1 .Lst_pick_%=\n\t"                                         \
    EMPTY                                                                     \
    SCAN("")                                                                  \
    "s_branch .Lst_pick_%=\n\t"                                               \
    /* next-step admission keeps no planned profile */                        \
    ".Lst_current_%=:\n"                                                      \
    "s_add_i32 s[eTe], %[t], s[eQ+2]\n\t"                                     \
    "s_branch .Lst_run_%=\n\t"                                                \
                                                                              \
    ".Lev_none_%=:\n"                                                         \
    "s_brev_b32 %[head], -2\n\t"                                              \
    "s_brev_b32 %[tf], -2\n\t"                                                \
    "s_branch .Lst_after_%=\n\t"                                              \
    ".Lst_fail1_%=:\n"                                                        \
    "s_brev_b32 %[tf], -2\n\t"                                                \
    "s_branch .Lst_blocked_%=\n\t"                                            \
    ".Lev_fail_%=:\n"                                                         \
    EV_REL                                                                    \
    ".Lst_blocked_%=:\n"                                                      \
    "s_mov_b32 %[head], s[eR]\n\t"                                            \
    CLOSE("c")                                                                \
                                                                              \
    /* evicted requests compete again from the next step */                   \
    ".Lst_after_%=:\n"                                                        \
    "s_cmp_lg_u32 %[nev], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_back_%=\n\t"                                         \
                                                                              \
    /* advance: the next finish, arrival ranked above the head, release step, or the\
       first step whose memory is over M */                                   \
    "s_cmp_gt_i32 %[nfin], %[n1]\n\t"                                         \
    "s_mov_b32 s[eV], s[eT1]\n\t"                                             \
    "s_cbranch_scc1 .Lst_advto_%=\n\t"                                        \
    "s_min_i32 s[eV], %[nextev], %[tstop]\n\t"                                \
    "s_min_i32 s[eV], s[eV], %[tf]\n\t"                                       \
    "v_cmp_gt_i32 vcc, %[head], v[vRk]\n\t"                                   \
    "s_and_b64 s[eX:eX+1], vcc, %[pend]\n\t"                                  \
    "s_cbranch_scc0 .Lst_advnone_%=\n\t"                                      \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "v_readlane_b32 s[eU], v[vA], s[eI]\n\t"                                  \
    ".Lst_advmin_%=:\n"                                                       \
    "s_min_i32 s[eV], s[eV], s[eU]\n\t"                                       \
    ".Lst_advmem_%=:\n"                                                       \
    "s_max_i32 s[eV], s[eV], s[eT1]\n\t"                                      \
    "s_sub_i32 s[eU], s[eV], s[eT1]\n\t"                                      \
    "s_mul_i32 s[eW], %[nA], s[eU]\n\t"                                       \
    "s_mul_hi_u32 s[eP], %[nA], s[eU]\n\t"                                    \
    "s_sub_i32 s[eFa], %[M], s[eMem]\n\t"                                     \
    "s_cmp_lg_u32 s[eP], 0\n\t"                                               \
    "s_cbranch_scc1 .Lst_div_%=\n\t"                                          \
    "s_cmp_gt_u32 s[eW], s[eFa]\n\t"                                          \
    "s_cbranch_scc1 .Lst_div_%=\n\t"                                          \
    ".Lst_advto_%=:\n"                                                        \
    "s_sub_i32 s[eU], s[eV], %[t]\n\t"                                        \
    "s_mul_i32 s[eW], %[nA], s[eU]\n\t"                                       \
    "s_mul_hi_u32 s[eP], %[nA], s[eU]\n\t"                                    \
    "s_sub_i32 s[eW], s[eW], %[nA]\n\t"                                       \
    "s_add_i32 s[eW], s[eW], s[eMem]\n\t"                                     \
    "s_max_i32 %[peak], %[peak], s[eW]\n\t"                                   \
    "s_mul_i32 s[eW], %[nA], s[eU]\n\t"                                       \
    "s_add_u32 %[rsl], %[rsl], s[eW]\n\t"                                     \
    "s_addc_u32 %[rsh], %[rsh], s[eP]\n\t"                                    \
    "s_mov_b32 %[t], s[eV]\n\t"                                               \
    "s_branch .Lst_visit_%=\n\t"                                              \
    /* none in the window: the next window's first, if there is one */        \
    ".Lst_advnone_%=:\n"                                                      \
    "s_add_i32 s[eU], %[wb], 63\n\t"                                          \
    "s_cmp_lt_i32 s[eU], %[n1]\n\t"                                           \
    "s_cbranch_scc0 .Lst_advmem_%=\n\t"                                       \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_readfirstlane_b32 s[eU], v[vNa]\n\t"                                   \
    "s_branch .Lst_advmin_%=\n\t"                                             \
    /* the memory passes M before that: floor((M - memory) / running) steps on, from\
       an estimate in 64-bit floating point, corrected */                     \
    ".Lst_div_%=:\n"                                                          \
    "v_cvt_f64_u32 v[vZ:vZ+1], %[nA]\n\t"                                     \
    "v_rcp_f64 v[vZ:vZ+1], v[vZ:vZ+1]\n\t"                                    \
    "v_cvt_f64_u32 v[vX:vX+1], s[eFa]\n\t"                                    \
    "s_nop 1\n\t"                                                             \
    "v_mul_f64 v[vX:vX+1], v[vX:vX+1], v[vZ:vZ+1]\n\t"                        \
    "v_cvt_u32_f64 v[vX], v[vX:vX+1]\n\t"                                     \
    "s_nop 1\n\t"                                                             \
    "v_readfirstlane_b32 s[eP], v[vX]\n\t"                                    \
    "s_mul_i32 s[eW], s[eP], %[nA]\n\t"                                       \
    "s_sub_i32 s[eW], s[eFa], s[eW]\n\t"                                      \
    ".Lst_div1_%=:\n"                                                         \
    "s_cmp_lt_i32 s[eW], 0\n\t"                                               \
    "s_cbranch_scc0 .Lst_div2_%=\n\t"                                         \
    "s_add_i32 s[eP], s[eP], -1\n\t"                                          \
    "s_add_i32 s[eW], s[eW], %[nA]\n\t"                                       \
    "s_branch .Lst_div1_%=\n\t"                                               \
    ".Lst_div2_%=:\n"                                                         \
    "s_cmp_ge_i32 s[eW], %[nA]\n\t"                                           \
    "s_cbranch_scc0 .Lst_div3_%=\n\t"                                         \
    "s_add_i32 s[eP], s[eP], 1\n\t"                                           \
    "s_sub_i32 s[eW], s[eW], %[nA]\n\t"                                       \
    "s_branch .Lst_div2_%=\n\t"                                               \
    ".Lst_div3_%=:\n"                                                         \
    "s_add_i32 s[eV], s[eT1], s[eP]\n\t"                                      \
    "s_branch .Lst_advto_%=\n\t"                                              \
                                                                              \
    /* evicted at t: their bits (the first 64 in vEv, the others in memory) */\
    ".Lst_back_%=:\n"                                                         \
    "s_mov_b32 s[eC1], 0\n\t"                                                 \
    ".Lst_back1_%=:\n"                                                        \
    "s_sub_i32 s[eP], %[nev], s[eC1]\n\t"                                     \
    "s_bfm_b64 s[eM1:eM1+1], s[eP], 0\n\t"                                    \
    "s_cmp_lt_i32 s[eP], 64\n\t"                                              \
    "s_cbranch_scc1 .Lst_back2_%=\n\t"                                        \
    "s_mov_b64 s[eM1:eM1+1], -1\n\t"                                          \
    ".Lst_back2_%=:\n"                                                        \
    SET("vEv", "e")                                                           \
    "s_add_i32 s[eC1], s[eC1], 64\n\t"                                        \
    "s_mov_b32 %[tf], 0\n\t"                                                  \
    "s_mov_b32 s[eV], s[eT1]\n\t"                                             \
    "s_sub_i32 s[eP], %[nev], s[eC1]\n\t"                                     \
    "s_cmp_gt_i32 s[eP], 0\n\t"                                               \
    "s_cbranch_scc0 .Lst_advto_%=\n\t"                                        \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "v_cmp_gt_i32 vcc, s[eP], %[lane]\n\t"                                    \
    "v_add_u32 v[vAd], s[eC1], %[lane]\n\t"                                   \
    "v_lshlrev_b32 v[vAd], 2, v[vAd]\n\t"                                     \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "global_load_dword v[vEv], v[vAd], %[evl]\n\t"                            \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_waitcnt vmcnt(0)\n\t"                                                  \
    "s_branch .Lst_back1_%=\n\t"                                              \
                                                                              \
    /* 64 staged admissions out */                                            \
    ".Lst_flush_%=:\n"                                                        \
    "v_lshlrev_b32 v[vAd], 2, %[sgi]\n\t"                                     \
    "v_add_u32 v[vX], %[seq], %[lane]\n\t"                                    \
    "global_store_dword v[vAd], %[sgt], %[start]\n\t"                         \
    "global_store_dword v[vAd], v[vX], %[adm]\n\t"                            \
    "s_add_i32 %[seq], %[seq], 64\n\t"                                        \
    "s_mov_b32 %[nstg], 0\n\t"                                                \
    "s_branch .Lst_next_%=\n\t"                                               \
                                                                              \
    /* true finishes at t, and the next one */                                \
    ".Lst_events_%=:\n"                                                       \
    "v_mov_b32 v[vM], %[vmax]\n\t"                                            \
    REP(ST_EVENT)                                                             \
    EV_REDUCE("v_min_i32_dpp", "vM")                                          \
    "v_readlane_b32 %[nextev], v[vM], 63\n\t"                                 \
    "s_cmp_eq_u64 %[ctr], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_evdone_%=\n\t"                                       \
    "s_sub_i32 s[eU], %[nfin], %[last]\n\t"                                   \
    "s_cmp_lt_i32 s[eU], 32\n\t"                                              \
    "s_cbranch_scc1 .Lst_evdone_%=\n\t"                                       \
    EV_PRIO("%[nfin]")                                                        \
    "s_branch .Lst_evdone_%=\n\t"                                             \
                                                                              \
    /* the lanes eIn of a group (F, 2c, index in vCF, vCC, vCI) finish */     \
    ".Lst_fin_%=:\n"                                                          \
    "s_bcnt1_i32_b64 s[eU], s[eIn:eIn+1]\n\t"                                 \
    "s_add_i32 %[nfin], %[nfin], s[eU]\n\t"                                   \
    "s_sub_i32 %[nA], %[nA], s[eU]\n\t"                                       \
    "s_mov_b32 %[tf], 0\n\t"                                                  \
    "s_mov_b64 exec, s[eIn:eIn+1]\n\t"                                        \
    "v_and_b32 v[vZ], 0xffff, v[vCI]\n\t"                                     \
    "v_lshlrev_b32 v[vZ], 2, v[vZ]\n\t"                                       \
    "v_mov_b32 v[vW], %[t]\n\t"                                               \
    "global_store_dword v[vZ], v[vW], %[fin]\n\t"                             \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_mov_b64 s[eX:eX+1], s[eIn:eIn+1]\n\t"                                  \
    ".Lst_fin1_%=:\n"                                                         \
    "s_ff1_i32_b64 s[eI], s[eX:eX+1]\n\t"                                     \
    "s_bitset0_b64 s[eX:eX+1], s[eI]\n\t"                                     \
    "v_readlane_b32 s[eCh], v[vCC], s[eI]\n\t"                                \
    "v_readlane_b32 s[eFa], v[vCF], s[eI]\n\t"                                \
    "s_ashr_i32 s[eCh], s[eCh], 1\n\t"                                        \
    "s_sub_i32 %[C], %[C], s[eCh]\n\t"                                        \
    /* (within its plan: it leaves the planned profile too) */                \
    "s_cmp_gt_i32 s[eFa], %[t]\n\t"                                           \
    "s_cbranch_scc0 .Lst_fin2_%=\n\t"                                         \
    "s_cmp_lg_u32 %[cur], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_fin2_%=\n\t"                                         \
    "s_call_b64 s[eRet2:eRet2+1], .Lst_del_%=\n\t"                            \
    ".Lst_fin2_%=:\n"                                                         \
    "s_cmp_lg_u64 s[eX:eX+1], 0\n\t"                                          \
    "s_cbranch_scc1 .Lst_fin1_%=\n\t"                                         \
    "s_setpc_b64 s[eRet:eRet+1]\n\t"                                          \
                                                                              \
    /* An entry with F = eFa and c = eCh leaves the list: the last lane q with that\
       F.  Those before q lose F + c, those from q on move down by one.  Of entries\
       with one F the first holds the sum over all of them, and that one is exact\
       and decides every check (a candidate with that te becomes the first).  The\
       others lose also what was never in them, without end while requests come\
       and go at one F: at -2^30 they stop, below any first (a sum of memory, not\
       negative) and far from wrapping in a check or by one more loss (F + c is a\
       request's size plus planned length, at most M). */                     \
    ".Lst_del_%=:\n"                                                          \
    "v_cmp_ge_i32 vcc, s[eFa], %[F]\n\t"                                      \
    "s_bcnt1_i32_b64 s[eP], vcc\n\t"                                          \
    "s_cmp_gt_u32 s[eP], 63\n\t"                                              \
    "s_cbranch_scc1 .Lst_deldeep_%=\n\t"                                      \
    ".Lst_delreg_%=:\n"                                                       \
    "s_add_i32 s[eP], s[eP], -1\n\t"                                          \
    "s_brev_b32 s[eV], -2\n\t"                                                \
    "s_brev_b32 s[eC1], -2\n\t"                                               \
    "s_cmp_gt_i32 %[ln1], 65\n\t"                                             \
    "s_cbranch_scc0 .Lst_del1_%=\n\t"                                         \
    "s_lshl3_add_u32 s[eU], %[ln1], %[pushb]\n\t"                             \
    "s_add_i32 s[eU], s[eU], -8\n\t"                                          \
    "v_mov_b32 v[vAd], s[eU]\n\t"                                             \
    "ds_read_b64 v[vZ:vZ+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_readfirstlane_b32 s[eV], v[vZ]\n\t"                                    \
    "v_readfirstlane_b32 s[eC1], v[vW]\n\t"                                   \
    ".Lst_del1_%=:\n"                                                         \
    "v_mov_b32_dpp v[vX], %[F] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"     \
    "v_mov_b32_dpp v[vY], %[G] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"     \
    "s_lshl_b64 s[eMk:eMk+1], -1, s[eP]\n\t"                                  \
    "v_add_u32 v[vAd], s[eCh], %[F]\n\t"                                      \
    "v_writelane_b32 v[vX], s[eV], 63\n\t"                                    \
    "v_writelane_b32 v[vY], s[eC1], 63\n\t"                                   \
    "v_sub_u32 v[vAd], %[G], v[vAd]\n\t"                                      \
    "v_max_i32 v[vAd], " ST_FLOOR ", v[vAd]\n\t"                              \
    "v_cndmask_b32 %[F], %[F], v[vX], s[eMk:eMk+1]\n\t"                       \
    "v_cndmask_b32 %[G], v[vAd], v[vY], s[eMk:eMk+1]\n\t"                     \
    "s_sub_i32 %[ln1], %[ln1], 1\n\t"                                         \
    "s_setpc_b64 s[eRet2:eRet2+1]\n\t"                                        \
    /* past the registers: find its group, then each group from there up moves down */\
    ".Lst_deldeep_%=:\n"                                                      \
    "s_add_i32 s[eW], %[ln1], -65\n\t"                                        \
    ".Lst_delf_%=:\n"                                                         \
    "s_lshl_b32 s[eU], s[eW], 3\n\t"                                          \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_cmp_ge_i32 vcc, s[eFa], v[vX]\n\t"                                     \
    "s_bcnt1_i32_b64 s[eP], vcc\n\t"                                          \
    "s_sub_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_cmp_gt_u32 s[eP], 63\n\t"                                              \
    "s_cbranch_scc1 .Lst_delf_%=\n\t"                                         \
    "s_add_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_cmp_lg_u32 s[eP], 0\n\t"                                               \
    "s_cbranch_scc1 .Lst_delg_%=\n\t"                                         \
    /* it is the last lane of the group before */                             \
    "s_mov_b32 s[eP], 64\n\t"                                                 \
    "s_add_i32 s[eU], %[ln1], -65\n\t"                                        \
    "s_cmp_eq_u32 s[eW], s[eU]\n\t"                                           \
    "s_cbranch_scc1 .Lst_delreg_%=\n\t"                                       \
    "s_add_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_lshl_b32 s[eU], s[eW], 3\n\t"                                          \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    ".Lst_delg_%=:\n"                                                         \
    "v_add_u32 v[vZ], s[eCh], %[F]\n\t"                                       \
    "v_sub_u32 %[G], %[G], v[vZ]\n\t"                                         \
    "v_max_i32 %[G], " ST_FLOOR ", %[G]\n\t"                                  \
    "v_add_u32 v[vZ], s[eCh], v[vX]\n\t"                                      \
    "v_sub_u32 v[vY], v[vY], v[vZ]\n\t"                                       \
    "v_max_i32 v[vY], " ST_FLOOR ", v[vY]\n\t"                                \
    "v_add_u32 v[vAd], -8, v[vAd]\n\t"                                        \
    "s_add_i32 s[eP], s[eP], -1\n\t"                                          \
    "s_bfm_b64 exec, s[eP], 0\n\t"                                            \
    "ds_write_b64 v[vAd], v[vX:vX+1]\n\t"                                     \
    "s_mov_b64 exec, -1\n\t"                                                  \
    ".Lst_delu_%=:\n"                                                         \
    "s_add_i32 s[eU], %[ln1], -65\n\t"                                        \
    "s_cmp_ge_i32 s[eW], s[eU]\n\t"                                           \
    "s_cbranch_scc1 .Lst_dele_%=\n\t"                                         \
    "s_add_i32 s[eW], s[eW], 64\n\t"                                          \
    "s_lshl_b32 s[eU], s[eW], 3\n\t"                                          \
    "v_add_u32 v[vAd], s[eU], %[rev]\n\t"                                     \
    "ds_read_b64 v[vX:vX+1], v[vAd]\n\t"                                      \
    "v_add_u32 v[vAd], -8, v[vAd]\n\t"                                        \
    "s_waitcnt lgkmcnt(0)\n\t"                                                \
    "v_add_u32 v[vZ], s[eCh], v[vX]\n\t"                                      \
    "v_sub_u32 v[vY], v[vY], v[vZ]\n\t"                                       \
    "v_max_i32 v[vY], " ST_FLOOR ", v[vY]\n\t"                                \
    "ds_write_b64 v[vAd], v[vX:vX+1]\n\t"                                     \
    "s_branch .Lst_delu_%=\n\t"                                               \
    ".Lst_dele_%=:\n"                                                         \
    "s_sub_i32 %[ln1], %[ln1], 1\n\t"                                         \
    "s_setpc_b64 s[eRet2:eRet2+1]\n\t"                                        \
                                                                              \
    /* Overflow of the true memory at t + 1: evict the largest believed remaining\
       volume (F' - t)(2c + F' + t + 1) / 2, F' = max(F, t + 1), latest index on */\
    /* ties, until it fits.  Staged admissions go out first: the victim's start and\
       admission number are taken back. */                                    \
    ".Lst_evict_%=:\n"                                                        \
    "s_cmp_eq_u32 %[nstg], 0\n\t"                                             \
    "s_cbranch_scc1 .Lst_evict1_%=\n\t"                                       \
    "s_bfm_b64 exec, %[nstg], 0\n\t"                                          \
    "v_lshlrev_b32 v[vZ], 2, %[sgi]\n\t"                                      \
    "v_add_u32 v[vW], %[seq], %[lane]\n\t"                                    \
    "global_store_dword v[vZ], %[sgt], %[start]\n\t"                          \
    "global_store_dword v[vZ], v[vW], %[adm]\n\t"                             \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_add_i32 %[seq], %[seq], %[nstg]\n\t"                                   \
    "s_mov_b32 %[nstg], 0\n\t"                                                \
    ".Lst_evict1_%=:\n"                                                       \
    REP(ST_VOLUME)                                                            \
    ".Lst_evict2_%=:\n"                                                       \
    "v_mov_b32 v[vM], 0\n\t"                                                  \
    REP(ST_LARGEST)                                                           \
    EV_REDUCE("v_max_u32_dpp", "vM")                                          \
    "v_readlane_b32 s[eFa], v[vM], 63\n\t"                                    \
    "s_mov_b32 s[eP], -1\n\t"                                                 \
    "s_nop 0\n\t"                                                             \
    REP(ST_VICTIM)                                                            \
    REP(ST_REMOVE)                                                            \
    ".Lst_gone_%=:\n"                                                         \
    "s_ashr_i32 s[eCh], s[eCh], 1\n\t"                                        \
    "s_sub_i32 %[C], %[C], s[eCh]\n\t"                                        \
    "s_sub_i32 %[nA], %[nA], 1\n\t"                                           \
    "s_lshr_b32 s[eR], s[eR], 16\n\t"                                         \
    "s_lshl_b32 s[eU], s[eP], 2\n\t"                                          \
    "s_mov_b64 exec, 1\n\t"                                                   \
    "v_mov_b32 v[vZ], s[eU]\n\t"                                              \
    "v_mov_b32 v[vW], -1\n\t"                                                 \
    "v_mov_b32 v[vX], 1\n\t"                                                  \
    "global_store_dword v[vZ], v[vW], %[start]\n\t"                           \
    "global_store_dword v[vZ], v[vW], %[adm]\n\t"                             \
    "global_atomic_add v[vZ], v[vX], %[pre]\n\t"                              \
    "s_cmp_lt_u32 %[nev], 64\n\t"                                             \
    "s_cbranch_scc1 .Lst_evreg_%=\n\t"                                        \
    "s_lshl_b32 s[eU], %[nev], 2\n\t"                                         \
    "v_mov_b32 v[vZ], s[eU]\n\t"                                              \
    "v_mov_b32 v[vW], s[eR]\n\t"                                              \
    "global_store_dword v[vZ], v[vW], %[evl]\n\t"                             \
    "s_branch .Lst_evput_%=\n\t"                                              \
    ".Lst_evreg_%=:\n"                                                        \
    "s_mov_b32 m0, %[nev]\n\t"                                                \
    "v_writelane_b32 v[vEv], s[eR], m0\n\t"                                   \
    ".Lst_evput_%=:\n"                                                        \
    "s_mov_b64 exec, -1\n\t"                                                  \
    "s_add_i32 %[nev], %[nev], 1\n\t"                                         \
    "s_mov_b32 %[tf], 0\n\t"                                                  \
    "s_mov_b32 s[eFa], s[eTe]\n\t"                                            \
    "s_cmp_gt_i32 s[eTe], %[t]\n\t"                                           \
    "s_cbranch_scc0 .Lst_evict3_%=\n\t"                                       \
    "s_cmp_lg_u32 %[cur], 0\n\t"                                              \
    "s_cbranch_scc1 .Lst_evict3_%=\n\t"                                       \
    "s_call_b64 s[eRet2:eRet2+1], .Lst_del_%=\n\t"                            \
    ".Lst_evict3_%=:\n"                                                       \
    "s_mul_i32 s[eMem], %[nA], s[eT1]\n\t"                                    \
    "s_add_i32 s[eMem], s[eMem], %[C]\n\t"                                    \
    "s_cmp_le_i32 s[eMem], %[M]\n\t"                                          \
    "s_cbranch_scc1 .Lst_evicted_%=\n\t"                                      \
    "s_cmp_eq_u32 %[nA], 0\n\t"                                               \
    "s_cbranch_scc1 .Lst_evicted_%=\n\t"                                      \
    "s_branch .Lst_evict2_%=\n\t"                                             \
                                                                              \
    ".Lst_drop_%=:\n"                                                         \
    "s_mov_b32 s[eU], %[dead]\n\t"                                            \
    EV_DROP                                                                   \
    "s_branch .Lst_evdone_%=\n\t"                                             \
    ".Lst_reload_%=:\n"                                                       \
    ST_RELOAD                                                                 \
    "s_branch .Lst_arr_%=\n\t"                                                \
    EV_DEEP                                                                   \
                                                                              \
    /* a full list, or all places of the running requests taken: the segment leaves\
       inside the admissions of step t */                                     \
    ".Lev_full_%=:\n"                                                         \
    "s_mov_b32 %[tf], -1\n\t"                                                 \
    CLOSE("g")                                                                \
    "v_lshlrev_b32 v[vAd], 2, %[lane]\n\t"                                    \
    "v_cmp_gt_i32 vcc, %[nev], %[lane]\n\t"                                   \
    "s_mov_b64 exec, vcc\n\t"                                                 \
    "global_store_dword v[vAd], v[vEv], %[evl]\n\t"                           \
    "s_mov_b64 exec, -1\n\t"                                                  \
    ".Lst_exit_%=:\n"                                                         \
    "s_mov_b32 s[eP], 0\n\t"                                                  \
    REP(ST_STOREU)                                                            \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t"                                       \
    "v_readfirstlane_b32 s[eU], v[vM0]\n\t"                                   \
    "s_mov_b32 m0, s[eU]\n\t"

#define ST_LOOP_1(E) ST_LOOP(ST_REP_##E, ST_PLACES_##E, EV_SET_1, EV_CLOSE_1, EV_EMPTY_1, EV_SCAN_1)
#define ST_LOOP_2(E) ST_LOOP(ST_REP_##E, ST_PLACES_##E, EV_SET_2, EV_CLOSE_2, EV_EMPTY_2, EV_SCAN_2)
#define ST_LOOP_0(E) ST_LOOP(ST_REP_##E, ST_PLACES_##E, EV_SET_0, EV_CLOSE_0, EV_EMPTY_0, EV_SCAN_0)

#define ST_STATE                                                              \
    [t] "+&s"(t), [head] "+&s"(head), [tf] "+&s"(t_f), [seq] "+&s"(seq),      \
    [nstg] "+&s"(nstg), [nfin] "+&s"(nfin), [nA] "+&s"(nA), [C] "+&s"(C),     \
    [nextev] "+&s"(next_ev), [rsl] "+&s"(rs_lo), [rsh] "+&s"(rs_hi),          \
    [peak] "+&s"(peak), [wb] "+&s"(wb), [pend] "+&s"(pend),                   \
    [ln1] "+&s"(ln1), [dead] "+&s"(L.dead), [nev] "+&s"(nev),                 \
    [last] "+&s"(prio.last), [F] "+&v"(L.F), [G] "+&v"(L.G),                  \
    [sgi] "+&v"(stg_idx), [sgt] "+&v"(stg_t)

#define ST_INPUT                                                              \
    [tstop] "s"(t_stop), [n1] "s"(n - 1), [M] "s"(P.M), [cap] "s"(L.cap),     \
    [pushb] "s"(stk - 65 * 8), [cur] "s"(cur), [places] "n"(64 * E),          \
    [rec] "s"(sg.rec), [rank] "s"(sg.rank), [arr] "s"(sg.a),                  \
    [start] "s"(sg.start), [adm] "s"(sg.admit_seq), [fin] "s"(sg.fin),        \
    [pre] "s"(sg.preempt), [evl] "s"(sg.evl), [act] "s"(sg.act),              \
    [ctr] "s"(prio.ctr), [th] "s"(prio.th), [lane] "v"(lane),                 \
    [vmin] "v"(INT32_MIN), [vmax] "v"(INT32_MAX), [rev] "v"(stk - 8 - 8 * lane)

// clang-format on
