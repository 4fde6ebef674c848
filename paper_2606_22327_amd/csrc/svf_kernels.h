// svf_kernels.h -- internal interface between the host runtime and the gfx950
// kernels of the batched scheduling simulator (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace svfk {

enum { POLICY_FCFS = 0, POLICY_SJF = 1, POLICY_SVF = 2, POLICY_SVF1BIT = 3 };
enum { ADMIT_CURRENT = 0x100 };  // added to a policy code: next-step admission
enum { STATUS_DONE = 0, STATUS_EXHAUSTED = 1, STATUS_RUNNING = 2 };

// Per-segment (instance x policy) simulation state, kept in HBM between launches.
struct SegState {
    int32_t t;          // next step to simulate
    int32_t cursor;     // next request (instance-local index) still to arrive
    int32_t seq;        // admissions so far
    int32_t status;     // STATUS_*
    int32_t nA;         // running requests (per-step path)
    int32_t nfin;       // finished (per-step path) / admitted (event path)
    int32_t max_fin;    // event path: latest scheduled finish
    int32_t head_rank;  // event path: blocked head (-1: none known)
    int32_t t_f;        // event path: the head cannot fit before this step
    int32_t N_O;        // per-step path: requests past their planned length
    int64_t C_O;        // per-step path: sum of (s - k) over those requests (k_sim_step: over all
                        //   running ones, modulo 2^32)
    int64_t peak;       // largest memory total over the steps folded so far
    int64_t req_steps;  // per-step path: sum over steps of running requests
    int32_t ln;         // with the list profile: its entries
    uint32_t lq;        //   and (k_sim_steplist) the prefix sum of (s - k) of the last entry
    int32_t resume_lim; // list full before step resume_lim: continue up to there (0: no)
    int32_t resume_nev; // per-step path: -1, or stopped in the admission phase of step t
                        //   with this many evictions of that step (ranks in evl)
};

// Same layout as svf_instance_stats of the public header.
struct StatsOut {
    int32_t makespan;
    int32_t status;
    int64_t sum_latency;
    int64_t request_steps;
    int64_t peak_mem;
    int64_t preemptions;
    int64_t t_end;
};

// Progress counters of one launch: one per cache line.
enum { PROG_LINES = 64, PROG_STRIDE = 16, PROG_WORDS = PROG_LINES * PROG_STRIDE };
// Behind the scratch of the no-allocation entry point: its two launches' progress counters.
enum { NOALLOC_PROG_BYTES = 2 * PROG_WORDS * 8 };

struct SortArgs {
    const int64_t* offsets;   // [I+1]
    const int32_t* a;         // [N]
    const int32_t* s;
    const int32_t* o;
    const int32_t* plan;      // [N] or null
    const int8_t* bit;        // [N] or null
    const int32_t* policies;  // [P] (device)
    const uint8_t* stepped;   // [G] 1: per-step path (its finishes and preemptions are cleared too)
    const int32_t* chunk_seg; // [nchunks] segment of each chunk
    const int32_t* chunk_lo;  // [nchunks] first rank position of each chunk
    const uint64_t* keys_in;  // [P*N]
    uint64_t* keys_out;       // [P*N]
    int4* rec;                // [P*N] rank-ordered {index, s, planned length, o}
    int32_t* rank;            // [P*N] index -> rank
    int32_t I, P;
    int64_t N;
    int32_t O0, O1;
    int32_t CH;
    int32_t kbits[8];         // [P] bits of the largest priority key of each policy
    int32_t* start;           // [P*N] outputs cleared by the fused sort (k_sort_rec)
    int32_t* fin;
    int32_t* preempt;
    int32_t* admit_seq;
    int32_t clear_all;        // 1: finishes and preemptions of event-path segments too
    SegState* st;             // [G] and the rest of a run's first state, written by the fused sort
    uint64_t* bitmap;         // [P*bw_total]
    const int64_t* bw_off;    // [I+1]
    int64_t bw_total;
    int32_t* ring;            // [G*(H+64)] or null
    int32_t H;
    unsigned long long* prog; // [2*PROG_WORDS]
};

// One launch copies arrays of n words (32 bits).
struct CopyArgs {
    const int32_t* src[4];
    int32_t* dst[4];
    int64_t n;
};

struct SimArgs {
    const int64_t* offsets;
    const int32_t* a;
    const int4* rec;
    const int32_t* rank;
    const uint8_t* stepped;   // [G] 1: per-step path (plans differ or next-step admission)
    const int32_t* policies;  // [P] policy codes
    const int64_t* bw_off;    // [I+1] bitmap word offset of each instance
    uint64_t* bitmap;         // [P*bw_total]
    int32_t* ring;            // [G*(H+64)] future profile plus step index (G = D + tau)
    int32_t* start;           // [P*N]
    int32_t* fin;
    int32_t* preempt;
    int32_t* admit_seq;
    int4* act;                // [P*N] or null: running list, record of each entry
    int2* actkr;              // [P*N] or null: running list, {start step, rank}
    int32_t* evl;             // [P*N] or null
    SegState* st;             // [G]
    int32_t I, P;
    int64_t N;
    int64_t bw_total;
    int32_t bw_max;           // largest bitmap size of one instance (words)
    int32_t H;                // ring length (power of two)
    int32_t M;
    int32_t max_steps;
    int64_t step_delta;       // steps to simulate in this launch
    int32_t* lst_f;           // [G*list_stride] list profile: planned finishes
    uint32_t* lst_q;          // [G*list_stride]   and D(F) + F (event path) or prefix sums of s - k
    int32_t list_stride;      // entries per segment in HBM (bound on concurrent requests)
    int32_t list_cap;         // entries per segment in this launch (in LDS and registers)
    int32_t list_nb;          // event path: bitmap pairs in registers (0: bitmap in LDS)
    int32_t step_regs;        // per-step path: its running requests in registers (k_sim_step)
    int32_t list_resume;      // not 0: only continue the segments that stopped with a full list
                              //   (per-step path in registers: 1 with STEP_E_MID, 2 with STEP_E_FULL)
    int32_t prio;             // 1: the waves set their issue priorities
    unsigned long long* prog; // [PROG_WORDS] progress counters of this launch, zero before it (and after
                              //   it: every wave takes back what it added)
};

struct FinArgs {
    const int64_t* offsets;
    const int32_t* a;
    const int32_t* o;
    const uint8_t* stepped;
    const int32_t* start;
    const int32_t* fin;
    const int32_t* preempt;
    const SegState* st;
    int32_t* fin_out;
    StatsOut* stats;
    int32_t I, P;
    int64_t N;
};

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s);
hipError_t launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s);
hipError_t launch_init_ring(int32_t* ring, int64_t n, int32_t H, hipStream_t s);
hipError_t launch_copy4(const CopyArgs& C, int arrays, hipStream_t s);
hipError_t launch_init_state(SegState* st, int32_t G, hipStream_t s);
hipError_t launch_chunk_sort(const SortArgs& A, int nchunks, hipStream_t s);
hipError_t launch_merge_pass(const SortArgs& A, int nchunks, int w, hipStream_t s);
hipError_t launch_build_rec(const SortArgs& A, int nchunks, hipStream_t s);
// Instances of at most SORT_REC_MAX requests: keys, stable radix sort, records,
// ranks and cleared outputs in one kernel, one workgroup per segment.
enum { SORT_REC_MAX = 8192 };
hipError_t prepare_sort_rec(int max_n);
hipError_t launch_sort_rec(const SortArgs& A, int G, int max_n, hipStream_t s);
hipError_t prepare_sim(bool d_lds, size_t lds_ring, bool step_list, size_t lds_step);
// per-step path: entries of LDS the finish-ordered list of capacity cap takes (F and Q each)
__host__ __device__ inline int list_slots(int cap) { return cap + 65; }
// Event path: the register form of the kernel for instances of at most max_n
// requests, the LDS of a list of capacity cap besides the bitmap, the finished
// entries that may wait at its front, and its kernels.
inline int list_bitmap_pairs(int max_n) { return max_n <= 4096 ? 1 : (max_n <= 8192 ? 2 : 0); }
inline size_t list_lds(int64_t cap) { return (size_t)(64 + (cap > 64 ? cap - 64 : 0)) * 8; }
enum { LIST_DEAD_MAX = 32 };
hipError_t prepare_list(int nb, size_t lds_first, size_t lds_full);
// resident waves per compute unit of its first launch
hipError_t list_occupancy(int nb, size_t lds_bytes, int* blocks);
// The per-step path with its running requests in registers: places of the
// first launch and of its two continuations (64 each), and what it assumes of a
// batch: the bound on running requests below its places, indexes and ranks in
// 16 bits, the factors of a remaining volume in 24 bits, twice a volume in 32.
enum { STEP_E = 6, STEP_E_MID = 10, STEP_E_FULL = 32 };
inline bool step_regs_ok(int64_t bound, int64_t max_n, int64_t M, uint64_t max_volume) {
    return bound < 64 * STEP_E_FULL && max_n <= 65536 && M < (1 << 23) - 1 &&
           max_volume < (uint64_t(1) << 31);
}
// step: 0 the first launch, 1 and 2 the continuations (SimArgs::list_resume)
hipError_t prepare_step(int nb, const size_t lds[3]);
hipError_t step_occupancy(int nb, size_t lds_bytes, int* blocks);
// list: the event path keeps its profile as the finish-ordered list
hipError_t launch_sim(const SimArgs& P, int G, bool d_lds, bool stepped, bool list,
                      size_t lds_bytes, hipStream_t s);
// resident waves per compute unit of the per-step kernel with the list
hipError_t sim_step_occupancy(size_t lds_bytes, int* blocks);
hipError_t launch_finalize(const FinArgs& F, int G, hipStream_t s);
// Device address and size of the calling thread's current device's scratch
// array of the no-allocation entry point (svf_noalloc.hip); NOALLOC_PROG_BYTES
// more follow it.
hipError_t noalloc_scratch(void** addr, size_t* bytes);

}  // namespace svfk
