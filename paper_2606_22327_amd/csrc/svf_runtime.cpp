// svf_runtime.cpp -- host side of the C ABI declared in include/svfsim.h:
// validation, buffer ownership, launch configuration, timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

#include "svf_kernels.h"
#include "svfsim.h"

using svfk::SegState;
using svfk::StatsOut;

static_assert(sizeof(StatsOut) == sizeof(svf_instance_stats), "stats layout");
static_assert(sizeof(SegState) == 80, "state layout");

namespace {

// message of the calling thread's last failure (a fixed buffer: no call
// allocates host memory for it)
thread_local char g_err[512];

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

int ok() { return SVF_OK; }

constexpr int64_t kLimit30 = int64_t(1) << 30;

int64_t next_pow2(int64_t x) {
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

struct Timed {
    int kind;  // 0 init, 1 sim, 2 final
    hipEvent_t a, b;
};

}  // namespace

struct svf_batch {
    hipStream_t stream = nullptr;
    // Second stream (default priority) on which the per-step segments run
    // concurrently with the event-driven ones, forked from and joined back
    // into ``stream`` with events; null: both launches on ``stream``.
    hipStream_t aux = nullptr;
    hipEvent_t fork_ev = nullptr, join_ev = nullptr;
    int device = 0;
    int32_t I = 0, P = 0;
    int64_t N = 0;
    int32_t M = 0, O0 = 0, O1 = 0, max_steps = 0;
    std::vector<int32_t> policies;
    int32_t H = 1, CH = 64, nchunks = 0, bw_max = 0, max_n = 0;
    bool fused_sort = false;  // every instance fits one workgroup of k_sort_rec
    bool list_known = false;  // event path: profile as the finish-ordered list
    bool ring_used = true;    // some segment keeps its profile in the ring
    int32_t list_stride = 0;  // list entries per segment in HBM (the bound)
    int32_t list_cap = 0;     // event path: list entries per segment (first launch)
    int32_t list_full = 0;    //   and with room for the bound (continuation)
    int32_t list_nb = 0;      // event path: bitmap pairs in registers (0: in LDS)
    size_t lds_list = 0;      // LDS of the event kernel with the list
    size_t lds_list_full = 0; //   and with room for the bound (continuation)
    bool list_stepped = false; // per-step path: profile as the finish-ordered list
    bool step_regs = false;    //   and its running requests in registers
    int32_t step_full = 0;     // its entries with room for the bound (continuation)
    int32_t step_cap = 0;      // its entries in LDS (first launch)
    int32_t step_mid = 0;      //   and in the first continuation (requests in registers)
    size_t lds_step = 0;       // LDS of the per-step kernel with the list
    size_t lds_step_full = 0;  //   and with room for the bound (continuation)
    size_t lds_step_mid = 0;   //   and in the first continuation
    bool prio = false;         // the first launch of each path sets issue priorities
    int32_t kbits[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int64_t bw_total = 0;
    bool d_lds = true;
    size_t lds_bytes = 0;
    bool any_stepped = false;
    int64_t n_known = 0, n_stepped = 0;
    bool was_reset = false, dirty = false;
    bool cleared = false;     // a reset outside of stream capture cleared every output
    bool prof = false;
    std::vector<Timed> timed;
    double acc_ms[3] = {0, 0, 0};
    int64_t sim_launches = 0;

    // device buffers, all in one allocation
    void* arena = nullptr;
    char* pinned = nullptr;   // host staging of large reads (READ_SLOTS * READ_SLOT bytes)
    int32_t* d_pack = nullptr; // [4*N] outputs of one slot side by side (small batches)
    int64_t* d_off = nullptr;
    int32_t *d_a = nullptr, *d_s = nullptr, *d_o = nullptr, *d_plan = nullptr;
    int8_t* d_bit = nullptr;
    int32_t* d_pol = nullptr;
    int32_t *d_chunk_seg = nullptr, *d_chunk_lo = nullptr;
    uint64_t *d_keys0 = nullptr, *d_keys1 = nullptr;
    int4* d_rec = nullptr;
    int32_t* d_rank = nullptr;
    uint8_t* d_stepped = nullptr;
    int64_t* d_bw_off = nullptr;
    uint64_t* d_bitmap = nullptr;
    int32_t* d_ring = nullptr;
    int32_t *d_start = nullptr, *d_fin = nullptr, *d_pre = nullptr, *d_seq = nullptr;
    int4* d_act = nullptr;
    int2* d_actkr = nullptr;
    int32_t* d_evl = nullptr;
    SegState* d_st = nullptr;
    int32_t* d_fin_out = nullptr;
    StatsOut* d_stats = nullptr;
    int32_t* d_lst_f = nullptr;
    uint32_t* d_lst_q = nullptr;
    unsigned long long* d_prog = nullptr;  // [2 * PROG_WORDS] progress counters of the simulation launches
};

namespace {

void free_all(svf_batch* h) {
    if (h->arena) (void)hipFree(h->arena);
    if (h->pinned) (void)hipHostFree(h->pinned);
    h->arena = nullptr;
    h->pinned = nullptr;
    for (auto& t : h->timed) {
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    h->timed.clear();
    if (h->fork_ev) (void)hipEventDestroy(h->fork_ev);
    if (h->join_ev) (void)hipEventDestroy(h->join_ev);
    if (h->aux) (void)hipStreamDestroy(h->aux);
    h->fork_ev = h->join_ev = nullptr;
    h->aux = nullptr;
}

#define HIPCHK(expr)                                                                  \
    do {                                                                              \
        hipError_t e_ = (expr);                                                       \
        if (e_ != hipSuccess)                                                         \
            return fail(SVF_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));     \
    } while (0)

#define RETCHK(expr)              \
    do {                          \
        int r_ = (expr);          \
        if (r_ != SVF_OK) return r_; \
    } while (0)

struct HostView {
    const int32_t *a, *s, *o, *plan;
    const int8_t* bit;
};

// Host threads for work on n items (1: in the calling thread only).
int threads_for(int64_t n) {
    if (n < (int64_t(1) << 20)) return 1;
    return (int)std::max(1u, std::min(8u, std::thread::hardware_concurrency()));
}

// f(0) .. f(count - 1), each on a thread of its own while threads can be had.
template <typename F>
void on_threads(int count, F f) {
    std::vector<std::thread> pool;
    int k = 1;
    try {
        pool.reserve((size_t)std::max(count, 1));
        for (; k < count; ++k) pool.emplace_back(f, k);
    } catch (const std::exception&) {
        // no further thread: the rest runs here
    }
    f(0);
    for (; k < count; ++k) f(k);
    for (std::thread& t : pool) t.join();
}

// What the launch plan needs to know of the requests.
struct Facts {
    int64_t max_plan = 1;     // longest planned length
    int64_t max_profile = 0;  // largest planned memory total at one future step
    uint64_t max_key[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // each policy's largest key
    int64_t bound = 0;        // most requests of one instance that can run at once
    int64_t sum_s = 0, sum_o = 0;
    int32_t max_s = 1;
    int32_t bad = INT32_MAX;  // first instance with an error
};

// Facts of one instance's requests under one source of planned lengths.
struct Lengths {
    bool differ = false;  // some planned length is not the true one
    int32_t longest = 0;
    int64_t sum = 0;
    uint64_t volume = 0;
};

// One instance in straight passes the compiler turns into vector code; true if
// anything is wrong with it.  volumes: whether the volumes are needed as keys.
__attribute__((always_inline)) inline bool scan_core(
    const int32_t* a, const int32_t* s, const int32_t* o, const int32_t* plan, const int8_t* bit,
    int64_t n, const int32_t O[2], uint32_t M, bool use_plan, bool use_bit, bool volumes, Facts& F,
    Lengths L[2]) {
    uint32_t bad = 0;
    for (int64_t j = 0; j < n; ++j) bad |= (uint32_t)a[j] >> 30;
    for (int64_t j = 1; j < n; ++j) bad |= (uint32_t)(a[j] < a[j - 1]);
    int64_t sum_s = 0, sum_o = 0;
    int32_t max_s = 1;
    for (int64_t j = 0; j < n; ++j) {
        bad |= (uint32_t)(s[j] < 1) | (uint32_t)(o[j] < 1);
        sum_s += s[j];
        sum_o += o[j];
        max_s = std::max(max_s, s[j]);
    }
    F.sum_s += sum_s;
    F.sum_o += sum_o;
    F.max_s = std::max(F.max_s, max_s);
    if (plan)
        for (int64_t j = 0; j < n; ++j) bad |= (uint32_t)(plan[j] < 1);
    if (bit)
        for (int64_t j = 0; j < n; ++j) bad |= (uint32_t)bit[j] & ~1u;
    auto lengths = [&](auto of, Lengths& out) {
        uint32_t differ = 0;
        int32_t longest = 0;
        int64_t sum = 0;
        for (int64_t j = 0; j < n; ++j) {
            const int32_t l = of(j);
            differ |= (uint32_t)(l ^ o[j]);
            longest = std::max(longest, l);
            sum += l;
            // (values below 1 are errors already: no wrap among the others)
            bad |= (uint32_t)((uint32_t)s[j] + (uint32_t)std::max(o[j], l) > M);
        }
        if (volumes) {
            uint64_t most = 0;
            for (int64_t j = 0; j < n; ++j) {
                const uint64_t l = (uint32_t)of(j);
                most = std::max(most, (uint64_t)(uint32_t)s[j] * l + ((l * l + l) >> 1));
            }
            out.volume = most;
        }
        out.differ = differ != 0;
        out.longest = longest;
        out.sum = sum;
    };
    if (use_plan) {
        if (plan) lengths([&](int64_t j) { return plan[j]; }, L[0]);
        else lengths([&](int64_t j) { return o[j]; }, L[0]);
    }
    if (use_bit && bit) lengths([&](int64_t j) { return bit[j] ? O[1] : O[0]; }, L[1]);
    return bad != 0;
}

typedef bool (*ScanFn)(const int32_t*, const int32_t*, const int32_t*, const int32_t*, const int8_t*,
                       int64_t, const int32_t*, uint32_t, bool, bool, bool, Facts&, Lengths*);
bool scan_any(const int32_t* a, const int32_t* s, const int32_t* o, const int32_t* plan,
              const int8_t* bit, int64_t n, const int32_t* O, uint32_t M, bool up, bool ub, bool vol,
              Facts& F, Lengths* L) {
    return scan_core(a, s, o, plan, bit, n, O, M, up, ub, vol, F, L);
}
__attribute__((target("avx2"))) bool scan_avx2(const int32_t* a, const int32_t* s, const int32_t* o,
                                               const int32_t* plan, const int8_t* bit, int64_t n,
                                               const int32_t* O, uint32_t M, bool up, bool ub,
                                               bool vol, Facts& F, Lengths* L) {
    return scan_core(a, s, o, plan, bit, n, O, M, up, ub, vol, F, L);
}

// Largest number of requests of one instance that can run at the same time, if
// it is above ``best``.  A running request holds at least s + 1 tokens at the
// next step, and the planned (and true) total of that step stays <= M once a
// step's admissions are done, so at most the k smallest values of s + 1 fit.
// Values at or above kCap count as kCap (a lower bound on each), which keeps k
// an upper bound.  h: counts per value, all zero before and after.
constexpr int kCap = 4096;
int64_t running_bound(const int32_t* s, int64_t n, int64_t sum_s, int64_t M, int64_t best, int32_t* h) {
    if (n <= best) return best;
    if (sum_s + n <= M) return n;
    auto value = [&](int64_t j) { return (int)std::min<int64_t>((int64_t)s[j] + 1, kCap); };
    for (int64_t j = 0; j < n; ++j) h[value(j)] += 1;
    int64_t sum = 0, k = 0;
    for (int v = 1; v <= kCap; ++v) {
        if (!h[v]) continue;
        const int64_t take = std::min<int64_t>(h[v], (M - sum) / v);
        k += take;
        sum += take * v;
        if (take < h[v]) break;
    }
    if (n < kCap / 4) for (int64_t j = 0; j < n; ++j) h[value(j)] = 0;
    else std::fill(h, h + kCap + 1, 0);
    return std::max(best, k);
}

// The instances [lo, hi): their facts into F (up to the first with an error),
// each segment's path (1: per-step) to stepped[P*I].
void scan(const svf_batch_desc* d, const HostView& v, const int64_t* off, int32_t lo, int32_t hi,
          uint8_t* stepped, Facts& F) {
    const int32_t I = d->num_instances, P = d->num_policies;
    bool use_plan = false, use_bit = false, volumes = false;
    for (int p = 0; p < P; ++p) {
        const int pol = d->policies[p] & 0xFF;
        (pol == SVF_POLICY_SVF1BIT ? use_bit : use_plan) = true;
        volumes |= pol == SVF_POLICY_SVF || pol == SVF_POLICY_SVF1BIT;
    }
    const int32_t O[2] = {d->O0, d->O1};
    const ScanFn fn = __builtin_cpu_supports("avx2") ? &scan_avx2 : &scan_any;
    int32_t h[kCap + 1];
    std::fill(h, h + kCap + 1, 0);
    F.max_profile = d->M;
    for (int32_t i = lo; i < hi; ++i) {
        const int64_t x = off[i], n = off[i + 1] - x;
        if (n == 0) {
            for (int p = 0; p < P; ++p) stepped[(size_t)p * I + i] = 0;
            continue;
        }
        Lengths L[2];
        const int64_t before = F.sum_s;
        bool bad = fn(v.a + x, v.s + x, v.o + x, v.plan ? v.plan + x : nullptr,
                      v.bit ? v.bit + x : nullptr, n, O, (uint32_t)d->M, use_plan, use_bit, volumes, F, L);
        const int64_t sum_s = F.sum_s - before;
        for (int p = 0; p < P; ++p) {
            const int pol = d->policies[p] & 0xFF;
            const bool current_rule = (d->policies[p] & SVF_ADMIT_CURRENT) != 0;
            const Lengths& l = L[pol == SVF_POLICY_SVF1BIT];
            uint64_t key;
            if (pol == SVF_POLICY_FCFS) key = (uint64_t)(uint32_t)v.a[x + n - 1];
            else if (pol == SVF_POLICY_SJF) key = (uint64_t)(uint32_t)l.longest;
            else key = l.volume;
            bad |= key >= (uint64_t(1) << 32);
            F.max_key[p] = std::max(F.max_key[p], key);
            // eviction is only possible when plans differ from the truth
            // or when admission looks at the next step only
            stepped[(size_t)p * I + i] = l.differ || current_rule;
            F.max_plan = std::max<int64_t>(F.max_plan, l.longest);
            // The forward-looking check keeps a step's planned total <= M;
            // with next-step admission only, the requests of an instance
            // bound it together: sum of s + o^.
            if (current_rule) F.max_profile = std::max(F.max_profile, sum_s + l.sum);
        }
        if (bad) {
            F.bad = i;
            return;
        }
        F.bound = running_bound(v.s + x, n, sum_s, d->M, F.bound, h);
    }
}

// The first error among the requests of instance i, as a message.
int first_error(const svf_batch_desc* d, const HostView& v, const int64_t* off, int32_t i) {
    const int32_t P = d->num_policies;
    const int64_t lo = off[i], hi = off[i + 1];
    for (int64_t j = lo; j < hi; ++j) {
        const int32_t a = v.a[j], s = v.s[j], o = v.o[j];
        if (a < 0 || a >= kLimit30)
            return fail(SVF_EINVAL, "instance %d request %lld: arrival %d out of [0, 2^30)", i,
                        (long long)(j - lo), a);
        if (j > lo && a < v.a[j - 1])
            return fail(SVF_EINVAL, "instance %d: arrivals not in order at request %lld", i,
                        (long long)(j - lo));
        if (s < 1) return fail(SVF_EINVAL, "instance %d request %lld: prompt %d < 1", i, (long long)(j - lo), s);
        if (o < 1) return fail(SVF_EINVAL, "instance %d request %lld: output %d < 1", i, (long long)(j - lo), o);
        if (v.plan && v.plan[j] < 1)
            return fail(SVF_EINVAL, "instance %d request %lld: plan_len %d < 1", i, (long long)(j - lo), v.plan[j]);
        if (v.bit && v.bit[j] != 0 && v.bit[j] != 1)
            return fail(SVF_EINVAL, "instance %d request %lld: long_bit %d not 0/1", i, (long long)(j - lo), v.bit[j]);
        for (int p = 0; p < P; ++p) {
            const int pol = d->policies[p] & 0xFF;
            int64_t oh;
            if (pol == SVF_POLICY_SVF1BIT) oh = v.bit[j] ? d->O1 : d->O0;
            else oh = v.plan ? v.plan[j] : o;
            if ((int64_t)s + std::max<int64_t>(o, oh) > d->M)
                return fail(SVF_EINFEASIBLE,
                            "instance %d request %lld: s + max(o, planned) = %lld exceeds M = %lld",
                            i, (long long)(j - lo), (long long)s + std::max<int64_t>(o, oh),
                            (long long)d->M);
            uint64_t key;
            if (pol == SVF_POLICY_FCFS) key = (uint64_t)a;
            else if (pol == SVF_POLICY_SJF) key = (uint64_t)oh;
            else key = (uint64_t)s * (uint64_t)oh + (((uint64_t)oh * oh + oh) >> 1);
            if (key >= (uint64_t(1) << 32))
                return fail(SVF_EINVAL, "instance %d request %lld: priority key %llu >= 2^32", i,
                            (long long)(j - lo), (unsigned long long)key);
        }
    }
    return fail(SVF_EINVAL, "instance %d: malformed requests", i);
}

// Everything that can be checked without a GPU, and the facts for the launch
// plan, on ``threads`` host threads (1: none is started, nothing is allocated).
int validate(const svf_batch_desc* d, const HostView& v, const int64_t* off, int64_t N,
             uint8_t* stepped, int threads, Facts* facts) {
    const int32_t I = d->num_instances, P = d->num_policies;
    bool has1bit = false;
    for (int p = 0; p < P; ++p) has1bit |= (d->policies[p] & 0xFF) == SVF_POLICY_SVF1BIT;
    if (N > 0 && (!v.a || !v.s || !v.o))
        return fail(SVF_EINVAL, "arrival, prompt and output must not be NULL");
    if (has1bit && N > 0 && !v.bit) return fail(SVF_EINVAL, "SVF1BIT needs long_bit");
    if (has1bit && (d->O0 < 1 || d->O1 < 1)) return fail(SVF_EINVAL, "SVF1BIT needs O0, O1 >= 1");
    Facts part[8];
    threads = std::max(1, std::min({threads, 8, (int)std::max(I, 1)}));
    auto work = [&](int k) {
        // the instances whose first request is in the k-th share of all requests
        auto cut = [&](int x) {
            if (x == 0) return (int32_t)0;
            if (x == threads) return I;
            return (int32_t)(std::lower_bound(off, off + I, N * x / threads) - off);
        };
        scan(d, v, off, cut(k), cut(k + 1), stepped, part[k]);
    };
    if (threads == 1) work(0);
    else on_threads(threads, work);
    Facts& F = *facts;
    F = part[0];
    for (int k = 1; k < threads; ++k) {
        const Facts& x = part[k];
        F.max_plan = std::max(F.max_plan, x.max_plan);
        F.max_profile = std::max(F.max_profile, x.max_profile);
        for (int p = 0; p < 8; ++p) F.max_key[p] = std::max(F.max_key[p], x.max_key[p]);
        F.bound = std::max(F.bound, x.bound);
        F.sum_s += x.sum_s;
        F.sum_o += x.sum_o;
        F.max_s = std::max(F.max_s, x.max_s);
        F.bad = std::min(F.bad, x.bad);
    }
    return F.bad == INT32_MAX ? SVF_OK : first_error(d, v, off, F.bad);
}

int check_desc_shape(const svf_batch_desc* d, int64_t* N) {
    if (!d) return fail(SVF_EINVAL, "desc is NULL");
    if (d->num_instances < 0) return fail(SVF_EINVAL, "num_instances < 0");
    if (!d->req_offsets) return fail(SVF_EINVAL, "req_offsets is NULL");
    if (d->num_policies < 1 || d->num_policies > 8)
        return fail(SVF_EINVAL, "num_policies must be in 1..8 (got %d)", d->num_policies);
    if (!d->policies) return fail(SVF_EINVAL, "policies is NULL");
    for (int p = 0; p < d->num_policies; ++p) {
        const int base = d->policies[p] & 0xFF, rule = d->policies[p] & ~0xFF;
        if (base < SVF_POLICY_FCFS || base > SVF_POLICY_SVF1BIT ||
            (rule != SVF_ADMIT_LOOKAHEAD && rule != SVF_ADMIT_CURRENT))
            return fail(SVF_EINVAL, "unknown policy %d", d->policies[p]);
    }
    if (d->M < 1 || d->M >= kLimit30) return fail(SVF_EINVAL, "M must be in [1, 2^30)");
    if (d->max_steps < 0 || d->max_steps >= kLimit30)
        return fail(SVF_EINVAL, "max_steps must be in [0, 2^30)");
    const int64_t* off = d->req_offsets;
    if (off[0] != 0) return fail(SVF_EINVAL, "req_offsets[0] must be 0");
    for (int32_t i = 0; i < d->num_instances; ++i) {
        const int64_t n = off[i + 1] - off[i];
        if (n < 0) return fail(SVF_EINVAL, "req_offsets decreases at instance %d", i);
        if (n >= (int64_t(1) << 31) - 1)
            return fail(SVF_EINVAL, "instance %d holds too many requests", i);
    }
    *N = off[d->num_instances];
    if (*N * (int64_t)d->num_policies >= (int64_t(1) << 31))
        return fail(SVF_EINVAL, "requests x policies must stay below 2^31");
    return SVF_OK;
}

// Largest LDS of a workgroup at which the kernel keeps the waves that its
// registers allow (those it reaches with ``least`` bytes).  For the kernels
// that keep the bitmap in registers (nb > 0) that is a constant of the kernel,
// found once.  0 without a GPU.
template <typename Occ>
size_t full_occupancy_lds(int kind, int nb, size_t least, Occ occ) {
    static std::atomic<size_t> known[2][3];
    const bool keep = kind < 2 && nb > 0;
    if (keep) {
        const size_t b = known[kind][nb].load(std::memory_order_relaxed);
        if (b) return b;
    }
    const int top = occ(least);
    if (top <= 0) return 0;
    size_t lo = least, hi = std::max<size_t>(least, 160 * 1024);
    while (hi - lo > 64) {
        const size_t mid = (lo + (hi - lo) / 2) & ~size_t(7);
        if (occ(mid) >= top) lo = mid;
        else hi = mid;
    }
    if (keep) known[kind][nb].store(lo, std::memory_order_relaxed);
    return lo;
}

// The launch plan of a validated batch: sizes, sort shape, profile kind
// (ring or finish-ordered list) and its LDS capacity per path, issue
// priorities.  Fills the host fields of ``h`` (not its buffers) and the
// bitmap word offsets bw_off[I+1].
int plan_batch(svf_batch* h, const svf_batch_desc* d, const int64_t* off,
               const uint8_t* stepped, const Facts& F, int64_t* bw_off) {
    const int32_t I = d->num_instances, P = d->num_policies;
    const int64_t N = off[I];
    h->I = I; h->P = P; h->N = N;
    h->M = (int32_t)d->M;
    h->O0 = d->O0; h->O1 = d->O1;
    h->max_steps = (int32_t)d->max_steps;
    const int64_t max_plan = F.max_plan, max_profile = F.max_profile;
    h->H = (int32_t)next_pow2(std::max<int64_t>(max_plan, 1));
    for (int32_t i = 0; i < I; ++i) h->max_n = std::max<int32_t>(h->max_n, (int32_t)(off[i + 1] - off[i]));
    h->CH = (int32_t)std::min<int64_t>(8192, std::max<int64_t>(64, next_pow2(h->max_n)));
    h->fused_sort = h->max_n <= svfk::SORT_REC_MAX;
    for (int32_t p = 0; p < P; ++p)
        h->kbits[p] = F.max_key[p] ? 64 - __builtin_clzll(F.max_key[p]) : 0;
    for (int64_t g = 0; g < (int64_t)P * I; ++g) {
        h->any_stepped |= stepped[g] != 0;
        (stepped[g] ? h->n_stepped : h->n_known) += 1;
    }
    // the profile ring stores memory + step index in int32
    if (max_profile + h->max_steps + 2 * (int64_t)h->H >= (int64_t(1) << 31) - 1)
        return fail(SVF_EINVAL, "M (or, under SVF_ADMIT_CURRENT, an instance's sum of s + planned "
                                "length) + max_steps + 2 * (longest planned length, rounded up to "
                                "a power of two) must stay below 2^31");

    // bitmap word offsets of the instances
    bw_off[0] = 0;
    for (int32_t i = 0; i < I; ++i) {
        const int64_t n = off[i + 1] - off[i];
        const int64_t W0 = (n + 63) / 64, W1 = (W0 + 63) / 64;
        bw_off[i + 1] = bw_off[i] + W0 + W1;
        h->bw_max = std::max<int32_t>(h->bw_max, (int32_t)(W0 + W1));
    }
    h->bw_total = bw_off[I];

    // ring placement: LDS when the ring and bitmap fit comfortably
    const char* env = getenv("SVFSIM_RING");
    const size_t ring_bytes = ((size_t)h->H + 64) * 4;  // H slots + spare slot
    const size_t bm_bytes = (size_t)h->bw_max * 8;
    h->d_lds = ring_bytes + bm_bytes <= 65536;
    if (env && !strcmp(env, "global")) h->d_lds = false;
    if (env && !strcmp(env, "lds") && ring_bytes + bm_bytes <= 160 * 1024) h->d_lds = true;
    h->lds_bytes = std::max<size_t>(8, bm_bytes + (h->d_lds ? ring_bytes : 0));
    // The event path keeps its profile as the finish-ordered list (8 bytes
    // per running request past the 64 in registers) when the ring does not fit
    // in LDS, or when few requests run at once: the list's checks and
    // insertions touch the running requests that finish before the candidate,
    // the ring's the candidate's whole planned length.  The estimate e = M /
    // (mean s + mean o / 2) is compared with 512.  Measured, simulation in ms,
    // list against ring: lengths to 2,048, 3 x 4096 x 1000 (e 140) 1.7 against
    // 4.2; lengths to 4,096, 16384 x 5000 (e 280) 11.1 against 59, 8,192
    // instances e 500 1.0 against 6.0, e 1000 2.2 against 11.5; lengths of 50
    // to 300, 8,192 instances e 350 1.35 against 1.75, e 550 2.5 against 1.9,
    // 64 instances e 150 0.61 against 0.63, e 450 0.74 against 0.57; lengths to
    // 8,192, mean 400, 64 x 200,000 (e 930) 412 against 159.  So 512 is right
    // for many instances of short requests, high for few of them and low for
    // long requests: the lengths are not in the rule.  The list gets the largest
    // capacity that still lets as many waves reside as the list kernel's
    // registers allow; segments that outgrow it stop, and a second launch with
    // room for the bound on concurrent requests (and for finished entries not
    // yet removed) continues them.
    const int64_t bound = std::max<int64_t>(1, F.bound);
    const size_t full_bytes = bm_bytes + (size_t)svfk::list_slots((int)std::min<int64_t>(bound, 1 << 24)) * 8;
    h->list_nb = svfk::list_bitmap_pairs(h->max_n);
    const size_t lds_bm = h->list_nb == 0 ? bm_bytes : 0;  // of the kernels that may keep the bitmap in registers
    if (h->n_known > 0) {
        const char* pe = getenv("SVFSIM_PROFILE");
        bool use = false;
        h->list_full = (int32_t)std::min<int64_t>(bound + svfk::LIST_DEAD_MAX, 1 << 24);
        h->lds_list_full = lds_bm + svfk::list_lds(h->list_full);
        int64_t cap = h->list_full;
        const bool fits = h->lds_list_full <= 160 * 1024;
        if (fits) {
            auto occ = [&](size_t bytes) {
                int w = 0;
                return svfk::list_occupancy(h->list_nb, bytes, &w) == hipSuccess ? w : -1;
            };
            const size_t most = full_occupancy_lds(0, h->list_nb, lds_bm + svfk::list_lds(64), occ);
            cap = std::min<int64_t>(cap, std::max<int64_t>(64, (int64_t)((most - std::min(most, lds_bm)) / 8)));
            const char* pc = getenv("SVFSIM_LIST_LDS_CAP");  // testing: a smaller list
            if (pc && atoll(pc) > 0) cap = std::min<int64_t>(cap, atoll(pc));
            const double running =
                N > 0 ? (double)d->M / (((double)F.sum_s + 0.5 * (double)F.sum_o) / (double)N) : 0.0;
            if (most > 0) use = !h->d_lds || running <= 512.0;
        }
        if (pe && !strcmp(pe, "ring")) use = false;
        if (pe && !strcmp(pe, "list")) use = fits;
        if (use) {
            h->list_known = true;
            h->list_cap = (int32_t)cap;
            h->lds_list = lds_bm + svfk::list_lds(cap);
        }
    }
    // The per-step path keeps its planned profile as the finish-ordered list
    // when the list with room for the bound fits in 64 KB of LDS.  As on the
    // event path, the first launch gives it the largest capacity that keeps
    // the kernel at the occupancy its registers allow, and a continuation
    // launch has room for the bound.
    if (h->any_stepped) {
        const char* ps = getenv("SVFSIM_STEP_PROFILE");
        bool use = full_bytes <= 64 * 1024;
        if (ps && !strcmp(ps, "ring")) use = false;
        if (ps && !strcmp(ps, "list")) use = full_bytes <= 160 * 1024;
        if (use) {
            // its running requests in registers, within that kernel's limits
            const uint64_t L = (uint64_t)max_plan;  // (no volume is larger than this one)
            h->step_regs = svfk::step_regs_ok(bound, h->max_n, d->M,
                                              (uint64_t)F.max_s * L + ((L * L + L) >> 1));
            h->step_full = (int32_t)(bound + (h->step_regs ? svfk::LIST_DEAD_MAX : 0));
            auto bytes = [&](int64_t c) {
                return h->step_regs ? lds_bm + svfk::list_lds(c)
                                    : bm_bytes + (size_t)svfk::list_slots((int)c) * 8;
            };
            auto occ = [&](size_t b) {
                int w = 0;
                return (h->step_regs ? svfk::step_occupancy(h->list_nb, b, &w)
                                     : svfk::sim_step_occupancy(b, &w)) == hipSuccess ? w : -1;
            };
            const size_t most = full_occupancy_lds(h->step_regs ? 1 : 2, h->step_regs ? h->list_nb : 0,
                                                   bytes(64), occ);
            int64_t cap = h->step_full;
            if (most > 0) {
                const size_t front = h->step_regs ? lds_bm : bm_bytes + (size_t)svfk::list_slots(0) * 8;
                cap = std::min<int64_t>(cap, std::max<int64_t>(64, (int64_t)((most - std::min(most, front)) / 8)));
            }
            const char* pc = getenv("SVFSIM_STEP_LDS_CAP");  // testing: a smaller list
            if (pc && atoll(pc) > 0) cap = std::min<int64_t>(cap, atoll(pc));
            h->list_stepped = true;
            h->step_cap = (int32_t)cap;
            h->lds_step = bytes(cap);
            h->lds_step_full = bytes(h->step_full);
            if (h->step_regs) {
                // (every planned entry is of a running request)
                h->step_mid = std::min<int32_t>(h->step_full, 64 * svfk::STEP_E_MID + svfk::LIST_DEAD_MAX);
                h->lds_step_mid = bytes(h->step_mid);
            }
        }
    }
    if (h->list_known || h->list_stepped) h->list_stride = (int32_t)bound;
    h->ring_used = (h->n_known > 0 && !h->list_known) || (h->any_stepped && !h->list_stepped);
    // The waves of the first simulation launch of each path set their issue
    // priorities (timing only).
    // With at most one segment per SIMD (four per CU) there is nothing to
    // arbitrate.  Measured, on against off, simulation in ms: heavy traffic 300
    // to 768 instances equal, 1,024 (if they were on there) 3.41 against 3.51,
    // 2,048 3.76 against 4.01, 16,384 11.1 against 12.6; planned with
    // predicted lengths 63.2 against 64.6, under next-step admission 141
    // against 149; Poisson 3 x 4,096 x 1,000 1.65 against 1.70, with 1-bit SVF
    // 3.47 against 3.52.
    {
        int ncu = 0;
        const char* pp = getenv("SVFSIM_ISSUE_PRIO");  // "0": all waves at one priority
        const bool on = !(pp && !strcmp(pp, "0"));
        h->prio = on && hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, h->device) == hipSuccess &&
                  ncu > 0 && (int64_t)P * I > 4 * (int64_t)ncu;
        (void)hipGetLastError();
    }
    if (h->lds_bytes > 160 * 1024)
        return fail(SVF_EINVAL, "an instance's rank bitmap needs %zu bytes of LDS (> 160 KB)", h->lds_bytes);

    return SVF_OK;
}

void record(svf_batch* h, int kind, hipEvent_t* a) {
    if (!h->prof) return;
    (void)hipEventCreate(a);
    (void)hipEventRecord(*a, h->stream);
    (void)kind;
}

void record_end(svf_batch* h, int kind, hipEvent_t a) {
    if (!h->prof) return;
    hipEvent_t b;
    (void)hipEventCreate(&b);
    (void)hipEventRecord(b, h->stream);
    h->timed.push_back({kind, a, b});
}

constexpr int32_t RING_BY_SORT = 1 << 14;

int do_reset(svf_batch* h) {
    const int32_t G = h->P * h->I;
    const int64_t PN = (int64_t)h->P * h->N;
    hipEvent_t e0 = nullptr;
    record(h, 0, &e0);
    svfk::SortArgs A{};
    A.offsets = h->d_off;
    A.a = h->d_a; A.s = h->d_s; A.o = h->d_o; A.plan = h->d_plan; A.bit = h->d_bit;
    A.policies = h->d_pol;
    A.chunk_seg = h->d_chunk_seg;
    A.chunk_lo = h->d_chunk_lo;
    A.rec = h->d_rec;
    A.rank = h->d_rank;
    A.I = h->I; A.P = h->P; A.N = h->N; A.O0 = h->O0; A.O1 = h->O1; A.CH = h->CH;
    for (int p = 0; p < 8; ++p) A.kbits[p] = h->kbits[p];
    A.start = h->d_start; A.fin = h->d_fin; A.preempt = h->d_pre; A.admit_seq = h->d_seq;
    A.stepped = h->d_stepped;
    // Finishes and preemption counts of event-path segments are never written:
    // cleared once, by the first reset that runs (one recorded into a graph
    // may not, and one whose launch fails does not).
    A.clear_all = !h->cleared;
    bool runs = false;
    if (!h->cleared) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(h->stream, &cs) != hipSuccess) (void)hipGetLastError();
        else runs = cs == hipStreamCaptureStatusNone;
    }
    A.st = h->d_st;
    A.bitmap = h->d_bitmap;
    A.bw_off = h->d_bw_off;
    A.bw_total = h->bw_total;
    // Short rings are written by the sort's workgroup of their segment, long
    // ones (per-step batches with the ring in global memory) by a launch of
    // their own over the whole GPU: one workgroup took 70 us for 2^17 slots
    // and 744 for 2^22 where the launch takes 54 and 59, the sort included.
    const bool long_ring = h->ring_used && h->H > RING_BY_SORT;
    A.ring = h->ring_used && !long_ring ? h->d_ring : nullptr;
    A.H = h->H;
    A.prog = h->d_prog;
    if (h->fused_sort) {
        if (long_ring)
            HIPCHK(svfk::launch_init_ring(h->d_ring, (int64_t)G * (h->H + 64), h->H, h->stream));
        // keys, sort, records, ranks, cleared outputs and the first state in one kernel
        HIPCHK(svfk::launch_sort_rec(A, G, h->max_n, h->stream));
        h->cleared |= runs;
        record_end(h, 0, e0);
        h->was_reset = true;
        h->dirty = true;
        return SVF_OK;
    }
    HIPCHK(svfk::launch_init_state(h->d_st, G, h->stream));
    HIPCHK(svfk::launch_fill_u64(h->d_bitmap, (int64_t)h->P * h->bw_total, 0ull, h->stream));
    HIPCHK(svfk::launch_fill_u64(reinterpret_cast<uint64_t*>(h->d_prog), 2 * svfk::PROG_WORDS, 0ull, h->stream));
    if (h->ring_used)
        HIPCHK(svfk::launch_init_ring(h->d_ring, (int64_t)G * (h->H + 64), h->H, h->stream));
    HIPCHK(svfk::launch_fill_i32(h->d_start, PN, -1, h->stream));
    HIPCHK(svfk::launch_fill_i32(h->d_fin, PN, -1, h->stream));
    HIPCHK(svfk::launch_fill_i32(h->d_pre, PN, 0, h->stream));
    HIPCHK(svfk::launch_fill_i32(h->d_seq, PN, -1, h->stream));
    if (PN > 0) {
        A.keys_in = nullptr;
        A.keys_out = h->d_keys0;
        HIPCHK(svfk::launch_chunk_sort(A, h->nchunks, h->stream));
        uint64_t* cur = h->d_keys0;
        uint64_t* other = h->d_keys1;
        for (int64_t w = h->CH; w < h->max_n; w *= 2) {
            A.keys_in = cur;
            A.keys_out = other;
            HIPCHK(svfk::launch_merge_pass(A, h->nchunks, (int)w, h->stream));
            std::swap(cur, other);
        }
        A.keys_in = cur;
        A.keys_out = nullptr;
        HIPCHK(svfk::launch_build_rec(A, h->nchunks, h->stream));
    }
    record_end(h, 0, e0);
    h->was_reset = true;
    h->dirty = true;
    return SVF_OK;
}

int do_sim(svf_batch* h, int64_t delta) {
    const int32_t G = h->P * h->I;
    if (G <= 0) return SVF_OK;
    svfk::SimArgs S{};
    S.offsets = h->d_off;
    S.a = h->d_a;
    S.rec = h->d_rec;
    S.rank = h->d_rank;
    S.stepped = h->d_stepped;
    S.policies = h->d_pol;
    S.bw_off = h->d_bw_off;
    S.bitmap = h->d_bitmap;
    S.ring = h->d_ring;
    S.start = h->d_start;
    S.fin = h->d_fin;
    S.preempt = h->d_pre;
    S.admit_seq = h->d_seq;
    S.act = h->d_act;
    S.actkr = h->d_actkr;
    S.evl = h->d_evl;
    S.st = h->d_st;
    S.I = h->I; S.P = h->P; S.N = h->N;
    S.bw_total = h->bw_total;
    S.bw_max = h->bw_max;
    S.H = h->H;
    S.M = h->M;
    S.max_steps = h->max_steps;
    S.step_delta = delta;
    S.lst_f = h->d_lst_f;
    S.lst_q = h->d_lst_q;
    S.list_stride = h->list_stride;
    S.list_cap = h->list_cap;
    S.list_nb = h->list_nb;
    S.step_regs = h->step_regs;
    S.list_resume = 0;
    S.prio = h->prio;
    S.prog = h->d_prog;
    hipEvent_t e0 = nullptr;
    record(h, 1, &e0);
    // The two paths simulate disjoint segments (each kernel leaves the other
    // path's segments alone) and keep separate progress counters, so with
    // segments on both the event-driven launch runs on the second stream,
    // concurrently with the per-step one.  The per-step launch (long serial
    // segments at low occupancy) goes first, on the caller's stream, so that
    // its waves are resident from the start; the event-driven waves fill the
    // remaining slots.
    const bool fork = h->aux && h->n_known > 0 && h->n_stepped > 0;
    const hipStream_t st_stepped = h->stream;
    hipStream_t st_known = h->stream;
    if (fork) {
        HIPCHK(hipEventRecord(h->fork_ev, h->stream));
        HIPCHK(hipStreamWaitEvent(h->aux, h->fork_ev, 0));
        st_known = h->aux;
    }
    // launch errors are kept until the second stream has been joined back
    hipError_t le = hipSuccess;
    if (h->n_stepped > 0) {
        svfk::SimArgs T = S;
        T.list_cap = h->step_cap;
        T.list_resume = 0;
        T.prog = h->d_prog + svfk::PROG_WORDS;
        le = svfk::launch_sim(T, G, h->d_lds, true, h->list_stepped,
                              h->list_stepped ? h->lds_step : h->lds_bytes, st_stepped);
        if (le == hipSuccess && h->list_stepped &&
            (h->step_cap < h->step_full || (h->step_regs && h->list_stride >= 64 * svfk::STEP_E))) {
            // Segments whose list outgrew the LDS capacity (or whose running
            // requests the registers: with every place taken a segment stops
            // at the next candidate, fit or not), up to the same step.  With
            // the running requests in registers first those of at most
            // 64 STEP_E_MID, at five waves per SIMD and a third of the places
            // to scan, then the others, at two.  Measured, 16384 x 5000 under
            // next-step admission (little more than 384 run at once there):
            // 225 ms with the large form alone, 140 ms with both.
            T.prio = 0;
            if (h->step_regs) {
                T.list_cap = h->step_mid;
                T.list_resume = 1;
                le = svfk::launch_sim(T, G, false, true, true, h->lds_step_mid, st_stepped);
            }
            if (le == hipSuccess && (!h->step_regs || h->list_stride >= 64 * svfk::STEP_E_MID)) {
                T.list_cap = h->step_full;
                T.list_resume = h->step_regs ? 2 : 1;
                le = svfk::launch_sim(T, G, false, true, true, h->lds_step_full, st_stepped);
            }
        }
    }
    if (le == hipSuccess && h->n_known > 0) {
        le = svfk::launch_sim(S, G, h->d_lds, false, h->list_known,
                              h->list_known ? h->lds_list : h->lds_bytes, st_known);
        if (le == hipSuccess && h->list_known && h->list_cap < h->list_full) {
            // segments whose list outgrew the LDS capacity, up to the same step
            S.list_cap = h->list_full;
            S.list_resume = 1;
            S.prio = 0;
            le = svfk::launch_sim(S, G, false, false, true, h->lds_list_full, st_known);
        }
    }
    if (fork) {
        HIPCHK(hipEventRecord(h->join_ev, h->aux));
        HIPCHK(hipStreamWaitEvent(h->stream, h->join_ev, 0));
    }
    if (le != hipSuccess)
        return fail(SVF_EHIP, "simulation launch failed: %s", hipGetErrorString(le));
    record_end(h, 1, e0);
    h->sim_launches += 1;
    h->dirty = true;
    return SVF_OK;
}

int do_finalize(svf_batch* h) {
    if (!h->dirty) return SVF_OK;
    const int32_t G = h->P * h->I;
    svfk::FinArgs F{};
    F.offsets = h->d_off;
    F.a = h->d_a;
    F.o = h->d_o;
    F.stepped = h->d_stepped;
    F.start = h->d_start;
    F.fin = h->d_fin;
    F.preempt = h->d_pre;
    F.st = h->d_st;
    F.fin_out = h->d_fin_out;
    F.stats = h->d_stats;
    F.I = h->I; F.P = h->P; F.N = h->N;
    hipEvent_t e0 = nullptr;
    record(h, 2, &e0);
    HIPCHK(svfk::launch_finalize(F, G, h->stream));
    record_end(h, 2, e0);
    h->dirty = false;
    return SVF_OK;
}

// A kernel on ``device`` may store ``bytes`` of words at p: memory of that
// device (another device's, or host memory, is left to the runtime's copy),
// word-aligned, all of it in p's allocation (one that is too short is left to
// the runtime, whose copy refuses it).
bool kernel_writable(const void* p, size_t bytes, int device) {
    hipPointerAttribute_t at;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&at, p) != hipSuccess ||
        hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const uintptr_t at_p = reinterpret_cast<uintptr_t>(p);
    return at.type == hipMemoryTypeDevice && at.device == device && (at_p & 3) == 0 &&
           at_p + bytes <= reinterpret_cast<uintptr_t>(base) + size;
}

// p is memory of the runtime's (page-locked, managed): it copies there directly.
bool known_to_runtime(const void* p) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type != hipMemoryTypeUnregistered;
}

// Sequential placement of buffers in a fixed device region (256-byte
// aligned); ``used`` may exceed the region, and is checked before any use.
struct Carve {
    uintptr_t base;  // 0: only the size is wanted
    size_t used;
    template <typename T>
    T* take(int64_t count) {
        if (count <= 0) return nullptr;
        used = (used + 255) & ~size_t(255);
        T* p = reinterpret_cast<T*>(base + used);
        used += sizeof(T) * (size_t)count;
        return p;
    }
};

// Host tables of svf_run_noalloc (per-segment path flags, bitmap word
// offsets, small inputs on their way up), static so that the call allocates nothing; guarded by g_na_mu.
std::mutex g_na_mu;
uint8_t g_na_stepped[(size_t)SVF_NOALLOC_MAX_INSTANCES * 8];
int64_t g_na_bw_off[SVF_NOALLOC_MAX_INSTANCES + 1];
char g_na_stage[256 << 10];

hipError_t prepare_step(const svf_batch* h) {
    const size_t lds[3] = {h->lds_step, h->lds_step_mid, h->lds_step_full};
    return svfk::prepare_step(h->list_nb, lds);
}

struct Destroy {
    void operator()(svf_batch* h) const {
        free_all(h);
        delete h;
    }
};

// Reads of at least READ_LARGE bytes into ordinary memory go through pinned
// staging, READ_SLOTS slots of READ_SLOT bytes, a host thread per slot: the
// copies out of the GPU run at the link's rate beside the stores into the
// caller's pages (which are often touched there for the first time).  Measured,
// four arrays into fresh pages, one pageable copy each against this, the first
// read of a handle (it pins the slots) and later ones: 8.5 MB 510 against 420
// and 380 us, 80 MB 6.1 against 2.5 and 2.1 ms; 2 to 4 MB of one array, 160 to
// 260 against 270 to 300 and 180 to 230 us: below 8 MB the copies stay.
// Page-locked destinations take no part: their one copy each runs at the
// link's rate (9.6 MB 0.21 ms, through the slots 0.42).
constexpr int READ_SLOTS = 8;
constexpr size_t READ_SLOT = size_t(2) << 20, READ_LARGE = size_t(8) << 20;
// Batches whose outputs of one slot take at most this are read in one copy.
constexpr size_t READ_SMALL = size_t(256) << 10;
// Host inputs and tables up to this size go up in one copy.
constexpr size_t STAGE_MAX = size_t(1) << 20;

int create(const svf_batch_desc* d, void* hip_stream, svf_batch** out) {
    int64_t N = 0;
    RETCHK(check_desc_shape(d, &N));
    const int32_t I = d->num_instances, P = d->num_policies;
    const int64_t* off = d->req_offsets;
    const int64_t G = (int64_t)P * I;
    const int64_t PN = (int64_t)P * N;

    // host view of the per-request arrays (device inputs are fetched first)
    std::unique_ptr<int32_t[]> ha, hs, ho, hp;
    std::unique_ptr<int8_t[]> hb;
    HostView v{d->arrival, d->prompt, d->output, d->plan_len, d->long_bit};
    if (d->inputs_on_device && N > 0) {
        if (!d->arrival || !d->prompt || !d->output)
            return fail(SVF_EINVAL, "arrival, prompt and output must not be NULL");
        auto fetch = [&](auto& buf, const auto* src) {
            typedef typename std::remove_const<typename std::remove_reference<decltype(*src)>::type>::type T;
            buf.reset(new T[(size_t)N]);
            return hipMemcpy(buf.get(), src, sizeof(T) * (size_t)N, hipMemcpyDeviceToHost);
        };
        HIPCHK(fetch(ha, d->arrival));
        HIPCHK(fetch(hs, d->prompt));
        HIPCHK(fetch(ho, d->output));
        if (d->plan_len) HIPCHK(fetch(hp, d->plan_len));
        if (d->long_bit) HIPCHK(fetch(hb, d->long_bit));
        v = HostView{ha.get(), hs.get(), ho.get(), hp.get(), hb.get()};
    }
    std::vector<uint8_t> stepped((size_t)G);
    std::vector<int64_t> bw_off((size_t)I + 1, 0);
    Facts facts;
    RETCHK(validate(d, v, off, N, stepped.data(), threads_for(N), &facts));

    std::unique_ptr<svf_batch, Destroy> own(new svf_batch());
    svf_batch* h = own.get();
    h->stream = (hipStream_t)hip_stream;
    (void)hipGetDevice(&h->device);
    RETCHK(plan_batch(h, d, off, stepped.data(), facts, bw_off.data()));
    // chunk table (segment, first position) of the sort for large instances
    std::vector<int32_t> cseg, clo;
    if (!h->fused_sort)
        for (int32_t p = 0; p < P; ++p)
            for (int32_t i = 0; i < I; ++i)
                for (int64_t lo = 0; lo < off[i + 1] - off[i]; lo += h->CH) {
                    cseg.push_back(p * I + i);
                    clo.push_back((int32_t)lo);
                }
    h->nchunks = (int32_t)cseg.size();

    // one allocation, the host's tables and the inputs first
    size_t tables = 0, inputs = 0;
    auto place = [&](Carve c) {
        h->d_off = c.take<int64_t>(I + 1);
        h->d_pol = c.take<int32_t>(P);
        h->d_stepped = c.take<uint8_t>(G);
        h->d_bw_off = c.take<int64_t>(I + 1);
        h->d_chunk_seg = c.take<int32_t>(h->nchunks);
        h->d_chunk_lo = c.take<int32_t>(h->nchunks);
        tables = c.used;
        h->d_a = c.take<int32_t>(N);
        h->d_s = c.take<int32_t>(N);
        h->d_o = c.take<int32_t>(N);
        if (d->plan_len) h->d_plan = c.take<int32_t>(N);
        if (d->long_bit) h->d_bit = c.take<int8_t>(N);
        inputs = c.used;
        if (!h->fused_sort) {
            h->d_keys0 = c.take<uint64_t>(PN);
            h->d_keys1 = c.take<uint64_t>(PN);
        }
        h->d_rec = c.take<int4>(PN);
        h->d_rank = c.take<int32_t>(PN);
        h->d_bitmap = c.take<uint64_t>((int64_t)P * h->bw_total);
        if (h->ring_used) h->d_ring = c.take<int32_t>(G * (h->H + 64));
        if (h->list_known || h->list_stepped) {
            h->d_lst_f = c.take<int32_t>(G * (int64_t)h->list_stride);
            h->d_lst_q = c.take<uint32_t>(G * (int64_t)h->list_stride);
        }
        h->d_start = c.take<int32_t>(PN);
        h->d_fin = c.take<int32_t>(PN);
        h->d_pre = c.take<int32_t>(PN);
        h->d_seq = c.take<int32_t>(PN);
        if (h->any_stepped) {
            h->d_act = c.take<int4>(PN);
            if (!h->step_regs) h->d_actkr = c.take<int2>(PN);
            h->d_evl = c.take<int32_t>(PN);
        }
        h->d_st = c.take<SegState>(G);
        h->d_prog = c.take<unsigned long long>(2 * svfk::PROG_WORDS);
        h->d_fin_out = c.take<int32_t>(PN);
        h->d_stats = c.take<StatsOut>(G);
        if (16 * (size_t)N <= READ_SMALL) h->d_pack = c.take<int32_t>(4 * N);
        return c.used;
    };
    const size_t total = place(Carve{0, 0});
    if (hipError_t e = hipMalloc(&h->arena, total); e != hipSuccess) {
        h->arena = nullptr;
        return fail(SVF_ENOMEM, "hipMalloc of %lld bytes failed: %s", (long long)total, hipGetErrorString(e));
    }
    const uintptr_t base = reinterpret_cast<uintptr_t>(h->arena);
    place(Carve{base, 0});
    h->policies.assign(d->policies, d->policies + P);

    // the host's tables in one copy, small host inputs with them
    const bool together = !d->inputs_on_device && inputs <= STAGE_MAX;
    const size_t front = together ? inputs : tables;
    std::unique_ptr<char[]> stage(new char[front]);
    auto put = [&](const void* dev, const void* src, size_t bytes) {
        if (dev && bytes) memcpy(stage.get() + (reinterpret_cast<uintptr_t>(dev) - base), src, bytes);
    };
    put(h->d_off, off, 8 * ((size_t)I + 1));
    put(h->d_pol, h->policies.data(), 4 * (size_t)P);
    put(h->d_stepped, stepped.data(), (size_t)G);
    put(h->d_bw_off, bw_off.data(), 8 * ((size_t)I + 1));
    put(h->d_chunk_seg, cseg.data(), 4 * cseg.size());
    put(h->d_chunk_lo, clo.data(), 4 * clo.size());
    hipError_t e = hipSuccess;
    if (together) {
        put(h->d_a, d->arrival, 4 * (size_t)N);
        put(h->d_s, d->prompt, 4 * (size_t)N);
        put(h->d_o, d->output, 4 * (size_t)N);
        put(h->d_plan, d->plan_len, 4 * (size_t)N);
        put(h->d_bit, d->long_bit, (size_t)N);
    }
    e = hipMemcpyAsync(h->arena, stage.get(), front, hipMemcpyHostToDevice, h->stream);
    if (!together) {
        const hipMemcpyKind kind = d->inputs_on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
        auto copy = [&](void* dev, const void* src, size_t bytes) {
            if (e == hipSuccess && dev && bytes) e = hipMemcpyAsync(dev, src, bytes, kind, h->stream);
        };
        copy(h->d_a, d->arrival, 4 * (size_t)N);
        copy(h->d_s, d->prompt, 4 * (size_t)N);
        copy(h->d_o, d->output, 4 * (size_t)N);
        if (d->plan_len) copy(h->d_plan, d->plan_len, 4 * (size_t)N);
        if (d->long_bit) copy(h->d_bit, d->long_bit, (size_t)N);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e == hipSuccess)
        e = svfk::prepare_sim(h->d_lds, h->lds_bytes, h->list_stepped && !h->step_regs, h->lds_step_full);
    if (e == hipSuccess && h->step_regs) e = prepare_step(h);
    if (e == hipSuccess && h->list_known) e = svfk::prepare_list(h->list_nb, h->lds_list, h->lds_list_full);
    if (e == hipSuccess && h->fused_sort) e = svfk::prepare_sort_rec(h->max_n);
    // both paths in one batch: a second stream for the per-step launches
    // (SVFSIM_CONCURRENT=0 keeps them on one stream)
    const char* pc = getenv("SVFSIM_CONCURRENT");
    if (e == hipSuccess && h->n_known > 0 && h->n_stepped > 0 && !(pc && !strcmp(pc, "0"))) {
        e = hipStreamCreateWithFlags(&h->aux, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&h->fork_ev, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&h->join_ev, hipEventDisableTiming);
    }
    if (e != hipSuccess) return fail(SVF_EHIP, "copying the inputs failed: %s", hipGetErrorString(e));
    *out = own.release();
    return ok();
}

// A large read: src[k] to dst[k], ``bytes`` each (dst[k] null: skipped), in
// slots over host threads.  The stream's earlier work is waited for here, in
// the calling thread: hipStreamPerThread names another stream in each of the
// others.  The caller's current device stays what it was.
int read_large(svf_batch* h, const int32_t* const src[4], int32_t* const dst[4], size_t bytes) {
    HIPCHK(hipStreamSynchronize(h->stream));
    int current = h->device;
    HIPCHK(hipGetDevice(&current));
    const int64_t per = (int64_t)((bytes + READ_SLOT - 1) / READ_SLOT);
    std::atomic<int64_t> next{0};
    std::atomic<int> err{0};
    const int threads = std::max(1, std::min(READ_SLOTS, threads_for(int64_t(1) << 20)));
    on_threads(threads, [&](int k) {
        char* slot = h->pinned + (size_t)k * READ_SLOT;
        hipEvent_t ev = nullptr;
        hipError_t e = hipSetDevice(h->device);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        while (e == hipSuccess) {
            const int64_t c = next.fetch_add(1);
            if (c >= 4 * per) break;
            const int x = (int)(c / per);
            if (!dst[x]) continue;
            const size_t at = (size_t)(c % per) * READ_SLOT, n = std::min(READ_SLOT, bytes - at);
            const char* from = reinterpret_cast<const char*>(src[x]) + at;
            e = hipMemcpyAsync(slot, from, n, hipMemcpyDeviceToHost, h->stream);
            if (e == hipSuccess) e = hipEventRecord(ev, h->stream);
            if (e == hipSuccess) e = hipEventSynchronize(ev);
            if (e == hipSuccess) memcpy(reinterpret_cast<char*>(dst[x]) + at, slot, n);
        }
        if (ev) (void)hipEventDestroy(ev);
        if (e != hipSuccess) err = (int)e;
    });
    (void)hipSetDevice(current);
    if (err) return fail(SVF_EHIP, "reading the outputs failed: %s", hipGetErrorString((hipError_t)err.load()));
    return SVF_OK;
}

}  // namespace

extern "C" {

const char* svf_last_error(void) { return g_err; }

int svf_abi_version(void) { return SVFSIM_ABI_VERSION; }

int svf_create(const svf_batch_desc* d, void* hip_stream, svf_batch** out) {
    g_err[0] = 0;
    if (!out) return fail(SVF_EINVAL, "out is NULL");
    *out = nullptr;
    try {
        return create(d, hip_stream, out);
    } catch (const std::exception&) {
        return fail(SVF_ENOMEM, "host allocation failed");
    }
}

int svf_reset(svf_batch* h) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    return do_reset(h);
}

int svf_step(svf_batch* h, int64_t nsteps) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    if (nsteps < 0) return fail(SVF_EINVAL, "nsteps < 0");
    if (!h->was_reset) RETCHK(do_reset(h));
    // nsteps == 0 still launches: instances that are already complete at their
    // current step (e.g. empty ones) get their final status
    return do_sim(h, std::min<int64_t>(nsteps, int64_t(1) << 40));
}

int svf_run(svf_batch* h) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    if (!h->was_reset) RETCHK(do_reset(h));
    return do_sim(h, int64_t(1) << 40);
}

int svf_read(svf_batch* h, int32_t slot, int32_t* start, int32_t* finish, int32_t* preempt,
             int32_t* admit_seq, int32_t outputs_on_device) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    if (slot < 0 || slot >= h->P) return fail(SVF_EINVAL, "policy slot %d out of range", slot);
    if (!h->was_reset) return fail(SVF_ESTATE, "nothing simulated yet (call svf_reset/svf_run)");
    RETCHK(do_finalize(h));
    const int64_t base = (int64_t)slot * h->N;
    const size_t bytes = 4 * (size_t)h->N;
    const hipMemcpyKind k = hipMemcpyDeviceToHost;
    if (outputs_on_device) {
        svfk::CopyArgs C{};
        C.n = h->N;
        int arrays = 0;
        const int32_t* const src[4] = {h->d_start, h->d_fin_out, h->d_pre, h->d_seq};
        int32_t* const dst[4] = {start, finish, preempt, admit_seq};
        for (int x = 0; x < 4; ++x) {
            if (!dst[x]) continue;
            if (kernel_writable(dst[x], bytes, h->device)) {
                C.src[arrays] = src[x] + base;
                C.dst[arrays++] = dst[x];
            } else if (bytes) {
                HIPCHK(hipMemcpyAsync(dst[x], src[x] + base, bytes, hipMemcpyDeviceToDevice, h->stream));
            }
        }
        HIPCHK(svfk::launch_copy4(C, arrays, h->stream));
        return ok();
    }
    const int32_t* const src[4] = {h->d_start + base, h->d_fin_out + base, h->d_pre + base, h->d_seq + base};
    int32_t* dst[4] = {start, finish, preempt, admit_seq};
    // Page-locked destinations need no staging: one copy each.
    int wanted = 0;
    for (int x = 0; x < 4; ++x) {
        if (!dst[x]) continue;
        if (bytes && known_to_runtime(dst[x])) {
            HIPCHK(hipMemcpyAsync(dst[x], src[x], bytes, k, h->stream));
            dst[x] = nullptr;
        } else {
            ++wanted;
        }
    }
    if (bytes && wanted > 1 && h->d_pack) {
        // side by side on the device, then one copy
        svfk::CopyArgs C{};
        C.n = h->N;
        int arrays = 0;
        for (int x = 0; x < 4; ++x)
            if (dst[x]) {
                C.src[arrays] = src[x];
                C.dst[arrays] = h->d_pack + (int64_t)arrays * h->N;
                ++arrays;
            }
        std::unique_ptr<char[]> host(new (std::nothrow) char[bytes * 4]);
        if (!host) return fail(SVF_ENOMEM, "host allocation failed");
        HIPCHK(svfk::launch_copy4(C, arrays, h->stream));
        HIPCHK(hipMemcpyAsync(host.get(), h->d_pack, bytes * arrays, k, h->stream));
        HIPCHK(hipStreamSynchronize(h->stream));
        arrays = 0;
        for (int x = 0; x < 4; ++x)
            if (dst[x]) memcpy(dst[x], host.get() + bytes * arrays++, bytes);
        return ok();
    }
    if (bytes * wanted >= READ_LARGE && !h->pinned &&
        hipHostMalloc((void**)&h->pinned, READ_SLOTS * READ_SLOT, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        h->pinned = nullptr;
    }
    if (bytes * wanted >= READ_LARGE && h->pinned) {
        try {
            return read_large(h, src, dst, bytes);
        } catch (const std::exception&) {
            return fail(SVF_ENOMEM, "host allocation failed");
        }
    }
    for (int x = 0; x < 4; ++x)
        if (bytes && dst[x]) HIPCHK(hipMemcpyAsync(dst[x], src[x], bytes, k, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    return ok();
}

int svf_stats(svf_batch* h, int32_t slot, svf_instance_stats* out) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    if (slot < 0 || slot >= h->P) return fail(SVF_EINVAL, "policy slot %d out of range", slot);
    if (!out && h->I > 0) return fail(SVF_EINVAL, "out is NULL");
    if (!h->was_reset) return fail(SVF_ESTATE, "nothing simulated yet (call svf_reset/svf_run)");
    RETCHK(do_finalize(h));
    if (h->I > 0)
        HIPCHK(hipMemcpyAsync(out, h->d_stats + (int64_t)slot * h->I,
                              sizeof(svf_instance_stats) * h->I, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    return ok();
}

int svf_set_profiling(svf_batch* h, int32_t enable) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    HIPCHK(hipStreamSynchronize(h->stream));
    for (auto& t : h->timed) {
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    h->timed.clear();
    h->acc_ms[0] = h->acc_ms[1] = h->acc_ms[2] = 0;
    h->sim_launches = 0;
    h->prof = enable != 0;
    return ok();
}

int svf_timings(svf_batch* h, svf_timing* out) {
    if (!h || !out) return fail(SVF_EINVAL, "NULL argument");
    HIPCHK(hipStreamSynchronize(h->stream));
    for (auto& t : h->timed) {
        float ms = 0;
        HIPCHK(hipEventElapsedTime(&ms, t.a, t.b));
        h->acc_ms[t.kind] += ms;
        (void)hipEventDestroy(t.a);
        (void)hipEventDestroy(t.b);
    }
    h->timed.clear();
    out->init_ms = h->acc_ms[0];
    out->sim_ms = h->acc_ms[1];
    out->final_ms = h->acc_ms[2];
    out->sim_launches = h->sim_launches;
    return ok();
}

int svf_shape(const svf_batch* h, int64_t* num_requests, int32_t* num_instances,
              int32_t* num_policies) {
    if (!h) return fail(SVF_EINVAL, "handle is NULL");
    if (num_requests) *num_requests = h->N;
    if (num_instances) *num_instances = h->I;
    if (num_policies) *num_policies = h->P;
    return ok();
}

int svf_destroy(svf_batch* h) {
    if (!h) return ok();
    (void)hipStreamSynchronize(h->stream);
    free_all(h);
    delete h;
    return ok();
}

int svf_run_noalloc(const svf_batch_desc* d, void* hip_stream, int32_t* start, int32_t* finish,
                    int32_t* preempt, int32_t* admit_seq, svf_instance_stats* stats) {
    g_err[0] = 0;
    int64_t N = 0;
    RETCHK(check_desc_shape(d, &N));
    const int32_t I = d->num_instances, P = d->num_policies;
    if (d->inputs_on_device)
        return fail(SVF_EINVAL, "svf_run_noalloc: the inputs must be host memory (inputs_on_device = 0)");
    if (I > SVF_NOALLOC_MAX_INSTANCES)
        return fail(SVF_EINVAL, "svf_run_noalloc: %d instances, at most %d", I,
                    SVF_NOALLOC_MAX_INSTANCES);
    const int64_t G = (int64_t)P * I, PN = (int64_t)P * N;
    if (PN > 0 && (!start || !finish || !preempt || !admit_seq))
        return fail(SVF_EINVAL, "svf_run_noalloc: an output array is NULL");
    if (G > 0 && !stats) return fail(SVF_EINVAL, "svf_run_noalloc: stats is NULL");
    const int64_t* off = d->req_offsets;
    for (int32_t i = 0; i < I; ++i)
        if (off[i + 1] - off[i] > svfk::SORT_REC_MAX)
            return fail(SVF_EINVAL, "svf_run_noalloc: instance %d holds %lld requests, at most %d",
                        i, (long long)(off[i + 1] - off[i]), (int)svfk::SORT_REC_MAX);

    std::lock_guard<std::mutex> lock(g_na_mu);
    const HostView v{d->arrival, d->prompt, d->output, d->plan_len, d->long_bit};
    Facts facts;
    RETCHK(validate(d, v, off, N, g_na_stepped, 1, &facts));
    svf_batch h;  // the launch plan; its buffers are the scratch and the caller's outputs
    h.stream = (hipStream_t)hip_stream;
    HIPCHK(hipGetDevice(&h.device));
    RETCHK(plan_batch(&h, d, off, g_na_stepped, facts, g_na_bw_off));

    void* base = nullptr;
    size_t cap = 0;
    HIPCHK(svfk::noalloc_scratch(&base, &cap));
    Carve c{reinterpret_cast<uintptr_t>(base), 0};
    h.d_off = c.take<int64_t>(I + 1);
    h.d_pol = c.take<int32_t>(P);
    h.d_stepped = c.take<uint8_t>(G);
    h.d_bw_off = c.take<int64_t>(I + 1);
    h.d_a = c.take<int32_t>(N);
    h.d_s = c.take<int32_t>(N);
    h.d_o = c.take<int32_t>(N);
    if (d->plan_len) h.d_plan = c.take<int32_t>(N);
    if (d->long_bit) h.d_bit = c.take<int8_t>(N);
    const size_t inputs = c.used;
    h.d_rec = c.take<int4>(PN);
    h.d_rank = c.take<int32_t>(PN);
    h.d_bitmap = c.take<uint64_t>((int64_t)P * h.bw_total);
    if (h.ring_used) h.d_ring = c.take<int32_t>(G * (h.H + 64));
    if (h.list_known || h.list_stepped) {
        h.d_lst_f = c.take<int32_t>(G * (int64_t)h.list_stride);
        h.d_lst_q = c.take<uint32_t>(G * (int64_t)h.list_stride);
    }
    h.d_fin = c.take<int32_t>(PN);
    if (h.any_stepped) {
        h.d_act = c.take<int4>(PN);
        if (!h.step_regs) h.d_actkr = c.take<int2>(PN);
        h.d_evl = c.take<int32_t>(PN);
    }
    h.d_st = c.take<SegState>(G);
    // (of the progress counters, 16 bytes count against the limit; the scratch
    // array has room for the rest behind it)
    h.d_prog = c.take<unsigned long long>(2);
    if (c.used > cap)
        return fail(SVF_EINVAL, "svf_run_noalloc: the batch needs %zu bytes of device scratch, "
                                "more than the %zu this entry point has", c.used, cap);
    h.d_start = start;
    h.d_pre = preempt;
    h.d_seq = admit_seq;
    h.d_fin_out = finish;
    h.d_stats = reinterpret_cast<StatsOut*>(stats);

    // inputs and host tables into the scratch; everything else the call reads
    // is rebuilt by its own kernels (the scratch keeps the previous call's data)
    // (small ones side by side in host memory first: one copy instead of nine)
    const hipMemcpyKind k = hipMemcpyHostToDevice;
    hipError_t e = hipSuccess;
    const bool together = inputs <= sizeof g_na_stage;
    auto put = [&](void* dst, const void* src, size_t bytes) {
        if (!dst || !bytes || e != hipSuccess) return;
        if (together) memcpy(g_na_stage + (static_cast<char*>(dst) - static_cast<char*>(base)), src, bytes);
        else e = hipMemcpyAsync(dst, src, bytes, k, h.stream);
    };
    put(h.d_off, off, 8 * ((size_t)I + 1));
    put(h.d_pol, d->policies, 4 * (size_t)P);
    put(h.d_stepped, g_na_stepped, (size_t)G);
    put(h.d_bw_off, g_na_bw_off, 8 * ((size_t)I + 1));
    put(h.d_a, d->arrival, 4 * (size_t)N);
    put(h.d_s, d->prompt, 4 * (size_t)N);
    put(h.d_o, d->output, 4 * (size_t)N);
    if (d->plan_len) put(h.d_plan, d->plan_len, 4 * (size_t)N);
    if (d->long_bit) put(h.d_bit, d->long_bit, (size_t)N);
    if (together && e == hipSuccess) e = hipMemcpyAsync(base, g_na_stage, inputs, k, h.stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h.stream);
    if (e != hipSuccess)
        return fail(SVF_EHIP, "svf_run_noalloc: copying the inputs failed: %s", hipGetErrorString(e));
    HIPCHK(svfk::prepare_sim(h.d_lds, h.lds_bytes, h.list_stepped && !h.step_regs, h.lds_step_full));
    if (h.step_regs) HIPCHK(prepare_step(&h));
    if (h.list_known) HIPCHK(svfk::prepare_list(h.list_nb, h.lds_list, h.lds_list_full));
    HIPCHK(svfk::prepare_sort_rec(h.max_n));
    RETCHK(do_reset(&h));
    RETCHK(do_sim(&h, int64_t(1) << 40));
    RETCHK(do_finalize(&h));
    return ok();
}

}  // extern "C"
