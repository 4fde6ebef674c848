// Test driver for the host runtime (svf_runtime.cpp) on a machine without a
// GPU: HIP's calls and the kernel launchers are replaced by the small host
// functions below ("device" memory is malloc'd and filled with 0xAB, copies
// are memcpy), so that the paths past the first device allocation run under
// the sanitizers.  No simulation result is looked at here.
// tests/test_host_runtime.py builds and runs it.
//
//   reset       a reset whose launch fails leaves the outputs to the next one
//   rings       who writes the first ring, by its length
//   reads       svf_read into host memory of every kind and size
//   device      svf_read into device memory, long enough and too short
//   whole       every call on batches of both paths side by side
//   validate    validation on several threads against one thread
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <random>
#include <string>
#include <vector>

#include "svf_kernels.h"
#include "svfsim.h"

// ---------------------------------------------------------------- stand-ins

namespace {

std::mutex g_mu;
std::map<uintptr_t, std::pair<size_t, hipMemoryType>> g_mem;  // known ranges
std::atomic<int> g_host_mallocs{0}, g_copies{0}, g_into_pinned{0}, g_copy_kernels{0}, g_ring_launches{0};
int g_fail_sort = 0;           // launch_sort_rec calls that fail from here on
bool g_pattern = false;        // launch_finalize writes outputs 4 i + {0, 1, 2, 3}
svfk::SortArgs g_sort;         // arguments of the last reset
svfk::SimArgs g_sim;           // and of the last simulation launch
int g_sims = 0, g_continued = 0;  // simulation launches, and continuations among them

void know(void* p, size_t n, hipMemoryType t) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_mem[(uintptr_t)p] = {n, t};
}
void forget(void* p) {
    std::lock_guard<std::mutex> lock(g_mu);
    g_mem.erase((uintptr_t)p);
}
// the known range that p is in
hipMemoryType kind_of(const void* p, uintptr_t* base = nullptr, size_t* size = nullptr) {
    std::lock_guard<std::mutex> lock(g_mu);
    auto it = g_mem.upper_bound((uintptr_t)p);
    if (it == g_mem.begin()) return hipMemoryTypeUnregistered;
    --it;
    if ((uintptr_t)p >= it->first + it->second.first) return hipMemoryTypeUnregistered;
    if (base) *base = it->first;
    if (size) *size = it->second.first;
    return it->second.second;
}
// n bytes at p lie in one range, or in none that is known
bool inside(const void* p, size_t n) {
    uintptr_t base = 0;
    size_t size = 0;
    return kind_of(p, &base, &size) == hipMemoryTypeUnregistered || (uintptr_t)p + n <= base + size;
}

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    *p = malloc(n);
    if (!*p) return hipErrorOutOfMemory;
    memset(*p, 0xAB, n);
    know(*p, n, hipMemoryTypeDevice);
    return hipSuccess;
}
hipError_t hipFree(void* p) { forget(p); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    ++g_host_mallocs;
    *p = malloc(n);
    know(*p, n, hipMemoryTypeHost);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { forget(p); free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    if (!inside(d, n) || !inside(s, n)) return hipErrorInvalidValue;  // as the runtime does
    ++g_copies;
    if (kind_of(d) == hipMemoryTypeHost) ++g_into_pinned;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof *a);
    a->type = kind_of(p);
    return a->type == hipMemoryTypeUnregistered ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    uintptr_t b = 0;
    if (kind_of(p, &b, size) == hipMemoryTypeUnregistered) return hipErrorNotFound;
    *base = (hipDeviceptr_t)b;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace svfk {
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t) { std::fill(p, p + n, v); return hipSuccess; }
hipError_t launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t) { std::fill(p, p + n, v); return hipSuccess; }
hipError_t launch_init_ring(int32_t* p, int64_t n, int32_t, hipStream_t) {
    ++g_ring_launches;
    std::fill(p, p + n, 0);
    return hipSuccess;
}
hipError_t launch_copy4(const CopyArgs& C, int arrays, hipStream_t) {
    ++g_copy_kernels;
    for (int x = 0; x < arrays; ++x)
        if (!inside(C.dst[x], 4 * (size_t)C.n)) abort();  // a write out of range
    for (int x = 0; x < arrays; ++x) memcpy(C.dst[x], C.src[x], 4 * (size_t)C.n);
    return hipSuccess;
}
hipError_t launch_init_state(SegState*, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_chunk_sort(const SortArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_merge_pass(const SortArgs&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_build_rec(const SortArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t prepare_sort_rec(int) { return hipSuccess; }
hipError_t launch_sort_rec(const SortArgs& A, int, int, hipStream_t) {
    g_sort = A;
    if (g_fail_sort > 0) {
        --g_fail_sort;
        return hipErrorLaunchFailure;
    }
    for (int64_t x = 0; x < A.P * A.N; ++x) {
        A.start[x] = A.admit_seq[x] = -1;
        if (A.clear_all) {
            A.fin[x] = -1;
            A.preempt[x] = 0;
        }
    }
    return hipSuccess;
}
hipError_t prepare_sim(bool, size_t, bool, size_t) { return hipSuccess; }
hipError_t prepare_list(int, size_t, size_t) { return hipSuccess; }
hipError_t prepare_step(int, const size_t[3]) { return hipSuccess; }
static hipError_t occupancy(size_t lds, int* b) {
    *b = (int)std::min<size_t>(32, 160 * 1024 / std::max<size_t>(lds, 1));
    return hipSuccess;
}
hipError_t list_occupancy(int, size_t lds, int* b) { return occupancy(lds, b); }
hipError_t step_occupancy(int, size_t lds, int* b) { return occupancy(lds, b); }
hipError_t sim_step_occupancy(size_t lds, int* b) { return occupancy(lds, b); }
hipError_t launch_sim(const SimArgs& P, int, bool, bool, bool, size_t, hipStream_t) {
    g_sim = P;
    ++g_sims;
    g_continued += P.list_resume != 0;
    return hipSuccess;
}
hipError_t launch_finalize(const FinArgs& F, int, hipStream_t) {
    const int64_t PN = F.P * F.N;
    for (int64_t x = 0; x < PN; ++x) {
        F.fin_out[x] = g_pattern ? (int32_t)(4 * x + 1) : F.fin[x];
        if (!g_pattern) continue;
        g_sort.start[x] = (int32_t)(4 * x);
        g_sort.preempt[x] = (int32_t)(4 * x + 2);
        g_sort.admit_seq[x] = (int32_t)(4 * x + 3);
    }
    return hipSuccess;
}
hipError_t noalloc_scratch(void** p, size_t* n) {
    static std::vector<char> scratch(size_t(256) << 20);
    *p = scratch.data();
    *n = scratch.size() - NOALLOC_PROG_BYTES;
    return hipSuccess;
}
}  // namespace svfk

// ---------------------------------------------------------------- the tests

namespace {

int failures = 0;

void expect(bool ok, const char* what, long long a = 0, long long b = 0) {
    if (ok) return;
    fprintf(stderr, "FAILED: %s (%lld, %lld; last error: %s)\n", what, a, b, svf_last_error());
    ++failures;
}

struct Batch {
    std::vector<int64_t> off;
    std::vector<int32_t> a, s, o, plan, pol;
    std::vector<int8_t> bit;
    int64_t M = 0;
    svf_batch_desc desc() const {
        svf_batch_desc d{};
        d.num_instances = (int32_t)off.size() - 1;
        d.req_offsets = off.data();
        d.arrival = a.data();
        d.prompt = s.data();
        d.output = o.data();
        d.plan_len = plan.empty() ? nullptr : plan.data();
        d.long_bit = bit.empty() ? nullptr : bit.data();
        d.M = M;
        d.num_policies = (int32_t)pol.size();
        d.policies = pol.data();
        d.O0 = 16;
        d.O1 = 700;
        d.max_steps = 1 << 20;
        return d;
    }
};

// n requests in equal instances of ``each``
Batch plain(int64_t n, int64_t each) {
    Batch b;
    for (int64_t x = 0; x <= n; x += each) b.off.push_back(x);
    if (b.off.back() < n) b.off.push_back(n);
    b.a.assign((size_t)n, 0);
    b.s.assign((size_t)n, 3);
    b.o.assign((size_t)n, 5);
    b.M = 1000;
    b.pol = {SVF_POLICY_SVF};
    return b;
}

void reset_mode() {
    Batch b = plain(1000, 50);
    const svf_batch_desc d = b.desc();
    svf_batch* h = nullptr;
    expect(svf_create(&d, nullptr, &h) == SVF_OK, "create");
    g_fail_sort = 2;
    expect(svf_reset(h) == SVF_EHIP, "the failing reset says so");
    expect(svf_run(h) == SVF_EHIP, "and the one a run starts with");
    expect(svf_reset(h) == SVF_OK && svf_run(h) == SVF_OK, "the next one");
    std::vector<int32_t> fin(1000), pre(1000);
    expect(svf_read(h, 0, nullptr, fin.data(), pre.data(), nullptr, 0) == SVF_OK, "read");
    for (int x = 0; x < 1000 && !failures; ++x)
        expect(fin[x] == -1 && pre[x] == 0, "outputs cleared by the first reset that ran", fin[x], pre[x]);
    expect(svf_reset(h) == SVF_OK && g_sort.clear_all == 0, "cleared once");
    svf_destroy(h);
}

void rings_mode() {
    // per-step path, too many running for the list: a ring of the longest plan
    for (int lg : {10, 14, 15, 20}) {
        Batch b = plain(8192, 8192);
        b.M = 1 << 25;
        b.plan = b.o;
        b.plan[7] = 1 << lg;
        b.pol = {SVF_POLICY_FCFS};
        const svf_batch_desc d = b.desc();
        svf_batch* h = nullptr;
        expect(svf_create(&d, nullptr, &h) == SVF_OK, "create");
        g_ring_launches = 0;
        expect(svf_reset(h) == SVF_OK, "reset");
        expect((g_sort.ring != nullptr) == (lg <= 14), "the sort writes short rings", lg);
        expect(g_ring_launches == (lg <= 14 ? 0 : 1), "a launch of their own for long ones", lg);
        svf_destroy(h);
    }
}

void reads_mode() {
    g_pattern = true;
    constexpr int64_t SLOT = 1 << 19;  // words of a slot
    for (int64_t n : {int64_t(1), int64_t(100), int64_t(16384), int64_t(16385), int64_t(100000),
                      SLOT + 1, 2 * SLOT, 5 * SLOT + 77}) {
        Batch b = plain(n, 1000);
        b.pol = {SVF_POLICY_SVF, SVF_POLICY_FCFS};
        const svf_batch_desc d = b.desc();
        svf_batch* h = nullptr;
        expect(svf_create(&d, nullptr, &h) == SVF_OK && svf_run(h) == SVF_OK, "create and run");
        g_host_mallocs = 0;
        // which arrays are wanted, and which of them are page-locked
        for (int wanted = 0; wanted < 16; wanted += n > SLOT ? 5 : 1)
            for (int locked : {0, 15, 5}) {
                int32_t* buf[4];
                for (int x = 0; x < 4; ++x) {
                    buf[x] = (int32_t*)malloc(4 * (size_t)n);
                    std::fill(buf[x], buf[x] + n, -7);
                    if (locked >> x & 1) know(buf[x], 4 * (size_t)n, hipMemoryTypeHost);
                }
                auto arg = [&](int x) { return wanted >> x & 1 ? buf[x] : nullptr; };
                const int slot = wanted & 1;
                g_copies = g_into_pinned = g_copy_kernels = 0;
                const int before = g_host_mallocs;
                expect(svf_read(h, slot, arg(0), arg(1), arg(2), arg(3), 0) == SVF_OK, "read");
                const int want = __builtin_popcount(wanted), lock = __builtin_popcount(wanted & locked);
                const int64_t pageable = 4 * n * (want - lock);
                for (int x = 0; x < 4; ++x) {
                    bool right = true;
                    for (int64_t y = 0; y < n && right; ++y)
                        right = buf[x][y] == (wanted >> x & 1 ? (int32_t)(4 * (slot * n + y) + x) : -7);
                    expect(right, "the outputs", n, wanted);
                    if (locked >> x & 1) forget(buf[x]);
                    free(buf[x]);
                }
                // page-locked memory is written directly, one copy per array
                expect(g_into_pinned == lock || pageable >= (8 << 20), "a copy per page-locked array", n, wanted);
                if (pageable >= (8 << 20)) {
                    const int64_t per = (4 * n + 4 * SLOT - 1) / (4 * SLOT);
                    expect(g_copies == lock + per * (want - lock), "copies of a large read", g_copies, wanted);
                    continue;
                }
                expect(g_host_mallocs == before, "no slots for less than 8 MB", n, wanted);
                // small ordinary ones side by side in one copy
                const bool packed = 16 * n <= (256 << 10) && want - lock > 1;
                expect(g_copy_kernels == packed, "packed", n, wanted);
                expect(g_copies == lock + (packed ? 1 : want - lock), "copies", g_copies, wanted);
            }
        // a page-locked destination that is too short is the runtime's to refuse
        if (n > 1) {
            int32_t* small = (int32_t*)malloc(4 * (size_t)n - 4);
            std::vector<int32_t> other((size_t)n);
            know(small, 4 * (size_t)n - 4, hipMemoryTypeHost);
            expect(svf_read(h, 0, other.data(), small, nullptr, nullptr, 0) == SVF_EHIP, "too short", n);
            forget(small);
            free(small);
        }
        expect(g_host_mallocs <= 1, "slots are pinned once per handle", g_host_mallocs);
        svf_destroy(h);
    }
    expect(g_mem.empty(), "everything released", (long long)g_mem.size());
}

void device_mode() {
    g_pattern = true;
    for (int64_t n : {int64_t(1000), int64_t(3000000)}) {
        Batch b = plain(n, 1000);
        const svf_batch_desc d = b.desc();
        svf_batch* h = nullptr;
        expect(svf_create(&d, nullptr, &h) == SVF_OK && svf_run(h) == SVF_OK, "create and run");
        int32_t* buf[4];
        for (int32_t*& p : buf) (void)hipMalloc((void**)&p, 4 * (size_t)n);
        g_copies = g_copy_kernels = 0;
        expect(svf_read(h, 0, buf[0], buf[1], buf[2], buf[3], 1) == SVF_OK, "read");
        expect(g_copy_kernels == 1 && g_copies == 0, "one launch", g_copy_kernels, g_copies);
        for (int x = 0; x < 4; ++x)
            expect(buf[x][0] == x && buf[x][n - 1] == (int32_t)(4 * (n - 1) + x), "the outputs", n, x);
        // a destination that is too short is the runtime's to refuse
        for (int x = 0; x < 4; ++x) {
            int32_t* dst[4] = {buf[0], buf[1], buf[2], buf[3]};
            int32_t* small = nullptr;
            (void)hipMalloc((void**)&small, 4 * (size_t)n - 4);
            dst[x] = small;
            expect(svf_read(h, 0, dst[0], dst[1], dst[2], dst[3], 1) == SVF_EHIP, "too short", n, x);
            dst[x] = buf[x] + 1;
            expect(svf_read(h, 0, dst[0], dst[1], dst[2], dst[3], 1) == SVF_EHIP, "too short at its end", n, x);
            (void)hipFree(small);
        }
        for (int32_t* p : buf) (void)hipFree(p);
        svf_destroy(h);
    }
}

// Ragged instances, some empty, of at least ``least`` requests together, plans
// that differ from the truth in a quarter of them, bits.
Batch ragged(std::mt19937_64& rng, int64_t least, int longest) {
    auto draw = [&](int lo, int hi) { return lo + (int32_t)(rng() % (uint64_t)(hi - lo + 1)); };
    Batch b;
    b.M = 30000;
    b.off.push_back(0);
    while (b.off.back() < least) {
        const int n = draw(0, 9) == 0 ? 0 : draw(1, longest);
        int32_t t = 0;
        for (int j = 0; j < n; ++j) {
            t += draw(0, 2);
            b.a.push_back(t);
            b.s.push_back(draw(1, 900));
            b.o.push_back(draw(1, 700));
            b.plan.push_back(draw(0, 3) ? b.o.back() : draw(1, 700));
            b.bit.push_back((int8_t)draw(0, 1));
        }
        b.off.push_back(b.off.back() + n);
    }
    return b;
}

void whole_mode() {
    std::mt19937_64 rng(11);
    const std::vector<std::vector<int32_t>> mixes = {
        {SVF_POLICY_SVF}, {SVF_POLICY_SVF, SVF_POLICY_SVF | SVF_ADMIT_CURRENT},
        {SVF_POLICY_SVF, SVF_POLICY_SJF | SVF_ADMIT_CURRENT, SVF_POLICY_FCFS, SVF_POLICY_SVF1BIT}};
    // up to 2,700 running: the register form with a continuation, and past it
    for (int64_t M : {3000, 30000, 400000, 4000000})
        for (int longest : {120, 5000, 9000})
            for (const auto& mix : mixes)
                for (bool predicted : {false, true}) {
                    Batch b = ragged(rng, 20000, longest);
                    b.M = M;
                    b.pol = mix;
                    if (!predicted) b.plan.clear();
                    const svf_batch_desc d = b.desc();
                    const size_t N = (size_t)b.off.back(), I = b.off.size() - 1, P = mix.size();
                    std::vector<int32_t> out(4 * N * P);
                    std::vector<svf_instance_stats> st(I * P);
                    svf_batch* h = nullptr;
                    expect(svf_create(&d, nullptr, &h) == SVF_OK, "create", M, longest);
                    if (!h) continue;
                    expect(svf_set_profiling(h, 1) == SVF_OK, "profiling");
                    expect(svf_run(h) == SVF_OK && svf_reset(h) == SVF_OK, "run");
                    for (int64_t k : {0, 7, 1, 100}) expect(svf_step(h, k) == SVF_OK, "step");
                    svf_timing t;
                    expect(svf_timings(h, &t) == SVF_OK && t.sim_launches == 5, "timings", t.sim_launches);
                    for (size_t p = 0; p < P; ++p) {
                        int32_t* o = out.data() + 4 * N * p;
                        expect(svf_read(h, (int)p, o, o + N, o + 2 * N, o + 3 * N, 0) == SVF_OK, "read");
                        expect(svf_read(h, (int)p, o, o + N, o + 2 * N, o + 3 * N, 1) == SVF_OK, "read");
                        expect(svf_stats(h, (int)p, st.data() + I * p) == SVF_OK, "stats");
                    }
                    expect(svf_destroy(h) == SVF_OK, "destroy");
                    const int rc = svf_run_noalloc(&d, nullptr, out.data(), out.data() + N * P,
                                                   out.data() + 2 * N * P, out.data() + 3 * N * P, st.data());
                    expect(rc == (longest > 8192 && rc ? SVF_EINVAL : SVF_OK), "run_noalloc", rc);
                }
    expect(g_continued > 0 && g_sims > g_continued, "continuations launched", g_sims, g_continued);
    expect(g_mem.empty(), "everything released", (long long)g_mem.size());
}

void validate_mode() {
    std::mt19937_64 rng(7);
    auto draw = [&](int lo, int hi) { return lo + (int32_t)(rng() % (uint64_t)(hi - lo + 1)); };
    Batch b = ragged(rng, (1 << 20) + 50000, 3000);
    const int64_t N = b.off.back(), I = (int64_t)b.off.size() - 1;
    b.pol = {SVF_POLICY_SVF, SVF_POLICY_FCFS | SVF_ADMIT_CURRENT, SVF_POLICY_SVF1BIT, SVF_POLICY_SJF};
    const size_t P = b.pol.size();
    std::vector<int32_t> out((size_t)N * P);
    std::vector<svf_instance_stats> st((size_t)I * P);
    auto noalloc = [&](const svf_batch_desc& d) {
        return svf_run_noalloc(&d, nullptr, out.data(), out.data(), out.data(), out.data(), st.data());
    };
    const svf_batch_desc d = b.desc();
    expect(I <= SVF_NOALLOC_MAX_INSTANCES, "instances");
    expect(noalloc(d) == SVF_OK, "one thread");
    const svfk::SortArgs s1 = g_sort;
    const svfk::SimArgs q1 = g_sim;
    const std::vector<uint8_t> step1(s1.stepped, s1.stepped + P * I);
    const std::vector<int64_t> bw1(s1.bw_off, s1.bw_off + I + 1);
    for (int round = 0; round < 3; ++round) {
        svf_batch* h = nullptr;
        expect(svf_create(&d, nullptr, &h) == SVF_OK && svf_run(h) == SVF_OK, "several threads");
        if (!h) return;
        const svfk::SortArgs& s = g_sort;
        const svfk::SimArgs& q = g_sim;
        expect(!memcmp(s.kbits, s1.kbits, sizeof s.kbits), "bits of the keys");
        expect(s.H == s1.H && s.bw_total == s1.bw_total && s.CH == s1.CH, "sizes");
        expect(!memcmp(s.stepped, step1.data(), step1.size()), "paths");
        expect(!memcmp(s.bw_off, bw1.data(), 8 * bw1.size()), "bitmap offsets");
        expect(q.list_stride == q1.list_stride && q.list_cap == q1.list_cap && q.list_nb == q1.list_nb &&
                   q.step_regs == q1.step_regs && q.prio == q1.prio && q.bw_max == q1.bw_max && q.M == q1.M,
               "launch plan");
        svf_destroy(h);
    }
    // malformed requests, several at once: the first in instance order is named
    for (int round = 0; round < 40; ++round) {
        Batch w = b;
        for (int k = 0; k < 3; ++k) {
            const int64_t x = (int64_t)(rng() % (uint64_t)N);
            switch (draw(0, 6)) {
            case 0: w.a[x] = -1; break;
            case 1: w.a[x] = 1 << 29; break;
            case 2: w.s[x] = 0; break;
            case 3: w.o[x] = INT32_MIN; break;
            case 4: w.plan[x] = 0; break;
            case 5: w.bit[x] = 2; break;
            default: w.s[x] = INT32_MAX; break;
            }
        }
        const svf_batch_desc e = w.desc();
        const int rc = noalloc(e);
        const std::string text = svf_last_error();
        svf_batch* h = nullptr;
        expect(svf_create(&e, nullptr, &h) == rc && rc != SVF_OK && text == svf_last_error(),
               "the error of one thread", rc);
        if (h) svf_destroy(h);
    }
}

}  // namespace

int main(int argc, char** argv) {
    const std::string mode = argc > 1 ? argv[1] : "";
    if (mode == "reset") reset_mode();
    else if (mode == "rings") rings_mode();
    else if (mode == "reads") reads_mode();
    else if (mode == "device") device_mode();
    else if (mode == "whole") whole_mode();
    else if (mode == "validate") validate_mode();
    else return 2;
    printf("%s: %s\n", mode.c_str(), failures ? "FAILED" : "ok");
    return failures ? 1 : 0;
}
