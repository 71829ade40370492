// Host side of the library (mc_api.hip) on a stand-in device: device memory is
// host memory filled with a pattern, launches run at once (or are recorded
// while their stream captures), and an allocation or a launch can be made to
// fail. The stand-in passes do what the kernels do to the state that the host
// keeps: the fast pass counts queued records, the large-list pass sets the
// queue counts back. One scenario per run (argv[1]); prints what is wrong.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "../include/mc.h"
#include "../paper_2106_08150_amd/csrc/mc_internal.hpp"

using namespace mc;

// -------------------------------------------------------------- stand-in ----
namespace {

hipError_t g_last = hipSuccess;                      // the runtime's last error
std::map<void*, size_t> g_live;                      // device blocks
std::function<bool(size_t)> g_fail_alloc = [](size_t) { return false; };
std::string g_fail_launch;                           // this launch fails once
std::map<hipStream_t, std::vector<std::function<void()>>> g_capture;   // capturing streams
std::vector<std::string> g_calls;                    // launches that ran
std::string g_wrong;

void wrong(const std::string& s) {
    if (g_wrong.empty()) g_wrong = s;
}

hipError_t raise(hipError_t e) {
    g_last = e;
    return e;
}

// A launch: refused, recorded or run; its status is the runtime's last error,
// as the library's launchers return it.
hipError_t launch(const char* name, hipStream_t st, std::function<void()> f) {
    if (g_fail_launch == name) {
        g_fail_launch.clear();
        raise(hipErrorLaunchFailure);
    } else {
        auto run = [name, f] {
            g_calls.push_back(name);
            f();
        };
        auto it = g_capture.find(st);
        if (it != g_capture.end()) it->second.push_back(run);
        else run();
    }
    return hipGetLastError();
}

int calls(const char* name) {
    int n = 0;
    for (auto& c : g_calls) n += c == name;
    return n;
}

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (g_fail_alloc(n)) {
        *p = nullptr;
        return raise(hipErrorOutOfMemory);
    }
    *p = std::malloc(n ? n : 1);
    std::memset(*p, 0xA5, n);
    g_live[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!g_live.erase(p)) wrong("hipFree of a pointer that is not allocated");
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = size_t(1) << 30; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    static uintptr_t next = 0x1000;
    *s = reinterpret_cast<hipStream_t>(next += 16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    return g_capture.count(s) ? raise(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
    *c = g_capture.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    g_capture[s].clear();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
    *g = reinterpret_cast<hipGraph_t>(new std::vector<std::function<void()>>(g_capture[s]));
    g_capture.erase(s);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    *x = reinterpret_cast<hipGraphExec_t>(g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    for (auto& f : *reinterpret_cast<std::vector<std::function<void()>>*>(x)) f();
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

namespace {
uint32_t g_queued = 7;                  // records the next fast pass passes on
unsigned long long g_grow_deferred = 0; // entries the next growth by slices puts off
unsigned long long g_cond_deferred = 0; // features the next conversion puts off
uint64_t g_cond_cap = 0;                // list of the last conversion pass

// What a pass expects of its workspace.
void check_ready(const QueryArgs& a, const char* who) {
    for (uint32_t i = 0; i < kNumQueryCounters; ++i)
        if (i != kQTooLong && a.counters[i]) wrong(std::string(who) + ": queue counts not at zero");
    if (a.counters[kQTooLong] == 0xA5A5A5A5u) wrong(std::string(who) + ": too-long count not cleared");
    const uint32_t regions = a.huge_groups ? a.huge_groups : kHugeGroups;
    for (uint32_t r = 0; r < regions; ++r) {
        auto* best = reinterpret_cast<unsigned long long*>(a.huge + r * kHugeRegionBytes);
        for (uint32_t t = 0; t < kHugeTargets; ++t)
            if (best[t]) return wrong(std::string(who) + ": per-target bests not at zero");
    }
    if (a.qstats && a.qstats[0] > (1ull << 40)) wrong(std::string(who) + ": statistics not cleared");
    if (!a.route_meta) wrong(std::string(who) + ": no routing data");
}
}  // namespace

namespace mc {
hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, unsigned long long v, hipStream_t st) {
    return launch("fill", st, [=] { for (uint64_t i = 0; i < n; ++i) p[i] = v; });
}
hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t st) {
    return launch("fill", st, [=] { for (uint64_t i = 0; i < n; ++i) p[i] = v; });
}
hipError_t launch_clear_workspace(uint32_t* counters, unsigned char* huge, uint32_t regions,
                                  unsigned long long* qstats, hipStream_t st) {
    return launch("clear_workspace", st, [=] {
        std::memset(counters, 0, 4 * kNumQueryCounters);
        if (qstats) std::memset(qstats, 0, 8 * kQsWords);
        for (uint32_t r = 0; r < regions; ++r)
            std::memset(huge + r * kHugeRegionBytes, 0, 8 * kHugeTargets);
    });
}
hipError_t launch_classify_fast(const QueryArgs& a, const ClassifyConfig&, hipStream_t st) {
    return launch("fast", st, [=] {
        check_ready(a, "fast pass");
        a.counters[kQOverflow] += g_queued;
    });
}
hipError_t launch_classify_class(const QueryArgs& a, const ClassifyConfig& c, uint32_t,
                                 hipStream_t st) {
    return launch_classify_fast(a, c, st);
}
hipError_t launch_route(const QueryArgs&, const RouteConfig&, hipStream_t st) {
    return launch("route", st, [] {});
}
hipError_t launch_classify_large(const QueryArgs& a, hipStream_t st, uint32_t) {
    return launch("large", st, [=] {
        if (a.counters[kQOverflow] != g_queued) wrong("large-list pass: not its own records queued");
        for (uint32_t i = 0; i < kNumQueryCounters; ++i)
            if (i != kQTooLong) a.counters[i] = 0u;
    });
}
bool classify_config_valid(const ClassifyConfig&) { return true; }
hipError_t launch_sketch(const BuildArgs&, bool, hipStream_t st) { return launch("sketch", st, [] {}); }
hipError_t launch_partition(const BuildArgs&, uint64_t, hipStream_t st) {
    return launch("partition", st, [] {});
}
hipError_t launch_insert(const BuildArgs& a, uint64_t n, hipStream_t st) {
    return launch("insert", st, [=] { a.counters[kCntInserted] += n; });
}
bool slice_mode_fits(uint32_t) { return true; }
hipError_t launch_cap_finalize(unsigned long long*, uint64_t, uint32_t, const uint32_t*, uint64_t,
                               hipStream_t st) { return launch("cap", st, [] {}); }
hipError_t launch_cap_scan(unsigned long long*, uint64_t, uint32_t, uint32_t, hipStream_t st) {
    return launch("cap", st, [] {});
}
bool grow_slices_fit(uint64_t a, uint64_t b) { return b >= a + a / 4; }
hipError_t launch_grow_slices(const unsigned long long*, uint64_t, unsigned long long*, uint32_t*,
                              uint64_t, unsigned long long* counters, unsigned long long*, uint64_t,
                              hipStream_t st) {
    return launch("grow_slices", st, [=] {
        counters[kCntMoved] = 11;
        counters[kCntDefer] = g_grow_deferred;
    });
}
hipError_t launch_rehash(const unsigned long long*, uint64_t, unsigned long long*, uint32_t*,
                         uint64_t, unsigned long long* counters, hipStream_t st) {
    return launch("rehash", st, [=] { counters[kCntMoved] = 22; });
}
hipError_t launch_dump(const unsigned long long*, uint64_t, uint32_t, uint32_t, unsigned long long*,
                       uint64_t, unsigned long long*, hipStream_t) { return hipSuccess; }
hipError_t launch_census(const unsigned long long*, uint64_t, unsigned long long*, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_rollback(unsigned long long*, uint64_t, uint32_t, hipStream_t st) {
    return launch("rollback", st, [] {});
}
hipError_t launch_condense_count(CondArgs c, hipStream_t st) {
    return launch("condense_count", st, [=] { *c.res = CondResult{100, 0, 100, 0, 50, 0}; });
}
hipError_t launch_condense_write(CondArgs c, uint32_t, hipStream_t st) {
    return launch("condense_write", st, [=] {
        c.res->deferred = g_cond_deferred;
        g_cond_cap = c.defer_cap;
    });
}
hipError_t launch_condense_dump(const unsigned int*, uint64_t, const uint32_t*, uint32_t, uint32_t,
                                unsigned long long*, uint64_t, unsigned long long*, hipStream_t) {
    return hipSuccess;
}
}  // namespace mc

// ------------------------------------------------------------- scenarios ----
namespace {

hipStream_t const S = reinterpret_cast<hipStream_t>(0x100);

mc_db* database() {
    mc_db* db = mc_db_create(16, 128, 16, 254);
    const uint32_t parents[2] = {0, 0};
    if (!db || mc_db_set_taxonomy(db, parents, 2) != MC_OK) wrong("no database");
    return db;
}

int classify(mc_db* db, uint32_t n = 100) {
    static char reads[16];
    static uint64_t offsets[16];
    static uint32_t labels[16];
    return mc_classify(db, reads, offsets, n, labels, S);
}

void expect(int rc, int want, const char* what) {
    if (rc != want)
        wrong(std::string(what) + ": returned " + std::to_string(rc) + " (" + mc_last_error() + ")");
}

// A caller's own capture of a classification.
std::vector<std::function<void()>> capture(mc_db* db, const char* what) {
    g_capture[S].clear();
    expect(classify(db), MC_OK, what);
    auto ops = g_capture[S];
    g_capture.erase(S);
    return ops;
}
void replay(const std::vector<std::function<void()>>& ops) {
    for (auto& f : ops) f();
}

// The first call of a stream is captured, not run; the next one is plain.
void first_call_captured() {
    mc_db* db = database();
    auto ops = capture(db, "captured first call");
    expect(classify(db), MC_OK, "plain call before a replay");
    replay(ops);
    expect(classify(db), MC_OK, "plain call after a replay");
    mc_db_destroy(db);
}

// A workspace whose clearing failed is cleared by the next call.
void clearing_fails() {
    mc_db* db = database();
    g_fail_launch = "clear_workspace";
    expect(classify(db), MC_ERR_HIP, "call whose clearing fails");
    if (calls("fast")) wrong("classified without a cleared workspace");
    expect(classify(db), MC_OK, "the next call");
    mc_db_destroy(db);
}

// Each allocation of a new workspace fails in turn.
void allocation_fails() {
    for (int k = 0; k < 5; ++k) {
        mc_db* db = database();
        int left = 2 * k;   // (a block that is kept for reuse is tried twice)
        g_fail_alloc = [&](size_t) { return left-- <= 0; };
        for (int tries = 0; tries < 12; ++tries) {
            left = k;
            if (classify(db) == MC_OK) break;
        }
        g_fail_alloc = [](size_t) { return false; };
        expect(classify(db), MC_OK, "call after a failed allocation");
        mc_db_destroy(db);
    }
}

// A sequence that stops after its fast pass leaves counts behind: the next
// call, a replay of an earlier capture and a new capture start at zero.
void sequence_stops() {
    mc_db* db = database();
    expect(classify(db), MC_OK, "first call");
    auto before = capture(db, "capture");
    replay(before);
    for (int i = 0; i < 2; ++i) {
        g_fail_launch = "large";
        expect(classify(db), MC_ERR_HIP, "call whose large-list pass fails");
        replay(before);
        expect(classify(db), MC_OK, "plain call after it");
        g_fail_launch = "large";
        expect(classify(db), MC_ERR_HIP, "call whose large-list pass fails");
        auto after = capture(db, "capture after it");
        expect(classify(db), MC_OK, "plain call before the capture's replay");
        replay(after);
        replay(after);
    }
    mc_db_destroy(db);
}

// The library's own graph: captured again after a failed launch and after a
// change of the database.
void graph_calls() {
    mc_db* db = database();
    static char reads[16];
    static uint64_t offsets[16];
    static uint32_t labels[16];
    mc_query_opts o{4, 4, 0, 0, 0};
    mc_graph* g = mc_classify_graph_create(db, reads, offsets, 100, &o, labels, nullptr, S);
    if (!g) return wrong("no graph");
    expect(mc_classify_graph_launch(g, S), MC_OK, "replay");
    const uint32_t parents[2] = {0, 0};
    expect(mc_db_set_taxonomy(db, parents, 2), MC_OK, "taxonomy");
    g_fail_launch = "large";
    expect(mc_classify_graph_launch(g, S), MC_ERR_HIP, "capture that fails");
    expect(mc_classify_graph_launch(g, S), MC_OK, "capture again");
    expect(mc_classify_graph_launch(g, S), MC_OK, "replay");
    mc_classify_graph_destroy(g);
    mc_db_destroy(db);
}

// A table with entries whose growth needs a list of its own (the add's scratch
// is smaller than the list).
mc_db* filled(uint64_t* used) {
    mc_db* db = database();
    mc_insert_path path{};
    path.chunk_slots = 4096;
    mc_db_set_insert_path(db, &path);
    const uint32_t n = 40, len = 1 << 18;
    std::vector<char> text((size_t)n * len, 'A');
    std::vector<uint64_t> lengths(n, len);
    std::vector<uint32_t> taxa(n, 1);
    expect(mc_db_add_targets(db, text.data(), lengths.data(), taxa.data(), n), MC_OK, "add");
    *used = (uint64_t)n * ((len - 16 + 1 + 112) / 113) * 16;
    return db;
}

// The list for a growth cannot be allocated: the entries are re-inserted, as
// they are where no list is used.
void growth_list_fails() {
    uint64_t used = 0;
    mc_db* db = filled(&used);
    g_calls.clear();
    const size_t list = (used / 16 + 4096) * 8;
    int refused = 0;
    g_fail_alloc = [&](size_t n) { return n == list && ++refused; };
    expect(mc_db_reserve(db, 4 * used, 0.0), MC_OK, "growth without memory for its list");
    g_fail_alloc = [](size_t) { return false; };
    if (!refused) wrong("the growth asked for no list");
    if (calls("grow_slices") || calls("rehash") != 1) wrong("growth: not by re-insertion");
    mc_db_destroy(db);
}

// An allocation that failed is reported once: later calls do not see it.
void refused_allocation_is_reported_once() {
    mc_db* db = database();
    g_fail_alloc = [](size_t n) { return n > (size_t(1) << 30); };
    expect(mc_db_reserve(db, 1ull << 32, 0.0), MC_ERR_OOM, "table that does not fit");
    g_fail_alloc = [](size_t) { return false; };
    expect(classify(db), MC_OK, "classification after it");
    if (hipGetLastError() != hipSuccess) wrong("the caller's next launch would report the allocation");
    mc_db_destroy(db);
}

// More entries leave their slice than a growth's list holds: the growth starts
// over. A conversion's list is made anew at the size it needs.
void lists_too_short() {
    uint64_t used = 0;
    mc_db* db = filled(&used);
    g_calls.clear();
    expect(mc_db_reserve(db, 4 * used, 0.0), MC_OK, "growth");
    if (calls("grow_slices") != 1 || calls("rehash")) wrong("growth: not by slices alone");
    mc_insert_path path{};
    path.defer_entries = 5;
    mc_db_set_insert_path(db, &path);
    g_calls.clear();
    g_grow_deferred = 5;
    expect(mc_db_reserve(db, 16 * used, 0.0), MC_OK, "growth with a list that just holds");
    if (calls("grow_slices") != 1 || calls("rehash")) wrong("growth: started over without a reason");
    g_calls.clear();
    g_grow_deferred = 6;
    expect(mc_db_reserve(db, 64 * used, 0.0), MC_OK, "growth with a list that is too short");
    if (calls("grow_slices") != 1 || calls("rehash") != 1) wrong("growth: not started over");
    g_calls.clear();
    g_cond_deferred = 9;
    expect(mc_db_condense(db, 0), MC_OK, "conversion with a list that is too short");
    if (calls("condense_write") != 2 || g_cond_cap != 9) wrong("conversion: not repeated with a longer list");
    g_calls.clear();
    g_cond_deferred = 5;
    expect(mc_db_condense(db, 0), MC_OK, "conversion with a list that just holds");
    if (calls("condense_write") != 1) wrong("conversion: repeated without a reason");
    mc_db_destroy(db);
}

}  // namespace

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> all = {
        {"first_call_captured", first_call_captured},
        {"clearing_fails", clearing_fails},
        {"allocation_fails", allocation_fails},
        {"sequence_stops", sequence_stops},
        {"graph_calls", graph_calls},
        {"growth_list_fails", growth_list_fails},
        {"refused_allocation_is_reported_once", refused_allocation_is_reported_once},
        {"lists_too_short", lists_too_short},
    };
    if (argc != 2 || !all.count(argv[1])) return 2;
    all.at(argv[1])();
    if (!g_live.empty()) wrong(std::to_string(g_live.size()) + " device blocks not freed");
    std::puts(g_wrong.empty() ? "ok" : g_wrong.c_str());
    return g_wrong.empty() ? 0 : 1;
}
