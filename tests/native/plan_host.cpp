// The plan and its step entry points (plan.cpp, noalloc.hip) on the CPU: a stub HIP
// runtime whose device memory is host memory with a register of live allocations, and
// stub launchers that check every pointer and size that the kernels would be given.
// usage: plan_host SCENARIO; exit status 0 where it passes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "internal.hpp"

using namespace rexi;

// ------------------------------------------------------------------ stub runtime
namespace {

std::map<char*, size_t> live;
std::set<void*> held;          // workspace that launches under a caller's capture were given
int bad = 0, mallocs = 0, events_made = 0, events_live = 0;
int fail_at = 0;               // the fail_at-th hipMalloc from now fails ...
bool fail_on = false;          // ... and those after it
size_t budget = ~size_t(0), used = 0;
bool capturing = false;
hipError_t last_error = hipSuccess;
long long new_at = 0;          // the new_at-th allocation of the host from now fails
double now_ms = 0, begin_ms = 0, graph_ms = 0;  // what the launches so far took
int last_wgs = 0, last_grid = 0;  // of the last pole-per-lane solve (0: a tiled one)
std::function<double(const Schedule&)> cost;  // of one step, ms

// The stub's own allocations do not fail.
struct Quiet {
    long long was = new_at;
    Quiet() { new_at = 0; }
    ~Quiet() { new_at = was; }
};

void complain(const std::string& what) {
    std::fprintf(stderr, "  %s\n", what.c_str());
    ++bad;
}

// [p, p + bytes) is device memory
void need(const void* p, size_t bytes, const char* what, const void* array = nullptr, size_t array_bytes = 0) {
    Quiet quiet;
    const char* c = static_cast<const char*>(p);
    const char* a = static_cast<const char*>(array);
    if (a && c >= a && c + bytes <= a + array_bytes) return;
    auto it = live.upper_bound(const_cast<char*>(c));
    if (p && it != live.begin()) {
        --it;
        if (c >= it->first && c + bytes <= it->first + it->second) {
            if (capturing) held.insert(it->first);
            return;
        }
    }
    complain(std::string(what) + (p ? ": not within a live allocation" : ": NULL"));
}

void expect(bool ok, const std::string& what) {
    if (!ok) complain("expected: " + what);
}

}  // namespace

void* operator new(size_t n) {
    if (new_at > 0 && --new_at == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
    return new_at > 0 && --new_at == 0 ? nullptr : std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    Quiet quiet;
    ++mallocs;
    const bool fails = (fail_at > 0 && --fail_at == 0) || used + n > budget;
    if (fails) {
        if (fail_on) fail_at = 1;
        *p = nullptr;
        return last_error = hipErrorOutOfMemory;
    }
    if (capturing) complain("allocation under a caller's capture");
    *p = std::malloc(n);
    live[static_cast<char*>(*p)] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    auto it = live.find(static_cast<char*>(p));
    if (it == live.end()) {
        complain("hipFree of something else");
        return hipErrorInvalidValue;
    }
    if (held.count(p)) complain("workspace of a captured step freed");
    used -= it->second;
    live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    need(d, n, "hipMemcpy");
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* s) {
    *p = const_cast<void*>(s);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(8);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
// (the plan's own graphs: an instance holds what its launches take)
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    begin_ms = now_ms;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = reinterpret_cast<hipGraph_t>(8);
    graph_ms = now_ms - begin_ms;
    now_ms = begin_ms;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
    *st = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    Quiet quiet;
    *e = reinterpret_cast<hipGraphExec_t>(new double(graph_ms));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    delete reinterpret_cast<double*>(e);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    now_ms += *reinterpret_cast<double*>(e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    Quiet quiet;
    ++events_made;
    ++events_live;
    *e = reinterpret_cast<hipEvent_t>(new double(0));
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    --events_live;
    delete reinterpret_cast<double*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    *reinterpret_cast<double*>(e) = now_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(*reinterpret_cast<double*>(b) - *reinterpret_cast<double*>(a));
    return hipSuccess;
}
}  // extern "C"

// ------------------------------------------------------------------ stub launchers
namespace rexi {

bool solve_variant_supported(int SE, int kind, int rot, bool) {
    return kind == 0 ? SE == 16 && rot == 1 : kind == 2 ? (SE == 4 || SE == 8) && rot <= 2 : SE <= 16;
}
int solve_waves_per_item() { return 4; }
int solve_variant_list(bool, int*, int*, int*, int) { return 0; }

static void need_ws(rexi_plan* pl, const void* p, size_t bytes, const char* what) {
    need(p, bytes, what, pl->scratch, pl->scratch_bytes);
}
static void need_chains(rexi_plan* pl, const Workspace& ws, int buf, int S) {
    need_ws(pl, ws.ch_var[buf], (size_t)S * (pl->nslots + 2) * 16, "ch_var");
    need_ws(pl, ws.ch_phi[buf], (size_t)S * pl->nspec * 16, "ch_phi");
}
hipError_t enqueue_prep(rexi_plan* pl, const Workspace& ws, const void*, int buf, int S, int, const MInfo* layout,
                        hipStream_t) {
    need_chains(pl, ws, buf, S);
    need(layout, sizeof(MInfo) * (pl->T + 1), "layout");
    return hipGetLastError();
}
hipError_t enqueue_solve(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf, int S, int adjoint,
                         hipStream_t) {
    need_chains(pl, ws, buf, S);
    need(sc.d_items, sc.items.size() * sizeof(Item), "items");
    need(sc.d_minfo, sc.minfo.size() * sizeof(MInfo), "minfo");
    need(pl->d_poles[adjoint], (size_t)pl->N * 96, "poles");
    need_ws(pl, ws.part, (size_t)sc.part_size * 16, "part");
    if (sc.persistent) need_ws(pl, ws.counters, kMaxLaunches * sizeof(int), "counters");
    last_wgs = last_grid = 0;
    if (cost) now_ms += cost(sc);
    return hipGetLastError();
}
hipError_t enqueue_reduce(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const double2* part, int buf_in,
                          int buf_out, void*, int S, int, const int*, hipStream_t) {
    need_chains(pl, ws, buf_in, S);
    need_chains(pl, ws, buf_out, S);
    need(sc.d_groups, sc.groups.size() * sizeof(Group), "groups");
    need_ws(pl, part, (size_t)sc.part_size * 16, "part");
    return hipGetLastError();
}
hipError_t enqueue_zero(double2* p, long long n, hipStream_t) {
    need(p, (size_t)n * 16, "zeroed");
    return hipGetLastError();
}
hipError_t enqueue_finish(rexi_plan* pl, const Workspace& ws, int buf, void*, int S, int, const MInfo*, hipStream_t) {
    need_chains(pl, ws, buf, S);
    return hipGetLastError();
}
hipError_t enqueue_per_term_pole(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int, int buf, int S,
                                 hipStream_t) {
    need_chains(pl, ws, buf, S);
    need(sc.d_items, sc.items.size() * sizeof(Item), "items");
    need(pl->d_acc, (size_t)sc.part_size * 16, "acc");
    return hipGetLastError();
}
hipError_t enqueue_fsphere_steps(rexi_plan*, const void*, void*, int, int, int, hipStream_t) { return hipGetLastError(); }

static void need_records(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf) {
    need_ws(pl, ws.rec[buf], ((size_t)(pl->sweep[sc.split].npairs + 1) * sc.S * kSweepRec + kSweepPad) * 8, "records");
}
hipError_t enqueue_sweep_prep(rexi_plan* pl, const Workspace& ws, const Schedule& sc, const void*, int buf, int,
                              int adjoint, hipStream_t) {
    const SweepTables& t = pl->sweep[sc.split];
    need_records(pl, ws, sc, buf);
    need(t.d_idx, (size_t)t.npairs * sizeof(int2), "idx");
    need(t.d_fin[adjoint], (size_t)t.npairs * 24, "fin");
    return hipGetLastError();
}
hipError_t enqueue_sweep_solve(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf, int, int adjoint,
                               hipStream_t) {
    const SweepTables& t = pl->sweep[sc.split];
    need_records(pl, ws, sc, buf);
    need(sc.d_sweep_items, sc.sweep_items.size() * sizeof(SweepItem), "sweep items");
    need(t.d_cst, ((size_t)t.npairs * kSweepCst + kSweepPad) * 8, "cst");
    need(t.d_poles[adjoint], (size_t)pl->N * 96, "sweep poles");
    need_ws(pl, ws.part, (size_t)sc.part_size * 16, "part");
    const int wgs = ((int)sc.sweep_items.size() + kSweepWaves - 1) / kSweepWaves;
    int grid = std::min(wgs, ws.sweep_groups);
    if (grid < 1) return hipErrorInvalidValue;
    if (sc.persistent || (ws.counters && sweep_resident(sc))) {
        need_ws(pl, ws.counters, sizeof(int), "counters");
        grid = std::min(grid, kSweepGroups);
    }
    if (sc.sweep_stride > 0)
        need_ws(pl, ws.sweep_scratch, (size_t)grid * kSweepWaves * sc.sweep_stride * 16, "boundary values");
    last_wgs = wgs;
    last_grid = grid;
    // register-resident chains take one group of items per workgroup
    if (sc.short_chains && !sc.persistent) expect(grid == wgs, "a workgroup for every group of items");
    if (cost) now_ms += cost(sc);
    return hipGetLastError();
}
hipError_t enqueue_sweep_reduce(rexi_plan* pl, const Workspace& ws, const Schedule& sc, int buf_in, int buf_out,
                                void* u_out, int, int adjoint, hipStream_t) {
    const SweepTables& t = pl->sweep[sc.split];
    need_records(pl, ws, sc, buf_in);
    if (!u_out) need_records(pl, ws, sc, buf_out);
    need(sc.d_sweep_tiles, sc.sweep_tiles.size() * sizeof(SweepTile), "tiles");
    need(sc.d_sweep_groups, sc.sweep_groups.size() * sizeof(SweepGroup), "sweep groups");
    need(t.d_fout[adjoint], (size_t)t.npairs * 24, "fout");
    need_ws(pl, ws.part, (size_t)sc.part_size * 16, "part");
    return hipGetLastError();
}
int sh_setup(rexi_plan*) { return REXI_OK; }
void sh_release(rexi_plan*) {}
int sh_run(rexi_plan*, const void*, void*, int, bool, hipStream_t) { return REXI_OK; }
int sh_vec_run(rexi_plan*, const void*, void*, long long, int, bool, hipStream_t) { return REXI_OK; }

}  // namespace rexi

// ------------------------------------------------------------------ scenarios
namespace {

// States are only passed on; their addresses have to be apart.
char* const kIn = reinterpret_cast<char*>(size_t(1) << 44);
char* const kOut = reinterpret_cast<char*>(size_t(1) << 45);

rexi_params make_plan_params(int T, int M, int max_states) {
    rexi_params p{};
    p.T = T;
    p.radius = 6.37122e6;
    p.omega = 7.292e-5;
    p.gravity = 9.80616;
    p.mean_depth = 1e4;
    p.dt = 3600;
    p.M = M;
    p.h = 0.2;
    p.L = 11;
    p.normalize = 1;
    p.max_states = max_states;
    p.max_fields = 1;
    return p;
}

rexi_plan* make_plan(int T, int M, int max_states) {
    const rexi_params p = make_plan_params(T, M, max_states);
    rexi_plan* pl = nullptr;
    const int rc = rexi_plan_create(&p, &pl);
    if (rc) {
        std::fprintf(stderr, "rexi_plan_create: %d %s\n", rc, rexi_last_error());
        std::exit(2);
    }
    return pl;
}

int step(rexi_plan* pl, int S) { return rexi_step(pl, kIn, kOut, S, 2, nullptr); }

void destroy(rexi_plan* pl) {
    held.clear();
    rexi_plan_destroy(pl);
    expect(live.empty(), "all device memory given back");
    expect(events_live == 0, "all events given back");
    for (auto& a : live) std::free(a.first);
    live.clear();
    used = 0;
}

// An allocation failure that a call has reported is not reported again by the next.
int handled_failure() {
    rexi_plan* pl = make_plan(31, 20, 8);
    expect(step(pl, 2) == REXI_OK, "a step");
    fail_at = 1;
    expect(rexi_step_per_term(pl, kIn, kOut, 2, nullptr) == REXI_ENOMEM, "REXI_ENOMEM where an allocation fails");
    expect(step(pl, 2) == REXI_OK, "the step after it");
    for (int n = 1; n <= 2; ++n) {  // (the schedules are uploaded before its two states)
        int index = 0;
        expect(rexi_plan_autotune(pl, 2, nullptr, &index) == REXI_OK, "the schedules timed");
        fail_at = n;
        expect(rexi_plan_autotune(pl, 2, nullptr, &index) != REXI_OK, "an error where a state's allocation fails");
        expect(step(pl, 2) == REXI_OK, "the step after it");
    }
    expect(last_error == hipSuccess, "no error left behind");
    destroy(pl);
    return bad;
}

void disarm() {
    fail_at = 0;
    fail_on = false;
}

// `first` succeeds; then the n-th allocation of `second` fails (alone, or with all
// after it), for every n that there is; then both succeed again, on sound buffers.
void fail_every(const char* what, int T, int M, std::function<int(rexi_plan*)> first,
                std::function<int(rexi_plan*)> second) {
    for (int all = 0; all < 2; ++all)
        for (int n = 1;; ++n) {
            rexi_plan* pl = make_plan(T, M, 8);
            expect(first(pl) == REXI_OK, std::string(what) + ": the first call succeeds");
            fail_at = n;
            fail_on = all != 0;
            const int before = mallocs, rc = second(pl);
            const bool hit = mallocs - before >= n;
            disarm();
            const std::string at = std::string(what) + ", allocation " + std::to_string(n) + (all ? " on" : "");
            expect(rc == REXI_OK || (hit && rc == REXI_ENOMEM), at + ": succeeds or reports REXI_ENOMEM");
            expect(first(pl) == REXI_OK, at + ": the first call again");
            expect(second(pl) == REXI_OK, at + ": the failed call again");
            expect(first(pl) == REXI_OK, at + ": the first call at last");
            destroy(pl);
            if (!hit || bad > 20) break;
        }
}

// Steps of more states than before, whose allocations fail one after another (with
// the tables of both there: T 63, chains in registers, without boundary values; T 100,
// split chains; T 200, whole ones).
int failed_growth() {
    for (int T : {63, 100, 200})
        for (int S : {1, 4})
            fail_every("more states", T, T == 200 ? 150 : 21,
                       [S](rexi_plan* p) { return step(p, S); }, [](rexi_plan* p) { return step(p, 8); });
    return bad;
}

// Where memory is short a schedule runs with fewer slots for boundary values, and its
// next steps allocate nothing.
int shortage() {
    for (int listed = 0; listed < 2; ++listed) {
        auto use = [&](rexi_plan* pl) {
            int n = 0;
            if (listed) expect(rexi_plan_set_schedule(pl, 8, -1, &n) == REXI_OK, "the schedules listed");
            expect(step(pl, 8) == REXI_OK, "a step");
        };
        rexi_plan* pl = make_plan(200, 150, 8);
        use(pl);
        const long long full = pl->sweep_scratch_capacity;
        const size_t all = used;
        destroy(pl);
        pl = make_plan(200, 150, 8);
        budget = all - (size_t)full * 16 * 5 / 8;
        use(pl);
        expect(pl->sweep_scratch_capacity > 0 && pl->sweep_scratch_capacity < full, "fewer slots");
        const int before = mallocs;
        for (int k = 0; k < 3; ++k) expect(step(pl, 8) == REXI_OK, "a further step");
        expect(mallocs == before, "no further allocation");
        expect(step(pl, 1) == REXI_OK && step(pl, 8) == REXI_OK, "steps of other states between them");
        budget = ~size_t(0);
        destroy(pl);
    }
    return bad;
}

// The first step of a plan, whose allocations fail one after another.
int failed_tables() {
    for (int T : {63, 100})
        for (int S : {1, 8})
            fail_every("a first step", T, 150, [](rexi_plan*) { return REXI_OK; }, [S](rexi_plan* p) { return step(p, S); });
    return bad;
}

// The workspace that a caller's captured step was given is there until the plan is
// destroyed, whatever state counts and schedules come after it.
int captured_buffers() {
    for (int T : {63, 100, 200}) {
        rexi_plan* pl = make_plan(T, T == 200 ? 150 : 21, 8);
        int n = 0;
        expect(step(pl, 1) == REXI_OK && rexi_step_per_term(pl, kIn, kOut, 1, nullptr) == REXI_OK, "steps of one state");
        capturing = true;
        expect(step(pl, 1) == REXI_OK && rexi_step_per_term(pl, kIn, kOut, 1, nullptr) == REXI_OK, "captured steps");
        capturing = false;
        expect(!held.empty(), "workspace in use");
        for (int S : {2, 4, 8}) {
            expect(step(pl, S) == REXI_OK && rexi_step_per_term(pl, kIn, kOut, S, nullptr) == REXI_OK, "steps of more states");
            expect(rexi_plan_set_schedule(pl, S, -1, &n) == REXI_OK && n > 0, "their schedules");
            expect(rexi_plan_set_schedule(pl, S, n - 1, nullptr) == REXI_OK && step(pl, S) == REXI_OK, "another one");
        }
        destroy(pl);
    }
    // without a capture nothing is kept: the buffers are one schedule's after the growth
    rexi_plan* pl = make_plan(63, 21, 8);
    for (int S : {1, 2, 4, 8}) expect(step(pl, S) == REXI_OK, "steps of more and more states");
    expect(pl->retired.empty(), "no smaller buffer kept");
    destroy(pl);
    return bad;
}

// The no-allocation step makes no events and is not timed, also where timing is on.
int noalloc_untimed() {
    for (int T : {31, 100}) {
        rexi_plan* pl = make_plan(T, 20, 8);
        expect(step(pl, 2) == REXI_OK, "a step");
        rexi_plan_set_timing(pl, 1);
        const int e = events_made, m = mallocs;
        expect(rexi_step_noalloc(pl, kIn, kOut, 2, 3, nullptr) == REXI_OK, "a no-allocation step");
        expect(events_made == e && mallocs == m, "no event and no allocation");
        double ms = 0;
        long long n = -1;
        expect(rexi_plan_kernel_time(pl, REXI_KERNEL_SOLVE, &ms, &n) == REXI_OK && n == 0, "nothing timed");
        expect(step(pl, 2) == REXI_OK, "a step");
        expect(rexi_plan_kernel_time(pl, REXI_KERNEL_SOLVE, &ms, &n) == REXI_OK && n == 2, "its two launches timed");
        destroy(pl);
    }
    return bad;
}

// Host allocations that fail end in REXI_ENOMEM, not in an exception that leaves the
// C interface, and nothing half built is used afterwards.
int host_allocations() {
    auto names = [](rexi_plan* pl, int S) {
        std::string all;
        int n = 0;
        expect(rexi_plan_set_schedule(pl, S, -1, &n) == REXI_OK, "the schedules");
        for (int i = 0; i < n; ++i) {
            char buf[128];
            expect(rexi_plan_schedule_name(pl, S, i, buf, sizeof buf) == REXI_OK, "a name");
            all += std::string(buf) + " ";
        }
        return all;
    };
    const int T = 26, S = 3;
    struct Call {
        const char* what;
        std::function<int(rexi_plan*)> f;
    };
    const Call calls[] = {
        {"rexi_step", [](rexi_plan* p) { return step(p, S); }},
        {"rexi_step_per_term", [](rexi_plan* p) { return rexi_step_per_term(p, kIn, kOut, S, nullptr); }},
        {"rexi_plan_set_schedule", [](rexi_plan* p) { return rexi_plan_set_schedule(p, S, 3, nullptr); }},
        {"rexi_plan_get_schedule", [](rexi_plan* p) { int i; return rexi_plan_get_schedule(p, S, &i); }},
        {"rexi_plan_schedule_name", [](rexi_plan* p) { char b[128]; return rexi_plan_schedule_name(p, S, 0, b, 128); }},
        {"rexi_plan_schedule_classes",
         [](rexi_plan* p) { int n; return rexi_plan_schedule_classes(p, S, 0, 0, nullptr, nullptr, nullptr, &n); }},
        {"rexi_plan_autotune", [](rexi_plan* p) { int i; return rexi_plan_autotune(p, S, nullptr, &i); }},
    };
    rexi_plan* ref = make_plan(T, 20, 8);
    expect(step(ref, S) == REXI_OK, "a step");
    const std::string want = names(ref, S);
    destroy(ref);
    for (const Call& c : calls)
        for (long long n = 1;; n += 1 + n / 25) {
            rexi_plan* pl = make_plan(T, 20, 8);
            rexi_plan_set_timing(pl, 1);
            new_at = n;
            int rc = -99;
            try {
                rc = c.f(pl);
            } catch (...) {
            }
            const bool hit = new_at == 0;
            new_at = 0;
            const std::string at = std::string(c.what) + ", host allocation " + std::to_string(n);
            expect(hit ? rc == REXI_ENOMEM || rc == REXI_OK : rc == REXI_OK, at + ": REXI_ENOMEM, got " + std::to_string(rc));
            expect(c.f(pl) == REXI_OK, at + ": the call again");
            expect(step(pl, S) == REXI_OK, at + ": a step");
            expect(names(pl, S) == want, at + ": the schedules as ever");
            destroy(pl);
            if (!hit || bad > 20) break;
        }
    for (long long n = 1;; n += 1 + n / 25) {  // a plan that is not made leaves nothing
        rexi_params p = make_plan_params(T, 20, 8);
        rexi_plan* pl = nullptr;
        new_at = n;
        int rc = -99;
        try {
            rc = rexi_plan_create(&p, &pl);
        } catch (...) {
        }
        const bool hit = new_at == 0;
        new_at = 0;
        expect(hit ? rc == REXI_ENOMEM && !pl : rc == REXI_OK, "rexi_plan_create: REXI_ENOMEM");
        if (!hit) {
            destroy(pl);
            break;
        }
        expect(live.empty(), "rexi_plan_create, host allocation " + std::to_string(n) + ": nothing left");
        if (bad > 20) break;
    }
    return bad;
}

// A pole-per-lane schedule that the no-allocation step's array does not hold is
// replaced where the plan chose it, and refused where the caller did.
int noalloc_selection() {
    rexi_plan* pl = make_plan(60, 500, 8);
    const int S = 4;
    auto noalloc = [&] { return rexi_step_noalloc(pl, kIn, kOut, S, 1, nullptr); };
    int n = 0, own = -1;
    expect(step(pl, S) == REXI_OK && noalloc() == REXI_OK, "the default, unlisted");
    expect(rexi_plan_get_schedule(pl, S, &own) == REXI_OK && noalloc() == REXI_OK, "the default, listed");
    expect(rexi_plan_set_schedule(pl, S, -1, &n) == REXI_OK, "the schedules");
    int refused = 0, ran = 0;
    for (int i = 0; i < n; ++i) {
        char name[128];
        expect(rexi_plan_set_schedule(pl, S, i, nullptr) == REXI_OK, "a selection");
        expect(rexi_plan_schedule_name(pl, S, i, name, sizeof name) == REXI_OK, "a name");
        if (std::string(name).find("sweep") != 0) continue;
        const int rc = noalloc();
        if (i == own) expect(rc == REXI_OK, "the plan's own choice, selected again");
        else expect(rc == REXI_EUNSUPPORTED, std::string(name) + " refused"), ++refused;
    }
    expect(refused > 0, "another pole-per-lane schedule");
    cost = [](const Schedule& sc) { return sc.sweep && !sc.persistent && sc.sweep_items.size() < 2000 ? 1.0 : 2.0; };
    int best = -1;
    expect(rexi_plan_autotune(pl, S, nullptr, &best) == REXI_OK && pl->sched[S][best].sweep, "the autotuner's choice");
    expect(noalloc() == REXI_OK, "the autotuner's choice");
    cost = nullptr;
    for (int i = 0; i < n; ++i)  // tiled schedules run or are refused as selected
        if (!pl->sched[S][i].sweep && !pl->sched[S][i].persistent) {
            expect(rexi_plan_set_schedule(pl, S, i, nullptr) == REXI_OK, "a selection");
            ran += noalloc() == REXI_OK;
        }
    expect(ran > 0, "tiled schedules that fit");
    destroy(pl);
    return bad;
}

// Which way the no-allocation step takes at the sizes that test_zz_no_alloc_paths.py
// runs on a GPU.
int noalloc_routes() {
    struct Case {
        int T, S, M;
        char route;  // 'a' a slot for every workgroup, 's' several items in turn, 't' the tiled schedule
    };
    for (const Case& c : {Case{100, 1, 250, 'a'}, Case{60, 1, 500, 'a'}, Case{100, 1, 500, 's'}, Case{31, 8, 1000, 's'},
                          Case{60, 4, 500, 't'}, Case{150, 1, 250, 't'}}) {
        rexi_plan* pl = make_plan(c.T, c.M, 8);
        expect(step(pl, c.S) == REXI_OK && last_wgs > 0, "a pole-per-lane step");
        expect(pl->first[c.S].sweep_stride > 0, "with boundary values");
        expect(rexi_step_noalloc(pl, kIn, kOut, c.S, 2, nullptr) == REXI_OK, "a no-allocation step");
        const char r = last_wgs == 0 ? 't' : last_grid == last_wgs ? 'a' : 's';
        expect(r == c.route, "T" + std::to_string(c.T) + " S" + std::to_string(c.S) + " M" + std::to_string(c.M) +
                                 ": route " + c.route + ", got " + r);
        if (c.route == 's') expect(last_grid >= kSweepGroups, "workgroups that fill the chip");
        destroy(pl);
    }
    return bad;
}

// States of an item of the default schedule: one or two where that leaves few waves;
// the default is among the candidates, by its name, once.
int few_poles() {
    struct Case {
        int T, S, M, most;
    };
    for (const Case& c : {Case{127, 4, 1, 1}, Case{127, 8, 1, 2}, Case{100, 6, 53, 3}, Case{63, 4, 1, 1}, Case{63, 6, 21, 3},
                          Case{256, 4, 1, 2}, Case{256, 1, 1, 1}, Case{200, 8, 150, 4}, Case{31, 3, 500, 3}}) {
        const std::string at = "T" + std::to_string(c.T) + " S" + std::to_string(c.S) + " M" + std::to_string(c.M);
        rexi_plan* pl = make_plan(c.T, c.M, 8);
        expect(step(pl, c.S) == REXI_OK, at + ": a step");
        expect(pl->first[c.S].sweep_nst == c.most, at + ": " + std::to_string(c.most) + " states an item, got " +
                                                      std::to_string(pl->first[c.S].sweep_nst));
        const std::string name = pl->first[c.S].name;
        int index = -1;
        expect(rexi_plan_get_schedule(pl, c.S, &index) == REXI_OK && pl->sched[c.S][index].name == name, at + ": listed");
        std::set<std::string> names;
        for (const Schedule& x : pl->sched[c.S])
            if (x.sweep && x.split) expect(names.insert(x.name).second, at + ": " + x.name + " once");
        for (int i = 0; i < (int)pl->sched[c.S].size(); ++i)
            if (pl->sched[c.S][i].sweep)
                expect(rexi_plan_set_schedule(pl, c.S, i, nullptr) == REXI_OK && step(pl, c.S) == REXI_OK, at + ": a step of each");
        destroy(pl);
    }
    return bad;
}

// Column chunks of the inverse transform: two groups of four where there are few
// workgroups, else as many columns as fit; every chunk is compiled (up to 32 columns).
int inverse_chunks() {
    struct Case {
        int B, per_wave, tiles, columns;
    };
    for (const Case& c : {Case{12, 1, 528, 8}, Case{16, 1, 528, 8}, Case{24, 1, 528, 24}, Case{32, 1, 528, 32},
                          Case{512, 1, 528, 32}, Case{8, 1, 840, 8}, Case{8, 1, 912, 16}, Case{12, 1, 912, 24},
                          Case{96, 1, 128, 8}, Case{1024, 1, 128, 32}, Case{5, 1, 264, 12}, Case{1, 1, 16, 4},
                          Case{16, 2, 4096, 32}, Case{17, 2, 4096, 20}}) {
        const int got = inverse_columns(2 * c.B, c.per_wave, c.tiles);
        expect(got == c.columns, std::to_string(c.B) + " fields, " + std::to_string(c.tiles) + " tiles: " +
                                     std::to_string(c.columns) + " columns, got " + std::to_string(got));
    }
    for (int B = 1; B <= 1024; ++B)
        for (int tiles : {8, 400, 2000})
            for (int per_wave : {1, 2}) {
                const int cw = inverse_columns(2 * B, per_wave, tiles);
                expect(cw >= 4 && cw <= 32 && cw % 4 == 0, "a compiled chunk");
            }
    return bad;
}

// The tiled solve's states are allocated where a tiled schedule or the per-term form
// runs; the default's steps have their records alone.
int chain_states() {
    rexi_plan* pl = make_plan(100, 21, 64);
    const size_t states = (size_t)64 * (pl->nslots + 2) * 16;
    expect(used < states, "a plan without states");
    expect(step(pl, 1) == REXI_OK && step(pl, 8) == REXI_OK, "steps");
    for (const auto& a : live) expect(a.second != states, "no states of the tiled solve");
    expect(rexi_step_noalloc(pl, kIn, kOut, 1, 1, nullptr) == REXI_OK, "a no-allocation step");
    expect(rexi_step_per_term(pl, kIn, kOut, 2, nullptr) == REXI_OK, "a step in the per-term form");
    destroy(pl);
    rexi_params p = make_plan_params(26, 20, 4);
    p.omega = 0;  // the default is a tiled schedule
    expect(rexi_plan_create(&p, &pl) == REXI_OK, "a plan without rotation");
    expect(step(pl, 2) == REXI_OK && step(pl, 4) == REXI_OK, "tiled steps");
    destroy(pl);
    for (bool term : {true, false})
        fail_every("tiled states", 40, 21, [](rexi_plan* q) {
            return rexi_plan_set_schedule(q, 2, 0, nullptr) ? -99 : step(q, 1);  // (0: a tiled one)
        }, [term](rexi_plan* q) { return term ? rexi_step_per_term(q, kIn, kOut, 2, nullptr) : step(q, 2); });
    fail_every("a tiled schedule", 40, 21, [](rexi_plan* q) { return step(q, 2); }, [](rexi_plan* q) {
        const int rc = rexi_plan_set_schedule(q, 2, 0, nullptr);
        return rc ? rc : step(q, 2);
    });
    return bad;
}

// The autotuner keeps a persistent schedule only where it is faster than every other by
// more than 3%, whatever the order of the candidates.
int autotune_margin() {
    struct Case {
        double first, second, ordinary;  // ms a step: the first and the last persistent candidate, an ordinary one between them
        int want;
    };
    const int S = 2;
    // (want: 0 the first, 1 the second, 2 the ordinary one)
    for (const Case& c : {Case{0.99, 2, 1.00, 2}, Case{2, 0.99, 1.00, 2}, Case{0.95, 2, 1.00, 0}, Case{2, 0.95, 1.00, 1},
                          Case{0.96, 0.95, 1.00, 1}, Case{0.95, 0.96, 1.00, 0}, Case{1.50, 1.60, 1.00, 2}}) {
        rexi_plan* pl = make_plan(26, 20, 4);  // (a plan's graphs hold their times)
        int n = 0, index = -1, at[3] = {-1, -1, -1};
        expect(rexi_plan_set_schedule(pl, S, -1, &n) == REXI_OK, "the schedules");
        const std::vector<Schedule>& list = pl->sched[S];
        for (int i = 0; i < n; ++i) {
            if (list[i].persistent && at[0] < 0) at[0] = i;
            if (list[i].persistent) at[1] = i;
            else if (at[0] >= 0) at[2] = i;
        }
        expect(at[0] >= 0 && at[0] < at[2] && at[2] < at[1], "candidates of both kinds in turn");
        cost = [&](const Schedule& sc) {
            const int i = (int)(&sc - list.data());
            return i == at[0] ? c.first : i == at[1] ? c.second : i == at[2] ? c.ordinary : 3.0;
        };
        expect(rexi_plan_autotune(pl, S, nullptr, &index) == REXI_OK && index == at[c.want] && pl->chosen[S] == index,
               "candidate " + std::to_string(at[c.want]) + ", got " + std::to_string(index));
        cost = nullptr;
        destroy(pl);
    }
    return bad;
}

const std::map<std::string, int (*)()> kScenarios = {
    {"handled_failure", handled_failure},
    {"failed_growth", failed_growth},
    {"failed_tables", failed_tables},
    {"shortage", shortage},
    {"captured_buffers", captured_buffers},
    {"noalloc_untimed", noalloc_untimed},
    {"host_allocations", host_allocations},
    {"noalloc_selection", noalloc_selection},
    {"noalloc_routes", noalloc_routes},
    {"few_poles", few_poles},
    {"inverse_chunks", inverse_chunks},
    {"chain_states", chain_states},
    {"autotune_margin", autotune_margin},
};

}  // namespace

int main(int argc, char** argv) {
    const auto it = kScenarios.find(argc > 1 ? argv[1] : "");
    if (it == kScenarios.end()) return 2;
    return it->second() ? 1 : 0;
}
