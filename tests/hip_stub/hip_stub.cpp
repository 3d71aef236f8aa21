// The HIP runtime and the kernel launchers, as far as mgk_host.cpp uses them, on the CPU: device
// memory is host memory, kernels only leave a line in a log.  Built together with mgk_host.cpp and
// mgk_reorder.cpp by tests/host_runtime.py, so that the host path of a solve (streams, recording,
// lifetimes, memory that runs out, how pairs are grouped) can be tested without a GPU.
//
// Work on a stream ends at once, unless the test holds the stream: then it ends when something waits
// for it.  A stream that waits for an event of such work is held too, and ordered behind it.  A test can also set a limit
// on device memory, mark streams as recording and have launches of a kernel fail.  Launches of the on-chip solvers are
// looked over as the kernels do it: every job has to fit the launch shape.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../../paper_1910_06310_amd/csrc/mgk_launch.h"

namespace {

typedef std::map<void*, uint64_t> Behind;            // stream -> what was enqueued on it up to there
struct Event { void* stream; bool done; Behind behind; };

std::map<char*, size_t> device_memory;              // block -> bytes
size_t in_use = 0, limit = SIZE_MAX, pinned_bytes = 0;
std::set<void*> held, recording;                    // streams
std::map<void*, std::map<char*, uint64_t>> readers; // held stream -> blocks its work uses, the last time each
std::map<void*, Behind> waited;                     // stream -> what its work is ordered behind
uint64_t now = 0;
std::set<Event*> events;
std::string log_text;
std::vector<std::string> violations;
std::map<std::string, int> counts;
int device = 0;
int converge_after = 3;
std::string failing;                                // kernel whose launches fail
hipStreamCaptureMode capture_mode = hipStreamCaptureModeGlobal;   // of the calling thread

void say(const char* fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    log_text += buf;
    log_text += '\n';
}

char* block_of(const void* p) {
    auto it = device_memory.upper_bound((char*)p);
    if (it == device_memory.begin()) return nullptr;
    --it;
    return (char*)p < it->first + it->second ? it->first : nullptr;
}

void finish(void* stream) {
    held.erase(stream);
    readers.erase(stream);
    if (waited.count(stream)) {
        const Behind before = waited[stream];
        waited.erase(stream);
        for (auto& b : before) finish(b.first);
    }
    for (Event* e : events)
        if (e->stream == stream) e->done = true;
}

void finish_all() {
    while (!held.empty()) finish(*held.begin());
}

void reads(void* stream, const void* p) {
    if (char* b = block_of(p))
        if (held.count(stream)) readers[stream][b] = ++now;
}

void* const no_stream = (void*)-1;
void check_write(const void* p, void* stream = no_stream) {   // not what unfinished work uses, unless behind it
    char* b = block_of(p);
    if (!b) { violations.push_back("write outside device memory"); return; }
    for (auto& r : readers)
        if (r.first != stream && r.second.count(b) && (!waited.count(stream) || waited[stream][r.first] < r.second[b]))
            violations.push_back("write to a block that work under way reads");
}

bool breaks_recording() {   // what a thread may not do while any stream is recording, unless it has relaxed its mode
    if (recording.empty() || capture_mode == hipStreamCaptureModeRelaxed) return false;
    counts["broken recordings"]++;
    return true;
}

hipError_t launched(const char* name, void* stream, const MgkBatchDev* X = nullptr, const MgkBatchDev* Y = nullptr, int pairs = 0) {
    if (failing == name) return hipErrorLaunchFailure;
    say("%s pairs=%d%s", name, pairs, recording.count(stream) ? " recorded" : "");
    if (X) reads(stream, X->graphs);
    if (Y) reads(stream, Y->graphs);
    return hipSuccess;
}

// The schedule of a graph as outer operand of the reduced solver with W wavefronts, read as the kernel does: every row and
// every nonzero once, rows whole, black vertices not joined to each other, as many nonzeros as the descriptor says at most.
bool schedule_ok(const MgkBatchDev& X, int g, int W) {
    const MgkGraphDesc& d = X.graphs[g];
    const uint16_t* split = X.red_split + (int64_t)g * MGK_RED_SPLIT_STRIDE + MGK_RED_SPLIT(W);
    const uint16_t* order = X.red_order + 3 * (int64_t)d.voff + MGK_RED_LIST(W) * d.n;
    const uint32_t* sched = X.list_sched + d.soff + MGK_RED_LIST(W) * d.nnz;
    const MgkEntry* list = X.list_outer + d.zoff;
    std::vector<int> place(d.n, -1), nonzero(d.nnz, 0), row(d.n, 0);
    for (int k = 0; k < d.n; ++k) {
        if (order[k] >= d.n || place[order[k]] >= 0) return false;
        place[order[k]] = k;
    }
    for (int w = 0; w < W; ++w) {
        const int begin = split[w], end = split[w + 1], blacks = split[W + 1 + w];
        if (begin > end || begin + blacks > end || end > d.nnz) return false;
        if (blacks > d.red_need[2 * MGK_RED_LIST(W)] || end - begin - blacks > d.red_need[2 * MGK_RED_LIST(W) + 1]) return false;
        int at[2] = {split[2 * W + 1 + w], split[3 * W + 1 + w]};   // place of the first row
        for (int k = begin; k < end; ++k) {
            const bool red = k >= begin + blacks;
            const int from = sched[k] & 0xffff, col = sched[k] >> 16;
            if (from >= d.nnz || nonzero[from]++) return false;
            const MgkEntry& e = list[from];
            if ((int)e.x != order[at[red]] || place[e.y] != col) return false;
            if ((place[e.x] < d.n_red) != red || (!red && col >= d.n_red)) return false;
            if (e.w >> 31) row[at[red]++]++;
        }
    }
    if (split[W] != d.nnz) return false;
    std::vector<int> ends(d.n, 0);
    for (int k = 0; k < d.nnz; ++k) ends[place[list[k].x]] |= list[k].w >> 31;
    return ends == row;
}

// Launches of the on-chip solvers: fits(batch and number of the outer graph, outer graph, inner graph) for every job, those
// of a swapped one from the other batch if the kernel takes both orientations.
template <class Fits>
hipError_t launched_jobs(const char* name, void* stream, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n,
                         size_t lds_bytes, bool both, const Fits& fits) {
    if (lds_bytes > MGK_LDS_LIMIT_BYTES) return hipErrorInvalidValue;
    for (int k = 0; k < n; ++k) {
        const bool other = both && jobs[k].out1 == MGK_OUT1_SWAPPED;
        const MgkBatchDev &O = other ? Y : X, &I = other ? X : Y;
        if (!fits(O, jobs[k].g1, O.graphs[jobs[k].g1], I.graphs[jobs[k].g2]))
            violations.push_back(std::string("a job of ") + name + " does not fit its launch");
    }
    return launched(name, stream, &X, &Y, n);
}

}  // namespace

extern "C" {

// ---- for the tests
void stub_reset() {
    finish_all();
    recording.clear();
    log_text.clear();
    violations.clear();
    counts.clear();
    limit = SIZE_MAX;
    converge_after = 3;
    failing.clear();
    capture_mode = hipStreamCaptureModeGlobal;
}
void stub_fail(const char* kernel) { failing = kernel; }
void stub_clear_log() { log_text.clear(); }
const char* stub_log() { return log_text.c_str(); }
int stub_count(const char* what) { return counts[what]; }
const char* stub_violations() {
    static std::string all;
    all.clear();
    for (const std::string& v : violations) all += v + "\n";
    return all.c_str();
}
void stub_hold(void* stream) { held.insert(stream); }
void stub_record(void* stream, int on) { if (on) recording.insert(stream); else recording.erase(stream); }
// The stream is destroyed with work under way and its handle given to a new one: the work goes on
// under a name that nothing else has.
void stub_replace_stream(void* stream) {
    if (!held.erase(stream)) return;
    void* name = new char;
    held.insert(name);
    readers[name].swap(readers[stream]);
    waited[name].swap(waited[stream]);
    auto rename = [&](Behind& b) {
        if (!b.count(stream)) return;
        b[name] = b[stream];
        b.erase(stream);
    };
    for (auto& w : waited) rename(w.second);
    for (Event* e : events)
        if (!e->done) {
            if (e->stream == stream) e->stream = name;
            rename(e->behind);
        }
}
void stub_set_limit(int64_t bytes) { limit = bytes < 0 ? SIZE_MAX : (size_t)bytes; }
int64_t stub_in_use() { return (int64_t)in_use; }
int64_t stub_pinned() { return (int64_t)pinned_bytes; }
void stub_converge_after(int iterations) { converge_after = iterations; }
void stub_set_device(int d) { device = d; }
int stub_device() { return device; }
// First elements that a thread of the vector kernels is given: how many, the smallest and the largest.
int64_t stub_quads(int block, int blocks, int thread, int end, int64_t* range) {
    int64_t n = 0;
    range[0] = INT64_MAX;
    range[1] = INT64_MIN;
    mgk_each_quad(block, blocks, thread, end, [&](int32_t at) {
        ++n;
        range[0] = std::min<int64_t>(range[0], at);
        range[1] = std::max<int64_t>(range[1], at);
    });
    return n;
}
int stub_lean_blocks(int64_t n_pairs, int max_npad) { return mgk_lean_blocks(n_pairs, max_npad); }

// ---- the runtime
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { device = d; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "stub error"; }
hipError_t hipMalloc(void** p, size_t bytes) {
    counts["malloc"]++;
    if (breaks_recording()) return hipErrorStreamCaptureUnsupported;
    if (bytes > limit || in_use + bytes > limit) return hipErrorOutOfMemory;
    *p = malloc(bytes ? bytes : 1);
    device_memory[(char*)*p] = bytes;
    in_use += bytes;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
    if (breaks_recording()) return hipErrorStreamCaptureUnsupported;
    finish_all();   // waits for the device
    counts["free"]++;
    auto it = device_memory.find((char*)p);
    if (it == device_memory.end()) { violations.push_back("free of unknown memory"); return hipErrorInvalidValue; }
    in_use -= it->second;
    device_memory.erase(it);
    free(p);
    return hipSuccess;
}
static std::map<void*, size_t> pinned;
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    *p = malloc(bytes);
    pinned[*p] = bytes;
    pinned_bytes += bytes;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { pinned_bytes -= pinned[p]; pinned.erase(p); free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    if (breaks_recording()) return hipErrorStreamCaptureUnsupported;
    if (k == hipMemcpyHostToDevice) check_write(d);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) {
    if (recording.count(st)) counts["recorded copies"]++;
    if (k == hipMemcpyHostToDevice) check_write(d, st);
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) { check_write(d, st); memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    counts["stream waits"]++;
    if (recording.count(s)) { counts["broken recordings"]++; return hipErrorStreamCaptureUnsupported; }
    if (breaks_recording()) return hipErrorStreamCaptureUnsupported;
    finish(s);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, capture_mode); return hipSuccess; }
hipError_t hipDeviceSynchronize() { counts["device waits"]++; if (breaks_recording()) return hipErrorStreamCaptureUnsupported; finish_all(); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = recording.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    Event* ev = new Event{nullptr, true, {}};
    events.insert(ev);
    *e = (hipEvent_t)ev;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { events.erase((Event*)e); delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    Event* ev = (Event*)e;
    if (recording.count(s)) counts["recorded events"]++;
    ev->stream = s;
    ev->done = held.count(s) == 0;
    ev->behind.clear();
    if (waited.count(s)) ev->behind = waited[s];
    ev->behind[s] = ++now;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    Event* ev = (Event*)e;
    if (recording.count(s)) counts["recorded waits"]++;
    if (ev->done || ev->stream == s) return hipSuccess;
    for (auto& b : ev->behind)
        if (b.first != s) waited[s][b.first] = std::max(waited[s][b.first], b.second);
    held.insert(s);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return ((Event*)e)->done ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t e) { counts["event waits"]++; if (!((Event*)e)->done) finish(((Event*)e)->stream); return hipSuccess; }

}  // extern "C"

// ---- the launchers
#define STUB_SMALL(NAME, W)                                                                                       \
    hipError_t NAME(int ept, bool, bool, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n, const MgkParams&, \
                    size_t lds, const MgkOutputs&, hipStream_t s) {                                               \
        return launched_jobs("small", s, X, Y, jobs, n, lds, false,                                               \
                             [=](const MgkBatchDev& O, int g, const MgkGraphDesc& a, const MgkGraphDesc& b) { return a.n * b.n <= W * 64 * ept; }); \
    }
STUB_SMALL(mgk_launch_small_w1, 1) STUB_SMALL(mgk_launch_small_w2, 2) STUB_SMALL(mgk_launch_small_w4, 4)
STUB_SMALL(mgk_launch_small_w8, 8) STUB_SMALL(mgk_launch_small_w16, 16) STUB_SMALL(mgk_launch_small_w4_fine, 4)
#define STUB_REGS(W, C)                                                                                           \
    hipError_t mgk_launch_regs_w##W##_c##C(int ept, bool, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n, \
                                           const MgkParams&, size_t lds, const MgkOutputs&, hipStream_t s) {      \
        return launched_jobs("regs", s, X, Y, jobs, n, lds, false, [=](const MgkBatchDev& O, int g, const MgkGraphDesc& a, const MgkGraphDesc& b) { \
            const int run = W == 4 ? a.regs_runs & 0xffff : (int)((uint32_t)a.regs_runs >> 16);                   \
            return a.n * b.n <= W * 64 * ept && b.lane_len <= 64 * C && b.max_deg <= MGK_REGS_MAX_DEG &&           \
                   run <= (W == 4 ? MGK_REGS_SMAX_W4 : MGK_REGS_SMAX_W8);                                         \
        });                                                                                                       \
    }
STUB_REGS(4, 1) STUB_REGS(4, 2) STUB_REGS(8, 1) STUB_REGS(8, 2)
#define STUB_REDUCED(W, C)                                                                                        \
    hipError_t mgk_launch_reduced_w##W##_c##C(int ept, bool, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n, \
                                              const MgkParams&, size_t lds, const MgkOutputs&, hipStream_t s) {   \
        return launched_jobs("reduced", s, X, Y, jobs, n, lds, true, [=](const MgkBatchDev& O, int g, const MgkGraphDesc& a, const MgkGraphDesc& b) { \
            const uint8_t* need = a.red_need + 2 * MGK_RED_LIST(W);                                               \
            return need[0] <= MGK_RED_BLACK(W) && need[1] <= MGK_RED_RED(W) && b.lane_len <= 64 * C &&            \
                   b.max_deg <= MGK_REGS_MAX_DEG && a.n_red * b.n <= W * 64 * ept &&                              \
                   W * 64 * ept + (a.n - a.n_red) * b.n <= MGK_RED_MAX_P &&                                       \
                   (size_t)mgk_reduced_plan(a.n, a.n_red, b.n, W, ept).total * 4 <= lds &&                        \
                   schedule_ok(O, g, W);                                                                          \
        });                                                                                                       \
    }
STUB_REDUCED(2, 1) STUB_REDUCED(4, 1) STUB_REDUCED(4, 2) STUB_REDUCED(8, 1) STUB_REDUCED(8, 2)
#define STUB_PCG_SEP(RK)                                                                                          \
    hipError_t mgk_launch_pcg_sep_rk##RK(int waves, int ept, int, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList& SX, \
                                         const MgkSepList& SY, const MgkJob* jobs, int n, const MgkParams&, int rb, size_t lds, \
                                         const MgkOutputs&, hipStream_t s) {                                      \
        reads(s, SX.packets);                                                                                     \
        reads(s, SY.packets);                                                                                     \
        return launched_jobs("pcg_sep", s, X, Y, jobs, n, lds, false, [=](const MgkBatchDev& O, int g, const MgkGraphDesc& a, const MgkGraphDesc& b) { \
            return a.n * b.n <= waves * 64 * ept &&                                                               \
                   (size_t)mgk_pcg_sep_plan(std::max(a.n, b.n), std::min(a.n, b.n), RK, rb).total * 4 <= lds;     \
        });                                                                                                       \
    }
STUB_PCG_SEP(1) STUB_PCG_SEP(4) STUB_PCG_SEP(5) STUB_PCG_SEP(6) STUB_PCG_SEP(7)
#define STUB_SELL(W)                                                                                              \
    hipError_t mgk_launch_sell_w##W(int, int, const MgkBatchDev& X, const MgkBatchDev& Y, const MgkJob* jobs, int n, \
                                    const MgkParams&, size_t lds, const MgkOutputs&, hipStream_t s) {             \
        return launched_jobs("sell", s, X, Y, jobs, n, lds, false, [](const MgkBatchDev&, int, const MgkGraphDesc&, const MgkGraphDesc&) { return true; }); \
    }
STUB_SELL(4) STUB_SELL(8) STUB_SELL(16)
hipError_t mgk_noalloc_job_storage(int, MgkJob** jobs, int64_t* capacity) {
    static MgkJob* storage = nullptr;
    if (!storage) {
        storage = (MgkJob*)malloc(MGK_NOALLOC_MAX_PAIRS * sizeof(MgkJob));
        device_memory[(char*)storage] = MGK_NOALLOC_MAX_PAIRS * sizeof(MgkJob);
    }
    *jobs = storage;
    *capacity = MGK_NOALLOC_MAX_PAIRS;
    return hipSuccess;
}
hipError_t mgk_launch_expand(const MgkBatchDev& B, const MgkParams&, MgkEntry*, MgkEntry*, hipStream_t s) { return launched("expand", s, &B); }
hipError_t mgk_launch_expand_dense(const MgkBatchDev& B, const MgkParams&, float*, float*, float*, hipStream_t s) { return launched("expand_dense", s, &B); }
hipError_t mgk_launch_large_init(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkLargePair*, MgkPairState*, float*,
                                 const MgkParams&, bool, int n, int, hipStream_t s) { return launched("init", s, &X, &Y, n); }
hipError_t mgk_launch_large_iteration(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkExpanded&, const MgkExpanded&,
                                      const MgkLargePair*, MgkPairState*, float*, const MgkParams&, bool, int n, int, int,
                                      int* n_active, int it, const MgkDenseTiles* D, const MgkDenseTiles*, int rows, int, int, hipStream_t s) {
    if (it + 1 >= converge_after) { n_active[0] = 0; n_active[1] = it + 1; }
    return launched(D ? "direct dense" : rows > 0 ? "direct rows" : "direct gather", s, &X, &Y, n);
}
hipError_t mgk_launch_large_final(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkExpanded&, const MgkExpanded&,
                                  const MgkLargePair*, MgkPairState*, float*, const MgkParams&, bool, int n, int, int,
                                  const MgkDenseTiles*, const MgkDenseTiles*, int, int, int, const MgkOutputs&, hipStream_t s) { return launched("final", s, &X, &Y, n); }
static MgkSepBasis basis;
extern "C" const MgkSepBasis* stub_basis() { return &basis; }   // of the last features
hipError_t mgk_launch_sep_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepLayout&, const MgkSepList&, const MgkSepGraph*,
                               int n_used, int, float* packets, hipStream_t s) {
    basis = S;
    check_write(packets, s);
    reads(s, packets);   // as under way as a reader
    return launched("sep pack", s, &B, nullptr, n_used);
}
hipError_t mgk_launch_sep_dense_pack(const MgkBatchDev& B, const MgkSepBasis& S, const MgkSepGraph*, int n_used, int, float*, hipStream_t s) { basis = S; return launched("sep dense pack", s, &B, nullptr, n_used); }
hipError_t mgk_launch_sep_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList&, const MgkSepList&,
                              const MgkSepLayout&, const MgkLargePair*, const MgkSepAt*, MgkPairState*, float*, const MgkParams&, int n, int max_n1,
                              int, int, bool, hipStream_t s) {
    if ((int64_t)((n + 7) / 8) * 8 * ((max_n1 + 15) / 16) * 1024 >= (int64_t)1 << 32) return hipErrorInvalidConfiguration;
    return launched("sep", s, &X, &Y, n);
}
hipError_t mgk_launch_sep_dense(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkSepList&, const MgkSepList&, int, bool parts,
                                const MgkLargePair*, const MgkSepAt*, MgkPairState*, float*, const MgkParams&, int n, int max_n1, int max_n2, int, bool, hipStream_t s) {
    if ((int64_t)((n + 7) / 8) * 8 * ((max_n1 + 31) / 32) * 256 >= (int64_t)1 << 32) return hipErrorInvalidConfiguration;
    if (parts && !mgk_sep_in_parts(max_n1, max_n2)) return hipErrorInvalidValue;
    return launched("sep dense", s, &X, &Y, n);
}
#ifdef STUB_WIDE   // the library does without these kernels where they are not linked
// Features of the form for graphs of many vertices where the last call put them: first record (outer graphs) or word (inner ones) -> graph
// and end.
struct WidePlace { int32_t graph; int64_t end; };
typedef std::map<int64_t, WidePlace> WidePlaces;
static WidePlaces wide_outer, wide_inner;
static void wide_place(WidePlaces& places, int64_t at, int64_t size, int64_t total, int32_t graph) {
    const auto next = places.lower_bound(at);
    if (at < 0 || at + size > total || (next != places.end() && next->first < at + size) || (next != places.begin() && std::prev(next)->second.end > at))
        violations.push_back("features of a graph overlap others or leave their buffer");
    places[at] = {graph, at + size};
}
hipError_t mgk_launch_wide_pack(const MgkBatchDev& B, const MgkWideBasis&, const MgkWideLayout& L, const int32_t*, const MgkSepGraph* outer_used,
                                int n_outer, const MgkSepGraph* inner_used, int n_inner, int max_n, int64_t outer_total, float* outer, float* inner,
                                hipStream_t s) {
    if (n_outer > 0) {
        wide_outer.clear();
        wide_inner.clear();
    }
    for (const float* to : {outer, inner}) check_write(to, s);
    auto words = [](const float* to) { return (int64_t)(device_memory[block_of(to)] / 4); };
    if (outer_total * L.passes * mgk_wide_record(L.hi) > words(outer)) violations.push_back("records of outer graphs leave their buffer");
    for (int k = 0; k < n_outer + n_inner; ++k) {
        const MgkSepGraph& u = k < n_outer ? outer_used[k] : inner_used[k - n_outer];
        const MgkGraphDesc& g = B.graphs[u.graph];
        if (g.n > max_n) violations.push_back("a graph of more vertices than the launch says");
        if (k < n_outer) wide_place(wide_outer, u.at, g.nnz, outer_total, u.graph);
        else if (g.n > MGK_WIDE_MAX_N) violations.push_back("an inner graph of more vertices than the kernel's table of groups");
        else wide_place(wide_inner, u.at, mgk_wide_inner_words(g, L.passes), words(inner), u.graph);
    }
    if (n_outer > 0) launched("wide outer", s, &B, nullptr, n_outer);
    return n_inner > 0 ? launched("wide inner", s, &B, nullptr, n_inner) : hipSuccess;
}
hipError_t mgk_launch_wide_xmv(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkWideFeatures& F, const MgkWideLayout& L, const MgkWidePair* pairs,
                               MgkPairState*, float*, const MgkParams&, int n, int max_n1, int max_n2, int, bool, hipStream_t s) {
    if (L.rows <= 0 || max_n2 > MGK_WIDE_MAX_ELEMENTS / L.rows || mgk_wide_lds_bytes(L, max_n2) > MGK_LDS_LIMIT_BYTES ||
        mgk_wide_grid(n, max_n1, L.rows) * MGK_WIDE_THREADS >= (int64_t)1 << 32)
        return hipErrorInvalidConfiguration;
    for (int k = 0; k < n; ++k) {
        const MgkWidePair& P = pairs[k];
        const auto o = wide_outer.find(P.f1), i = wide_inner.find(P.f2);
        if (o == wide_outer.end() || i == wide_inner.end()) { violations.push_back("a pair without features"); continue; }
        const MgkGraphDesc &a = X.graphs[o->second.graph], &b = Y.graphs[i->second.graph];
        if (P.n1 != a.n || P.n2 != b.n || P.n1 > max_n1 || P.n2 > max_n2 || P.nnz1 != a.nnz || P.voff1 != a.voff || P.voff2 != b.voff ||
            P.cap2 != mgk_wide_steps(b) || P.npad < a.n * b.n)
            violations.push_back("a pair with features of other graphs");
    }
    reads(s, F.outer);
    reads(s, F.inner);
    return launched("wide", s, &X, &Y, n);
}
#endif
hipError_t mgk_launch_large_vectors(const MgkLargePair*, MgkPairState*, float*, int n, int, int it, float, int* n_active, hipStream_t s) {
    if (it + 1 >= converge_after) { n_active[0] = 0; n_active[1] = it + 1; }
    return launched("vectors", s, nullptr, nullptr, n);
}
hipError_t mgk_launch_large_outputs(const MgkBatchDev& X, const MgkBatchDev& Y, const MgkLargePair*, MgkPairState*, float*,
                                    const MgkParams&, int n, int, const MgkOutputs&, int, hipStream_t s) { return launched("outputs", s, &X, &Y, n); }
hipError_t mgk_launch_normalize(float*, float*, int, hipStream_t s) { return launched("normalize", s); }
