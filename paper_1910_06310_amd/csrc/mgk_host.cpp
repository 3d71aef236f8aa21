// C ABI of the solver: contexts, graph loading (validate, reorder, cut into
// octiles, bitmap-pack, upload), job lists and kernel launches.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <numeric>
#include <optional>
#include <stdexcept>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include <unistd.h>

#include "../../include/mgk.h"
#include "mgk_internal.h"
#include "mgk_launch.h"
#include "mgk_reorder.h"

namespace {

constexpr int kTile = 8;

// What the separable product of a streaming on-chip solve would take, for the choice at launch (the edge
// kernel's parameters and label ranges are not known before); of a pair, or over the pairs of a launch.
struct SepWork {
    int32_t rows = 0, cols = 0, elements = 0;   // most vertices of a larger and of a smaller graph, most n n'
    int64_t entries = 0;                        // pairs of nonzeros, nnz nnz'
    int64_t halves = 0;                         // nnz n' + n nnz'
    int64_t blocks = 0;                         // of 16 rows
    void add(const SepWork& s) {
        rows = std::max(rows, s.rows);
        cols = std::max(cols, s.cols);
        elements = std::max(elements, s.elements);
        entries += s.entries;
        halves += s.halves;
        blocks += s.blocks;
    }
};

SepWork sep_work(const MgkGraphDesc& a, const MgkGraphDesc& b) {
    SepWork s;
    s.rows = std::max(a.n, b.n);
    s.cols = std::min(a.n, b.n);
    s.elements = (int32_t)((int64_t)a.n * b.n);
    s.entries = (int64_t)a.nnz * b.nnz;
    s.halves = (int64_t)a.nnz * b.n + (int64_t)a.n * b.nnz;
    s.blocks = (s.rows + 15) / 16;
    return s;
}

struct JobBin {
    int64_t first = 0;   // index of the bin's first job in the job array
    int64_t count = 0;
    size_t lds_bytes = 0;
    int waves = 0, ept = 0;
    int chunks = 0;            // > 0: register-resident solver with this many inner chunks
    bool reduced = false;      // of the reduced system
    int sell_regs = 0;         // > 0: owner-computes solver with this many entry registers per lane
    bool atomic_rows = false;  // an inner graph has a row longer than one lane group
    bool swapped = false;      // outer graphs come from batch Y, inner from X
    SepWork sep;
};

struct JobList {
    MgkJob* dev = nullptr;
    int64_t n = 0;
    std::vector<JobBin> bins;
    // pairs whose vectors do not fit on chip: [outer graph from X / from Y]
    std::vector<MgkLargePair> large[2];
};

// growable device allocation owned by a context
struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
};

// Pinned host memory for what a call copies to the device without waiting: slots in turn, each used
// again when the call that copied out of it has completed.  All start in one block, allocated by the first
// call that needs it (30 us or more, and as much to give back: contexts that never do go without).
struct CallEnd;
constexpr size_t kSlotBytes = (size_t)128 << 10;
struct Staging {
    struct Slot {
        void* p = nullptr;
        size_t cap = 0;
        bool own = false;                // an allocation of its own, not part of the block
        bool open = false;               // copied from by a call whose end is not recorded (yet)
        hipStream_t stream = nullptr;    // of that call
        std::shared_ptr<CallEnd> end;    // of the last call
    } slot[4];
    void* block = nullptr;
    int next = 0;
};

// Device memory of freed batches, kept for the next ones (at most kMaxBlobs blocks of at most
// kMaxBlobBytes).  A block is handed out again when the calls that read its batch have completed.
constexpr size_t kMaxBlobs = 4, kMaxBlobBytes = (size_t)16 << 20;
constexpr size_t kMaxReads = 8;    // calls under way that a batch keeps track of
struct FreeBlob {
    void* p = nullptr;
    size_t cap = 0;
    std::vector<std::shared_ptr<CallEnd>> reads;
};
// Shared by a context and its batches: a batch may be freed after its context, and by another thread
// than the one that uses the context.
struct BatchMemory {
    std::mutex m;
    std::vector<FreeBlob> blobs;
    std::vector<hipEvent_t> events;   // of the device, not in use
    bool open = true;                 // until the context is destroyed
    ~BatchMemory() {
        for (hipEvent_t e : events) (void)hipEventDestroy(e);
    }
};
// Completes with the kernels of a call.  The event is recorded before the call returns, when its
// stream is there for certain; the stream is not looked at again.
struct CallEnd {
    std::shared_ptr<BatchMemory> memory;
    hipEvent_t event = nullptr;
    ~CallEnd() {
        if (!event) return;
        try {
            std::lock_guard<std::mutex> lock(memory->m);
            if (memory->events.size() < 4 * kMaxReads) { memory->events.push_back(event); return; }
        } catch (...) {
        }
        (void)hipEventDestroy(event);
    }
    bool over() {
        if (seen_over) return true;
        seen_over = hipEventQuery(event) == hipSuccess;
        if (!seen_over) (void)hipGetLastError();   // "not ready" is no error of a later launch
        return seen_over;
    }
    bool seen_over = false;
};

// Threads of a context for the host work of a call.  run(n, f, helpers) calls f(0) .. f(n - 1), on
// the calling thread and on at most `helpers` (and kMaxWorkers) others, and returns when all have
// returned; f must not throw.  The threads sleep in between and end with the pool.  They do not
// exist in a forked child, where waiting for them would never end: it starts its own, and what
// the parent's left is abandoned there.
class WorkerPool {
public:
    ~WorkerPool() {
        if (!crew_ || crew_->process != getpid()) return;
        crew_->end();
        delete crew_;
    }
    void run(int n, const std::function<void(int)>& f, int helpers = kMaxWorkers) {
        const int want = std::min({n - 1, helpers, kMaxWorkers, (int)std::thread::hardware_concurrency() - 1});
        if (want > 0) {
            try {
                if (!crew_ || crew_->process != getpid()) crew_ = new Crew;
                while ((int)crew_->threads.size() < want) crew_->threads.emplace_back([c = crew_] { c->work(); });
            } catch (...) {   // fewer threads, then
            }
        }
        if (want <= 0 || !crew_ || crew_->process != getpid() || crew_->threads.empty()) {
            for (int i = 0; i < n; ++i) f(i);
            return;
        }
        crew_->run(n, f, want);
    }

private:
    static constexpr int kMaxWorkers = 15;
    struct Crew {
        const pid_t process = getpid();
        std::mutex m;
        std::condition_variable wake, done;
        std::vector<std::thread> threads;
        const std::function<void(int)>* f = nullptr;
        int n = 0, taken = 0, left = 0;
        bool stop = false;
        void run(int count, const std::function<void(int)>& task, int want) {
            std::unique_lock<std::mutex> lock(m);
            f = &task;
            n = left = count;
            taken = 0;
            lock.unlock();
            for (int k = 0; k < want; ++k) wake.notify_one();
            lock.lock();
            take(lock);
            done.wait(lock, [this] { return left == 0; });
            f = nullptr;
        }
        void take(std::unique_lock<std::mutex>& lock) {   // tasks until none is left to take
            while (f && taken < n) {
                const int i = taken++;
                const std::function<void(int)>* task = f;
                lock.unlock();
                (*task)(i);
                lock.lock();
                if (--left == 0) done.notify_one();
            }
        }
        void work() {
            std::unique_lock<std::mutex> lock(m);
            while (true) {
                wake.wait(lock, [this] { return stop || (f && taken < n); });
                if (stop) return;
                take(lock);
            }
        }
        void end() {
            {
                std::lock_guard<std::mutex> lock(m);
                stop = true;
            }
            wake.notify_all();
            for (std::thread& t : threads) t.join();
        }
    };
    Crew* crew_ = nullptr;
};

}  // namespace

struct mgk_batch {
    mgk_ctx* owner = nullptr;
    std::shared_ptr<BatchMemory> memory;
    int32_t n_graphs = 0;
    int64_t n_vertices = 0, nnz = 0, n_tiles = 0, n_offdiag = 0;
    bool weighted = false;
    int label_dim = 1;
    double label_mean = 0.0;
    // host copies
    std::vector<MgkGraphDesc> graphs;
    std::vector<MgkTile> tiles;
    std::vector<float> w, e;
    std::vector<int32_t> perm;     // [n_vertices], perm[voff + old] = new
    std::vector<int64_t> vtx_off;  // [G+1]
    std::vector<MgkSellDesc> sell_desc;   // per graph, for the planner
    float label_lo = 0.f, label_hi = 0.f; // range of attribute 0 of the edge labels
    std::vector<int32_t> packet_off[2];   // [G+1], packet steps before each graph with 2 / 8 nonzeros per packet
    MgkSepList sep[2] = {};               // the batch's part of it for the two packet sizes
    // device
    void* blob = nullptr;
    size_t blob_cap = 0;
    std::vector<std::shared_ptr<CallEnd>> reads;   // calls that read the batch and may be under way
    bool untracked = false;             // others may be: freeing the batch waits for the device
    MgkBatchDev dev{};
    struct GramJobs {
        JobList list;
        int waves = 0;       // settings the list was built for: waves_per_pair
        int max_iter = 0;
        int limit = 0;       // on-chip limit
        int cache = 0;       // product cache
        int sorted = 0;      // schedule
        int attr_dim = -1;   // label attributes of the edge kernel (LDS plan)
        bool any_big = false, separable = false;   // streaming pairs too large for the separable product on chip; whether that might be taken
        bool joined = false; // pairs of the reduced solver are with the streaming one, see join_few
    } gram_jobs[2];          // small pairs by the full system, by the reduced one
    std::vector<void*> old_jobs;   // lists replaced while a graph was recorded, when none may be freed
};

struct KeptBasis {
    int kernel = -1;
    float param = 0.f, lo = 0.f, hi = 0.f;
    MgkSepBasis basis{};
    bool has_wide = false;
    MgkWideBasis wide{};   // for graphs of many vertices
};

struct mgk_ctx {
    int device = 0;
    std::string err;
    float q = 0.05f, h = 1.0f, length_scale = 1.0f, ke_const = 1.0f, rtol = 1e-6f;
    int edge_kernel = MGK_EK_CONST;
    int label_dim = 1;                          // attributes the edge kernel reads
    float attr_ls[MGK_MAX_LABEL_DIM] = {1.f, 1.f, 1.f, 1.f};  // length scales of kron_se / rconv_se
    float poly_c[MGK_POLY_MAX_COEF] = {};
    float poly_rho = 1.f;
    int max_iter = 0;
    int tile_path = MGK_TILE_AUTO;
    int waves = 0;
    int onchip_limit = MGK_SMALL_MAX_N;  // largest n n' given to the on-chip solver
    int product_cache = 1;      // small pairs keep their matrix entries in registers (2, 3: one of the two kernels only)
    int reduced_system = 1;     // small pairs: 0 full system, 1 reduced one where nobody sees the iterates, 2 reduced one
    int cost_sorted = 1;        // expensive pairs first inside a launch
    int row_staging = 1;        // global-memory sparse product stages rows of p in LDS
    JobList pair_jobs;          // reused by mgk_pairs
    int64_t pair_jobs_cap = 0;
    hipStream_t pair_jobs_stream = nullptr;
    bool pair_jobs_busy = false;
    hipStream_t fixed_jobs_stream = nullptr;   // last mgk_pairs_noalloc call of this context
    bool fixed_jobs_busy = false;
    // scratch of the global-memory solver
    DevBuf exp_outer[2], exp_inner[2];  // expanded entry lists of batch X / batch Y
    DevBuf dense_tiles[2][3];           // dense 8x8 expansions (weight, label, log2 weight)
    DevBuf sep_packets[2];              // packets of the separable product, batch X / batch Y
    DevBuf sep_dense[2];                // dense F_k of the graphs of batch X / batch Y
    DevBuf wide_outer, wide_inner;      // features of graphs of many vertices as outer and as inner ones
    DevBuf onchip_packets;              // packets of the separable product on chip, of both batches of a call
    std::vector<void*> old_packets;     // smaller ones before it, half as large each: kernels may still read them
    hipEvent_t onchip_packets_end = nullptr;   // of the last kernel that reads them
    bool features_in_use = false;       // by the call under way
    KeptBasis bases[4];                 // of the last label ranges and edge kernels, see sep_basis_for
    int next_basis = 0;
    DevBuf vec, lpairs, lstate, lactive, nodal_off, diag;
    int* active_host = nullptr;         // pinned: {pairs still iterating, most iterations needed}
    Staging staging;                    // pair records, job lists and offsets of a call on their way to the device
    std::shared_ptr<BatchMemory> memory;
    int64_t calls = 0;                  // solver calls so far
    bool idle = false;                  // the last call has waited for all of its kernels
    hipStream_t upload = nullptr;       // loading a batch does not wait for the caller's streams
    WorkerPool workers;
    int large_iter_guess = 12;          // iterations the last call of the global-memory solver needed
    std::string launch_log;             // kernels the last solve call enqueued, one line each
};

namespace {

mgk_status fail(mgk_ctx* ctx, mgk_status st, const char* fmt, ...) noexcept {
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        try { ctx->err = buf; } catch (...) { ctx->err.clear(); }   // capacity is reserved at creation
    }
    return st;
}

void log_launch(mgk_ctx* ctx, const char* fmt, ...) {
    char buf[256];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    ctx->launch_log += buf;
    ctx->launch_log += '\n';
}

#define MGK_HIP(ctx, call)                                                              \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(ctx, MGK_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

// Runs `body` and turns any C++ exception into a status, so that nothing unwinds
// across the C ABI.  The message is stored without allocating when memory is short.
template <class F>
mgk_status guarded(mgk_ctx* ctx, F&& body) noexcept {
    mgk_status st = MGK_EINVAL;
    const char* what = "unexpected exception";
    try {
        return body();
    } catch (const std::bad_alloc&) {
        st = MGK_ENOMEM;
        what = "out of host memory";
    } catch (const std::length_error&) {
        st = MGK_ELIMIT;
        what = "request exceeds the largest host array";
    } catch (const std::system_error&) {
        st = MGK_ENOMEM;
        what = "could not start a worker thread";
    } catch (...) {
    }
    if (ctx) {
        try { ctx->err = what; } catch (...) { ctx->err.clear(); }
    }
    return st;
}

// Arrays of a batch on their way into one block of memory, 256-byte aligned each.
struct BlobPlan {
    struct Part { size_t at; const void* src; size_t bytes; };
    std::vector<Part> parts;
    size_t total = 0;
    template <class T>
    size_t add(const std::vector<T>& v) {
        const size_t at = (total + 255) & ~(size_t)255;
        total = at + std::max<size_t>(v.size() * sizeof(T), 16);
        parts.push_back({at, v.data(), v.size() * sizeof(T)});
        return at;
    }
    void copy_to(char* dst) const {
        for (const Part& p : parts)
            if (p.bytes) memcpy(dst + p.at, p.src, p.bytes);
    }
};

// Contiguous division of the rows of a graph among `waves` wavefronts for the
// register-resident solver: bounds[w] .. bounds[w+1] are wavefront w's rows.  A row of
// deg nonzeros costs about 4 deg + 9 wave instructions of an XMV (two inner chunks: an
// address add and a multiply-add per nonzero and chunk, the row sums and the store at its
// end); the largest cost of a wavefront is made as small as whole rows allow (bisection
// on the bound, rows filled in greedily).  Returns the most nonzeros a wavefront gets.
int balanced_split(const std::vector<int32_t>& deg, int n, int waves, int32_t* bounds) {
    auto row_cost = [&](int i) { return (int64_t)4 * deg[i] + 9; };
    int64_t lo = 0, hi = 0;
    for (int i = 0; i < n; ++i) { lo = std::max(lo, row_cost(i)); hi += row_cost(i); }
    // no bound below the mean will do, and the mean and the longest row always do
    const int64_t mean = (hi + waves - 1) / waves;
    hi = std::min(hi, mean + lo);
    lo = std::max(lo, mean);
    auto parts_needed = [&](int64_t bound) {
        int parts = 1;
        int64_t cur = 0;
        for (int i = 0; i < n; ++i) {
            const bool over = cur + row_cost(i) > bound;   // without a branch: rows of molecules are hard to foresee
            parts += over;
            cur = (over ? 0 : cur) + row_cost(i);
        }
        return parts;
    };
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (parts_needed(mid) <= waves) hi = mid; else lo = mid + 1;
    }
    int w = 0, longest = 0, run = 0;
    int64_t cur = 0;
    bounds[0] = 0;
    for (int i = 0; i < n; ++i) {
        if (cur + row_cost(i) > lo) { bounds[++w] = i; cur = 0; run = 0; }
        cur += row_cost(i);
        run += deg[i];
        longest = std::max(longest, run);
    }
    while (w < waves) bounds[++w] = n;
    return longest;
}

// Schedule of a graph as outer operand of the reduced solver (see MgkReducedPlan), one graph after another.  New graphs
// are often few and compared at once, so that the schedules count: 4.4 us a molecule-like graph of 35 vertices with a
// scan over all vertices for the next one to colour, a branch for every row and nonzero and all three divisions, 2.0 us like this.
class ReducedSchedule {
public:
    static bool makes(const MgkGraphDesc& gd) { return gd.nnz <= MGK_RED_MAX_NNZ && gd.n < 65536; }

    // The graph's n vertices (deg_order: by descending degree) and nonzeros by rows; what is filled: its parts of list_sched,
    // red_split and red_order of MgkBatchDev.
    void make(MgkGraphDesc& gd, const int32_t* rowptr, const MgkEntry* entries, const int32_t* deg_order, uint32_t* list, uint16_t* split,
              uint16_t* order) {
        const int n = gd.n;
        for (int k = 0; k < gd.nnz; ++k) col_[k] = (uint16_t)entries[k].y;
        std::fill_n(col_ + gd.nnz, 4, (uint16_t)0);
        deg_.resize((size_t)n);
        for (int i = 0; i < n; ++i) deg_[(size_t)i] = (i + 1 < n ? rowptr[i + 1] : gd.nnz) - rowptr[i];
        gd.n_red = colour(n, rowptr);
        int count[2] = {}, nnz[2] = {};
        for (auto& r : rows_) r.resize((size_t)n);
        for (int k = 0; k < n; ++k) {   // by descending number of nonzeros
            const int i = deg_order[k], c = black_[(size_t)i];
            rows_[0][(size_t)count[0]] = rows_[1][(size_t)count[1]] = i;
            count[c]++;
            nnz[c] += deg_[(size_t)i];
        }
        pos_.resize((size_t)n);
        of_wave_.resize((size_t)n);
        divide<2>(gd, rowptr, count, nnz, list, split, order);
        divide<4>(gd, rowptr, count, nnz, list, split, order);
        // eight cost more than four wherever both fit, but for elements that only eight hold: more than 64 vertices against 32 red ones
        if (gd.red_need[2] > MGK_RED_BLACK(4) || gd.red_need[3] > MGK_RED_RED(4)) divide<8>(gd, rowptr, count, nnz, list, split, order);
    }

private:
    // black_[i] = 1 for a set of vertices of which no two are adjacent, found greedily (a vertex with the fewest undecided
    // neighbours next, the first of them; neighbours of a black vertex are red), at least one vertex red.
    // Molecule-like graphs have 55 % black vertices, rings 50 %.  Returns the number of red ones.
    int colour(int n, const int32_t* rowptr) {
        int count = 0, most = 0;
        slot_.resize((size_t)n);
        black_.assign((size_t)n, 1);   // as those without a neighbour stay
        for (int i = 0; i < n; ++i)
            if (deg_[(size_t)i] > 0) {
                slot_[(size_t)i] = (uint8_t)count;
                vertex_[count++] = i;
                most = std::max(most, deg_[(size_t)i]);
            }
        const int reds = count <= 64 ? colour_sets<1>(count, most, rowptr) : colour_sets<3>(count, most, rowptr);
        if (reds > 0) return reds;
        black_[0] = 0;   // no edges
        return 1;
    }
    // Sets of vertices as Q words of 64; plane p: bit p of the number of undecided neighbours.
    template <int Q>
    int colour_sets(int count, int most, const int32_t* rowptr) {
        static_assert(MGK_RED_MAX_NNZ <= 192, "a vertex with edges has one nonzero at least");
        uint64_t adj[64 * Q][Q], left[Q] = {}, plane[8][Q] = {};
        int planes = 0;
        while (most >> planes) ++planes;
        for (int c = 0; c < count; ++c) {
            const int i = vertex_[c], d = deg_[(size_t)i];
            for (int q = 0; q < Q; ++q) adj[c][q] = 0;
            for (int k = rowptr[i]; k < rowptr[i] + d; ++k) {
                const int u = slot_[col_[k]];
                adj[c][u >> 6] |= 1ull << (u & 63);
            }
            left[c >> 6] |= 1ull << (c & 63);
            for (int p = 0; p < planes; ++p) plane[p][c >> 6] |= (uint64_t)(d >> p & 1) << (c & 63);
        }
        int reds = 0;
        while (true) {
            uint64_t fewest[Q], any = 0;
            for (int q = 0; q < Q; ++q) any |= fewest[q] = left[q];
            if (any == 0) return reds;
            for (int p = planes - 1; p >= 0; --p) {   // those without the bit, if there are any
                uint64_t without[Q], some = 0;
                for (int q = 0; q < Q; ++q) some |= without[q] = fewest[q] & ~plane[p][q];
                for (int q = 0; q < Q; ++q) fewest[q] = some ? without[q] : fewest[q];
            }
            int v = 0;
            for (int q = Q - 1; q >= 0; --q)
                if (fewest[q]) v = 64 * q + __builtin_ctzll(fewest[q]);
            left[v >> 6] &= ~(1ull << (v & 63));
            uint64_t red[Q];
            for (int q = 0; q < Q; ++q) {
                red[q] = adj[v][q] & left[q];
                left[q] &= ~red[q];
            }
            for (int q = 0; q < Q; ++q)
                for (; red[q]; red[q] &= red[q] - 1) {
                    const int u = 64 * q + __builtin_ctzll(red[q]);
                    black_[(size_t)vertex_[u]] = 0;
                    ++reds;
                    for (int w = 0; w < Q; ++w) {   // one undecided neighbour less
                        uint64_t borrow = adj[u][w] & left[w];
                        for (int p = 0; p < planes; ++p) {
                            const uint64_t was = plane[p][w];
                            plane[p][w] = was ^ borrow;
                            borrow &= ~was;
                        }
                    }
                }
        }
    }

    // Rows of one colour (by descending number of nonzeros) divided among W wavefronts: each row goes to the
    // one with the least work so far.  A row of deg nonzeros costs about 4 deg + 9 wave instructions of a product
    // (two inner chunks: an address add and a multiply-add per nonzero and chunk, the row sums and the
    // store at its end).  rows_in[w]: rows wavefront w gets.  Returns the most nonzeros a wavefront gets.
    template <int W>
    int divide_rows(const std::vector<int32_t>& rows, int count, int* rows_in) {
        int32_t cost[W];   // times 8, and the wavefront
        int nnz[W] = {};
        for (int w = 0; w < W; ++w) cost[w] = w;
        std::fill_n(rows_in, W, 0);
        for (int k = 0; k < count; ++k) {   // those without any come last: nothing is stored for them
            const int d = deg_[(size_t)rows[(size_t)k]];
            int32_t least = cost[0];
            for (int w = 1; w < W; ++w) least = std::min(least, cost[w]);
            const int w = least & 7;
            cost[w] = least + 8 * (4 * d + 9);
            nnz[w] += d;
            of_wave_[(size_t)k] = (uint8_t)w;
            rows_in[w]++;
        }
        return *std::max_element(nnz, nnz + W);
    }

    template <int W>
    void divide(MgkGraphDesc& gd, const int32_t* rowptr, const int* count, const int* nnz, uint32_t* list, uint16_t* split, uint16_t* order) {
        constexpr int which = MGK_RED_LIST(W);
        // more nonzeros than the wavefronts hold: no need to divide them (the place stays, unread)
        if (nnz[0] > W * MGK_RED_RED(W) || nnz[1] > W * MGK_RED_BLACK(W)) return;
        uint16_t* sp = split + MGK_RED_SPLIT(W);
        uint16_t* ord = order + (int64_t)which * gd.n;
        int at = 0, rows_in[2][W];
        for (int c = 0; c < 2; ++c) {
            const int most = divide_rows<W>(rows_[c], count[c], rows_in[c]);
            gd.red_need[2 * which + 1 - c] = (uint8_t)std::min(most, 255);
            int next[W];
            for (int w = 0; w < W; ++w) {
                sp[(3 - c) * W + 1 + w] = (uint16_t)(next[w] = at);
                at += rows_in[c][w];
            }
            for (int k = 0; k < count[c]; ++k) {
                const int to = next[of_wave_[(size_t)k]]++, i = rows_[c][(size_t)k];
                pos_[(size_t)i] = (uint16_t)to;
                ord[to] = (uint16_t)i;
            }
        }
        uint32_t* out = sched_;
        for (int w = 0; w < W; ++w) {
            uint32_t* const begin = out;
            sp[w] = (uint16_t)(begin - sched_);
            for (int c = 1; c >= 0; --c) {
                const uint16_t* row = ord + sp[(3 - c) * W + 1 + w];
                for (int r = 0; r < rows_in[c][w]; ++r) {
                    const int k = rowptr[row[r]], d = deg_[row[r]];
                    for (int a = 0; a < 4; ++a)   // most rows have no more; the next one overwrites what is none of this row's
                        out[a] = (uint32_t)(k + a) | (uint32_t)pos_[col_[k + a]] << 16;
                    for (int a = 4; a < d; ++a) out[a] = (uint32_t)(k + a) | (uint32_t)pos_[col_[k + a]] << 16;
                    out += d;
                }
                if (c) sp[W + 1 + w] = (uint16_t)(out - begin);
            }
        }
        sp[W] = (uint16_t)(out - sched_);
        std::copy_n(sched_, gd.nnz, list + (int64_t)which * gd.nnz);
    }

    uint16_t col_[MGK_RED_MAX_NNZ + 4];        // columns of the nonzeros, then four zeros
    int32_t vertex_[MGK_RED_MAX_NNZ];          // those with edges
    uint32_t sched_[MGK_RED_MAX_NNZ + 4];
    std::vector<uint8_t> slot_, black_, of_wave_;
    std::vector<int32_t> deg_, rows_[2];
    std::vector<uint16_t> pos_;                // places of the vertices in the order
};

// attributes per edge label that the edge kernel reads (0 for the kernels on plain
// scalar labels); the streaming on-chip solver keeps them in LDS for the outer graph
int attr_dim_of(const mgk_ctx* ctx) {
    return ctx->edge_kernel == MGK_EK_KRON_SE || ctx->edge_kernel == MGK_EK_RCONV_SE ? ctx->label_dim : 0;
}

// Small pairs by the reduced system: its iterates are others than those of Alg. 1 on the full system, so by
// default only where a call does not show them (iteration counts) or stop at one of them (an iteration limit).
bool solve_reduced(const mgk_ctx* ctx, const int32_t* iters_dev) {
    if (!mgk_launch_reduced_w2_c1) return false;   // linked without the kernels
    return ctx->reduced_system == 2 || (ctx->reduced_system == 1 && !iters_dev && ctx->max_iter <= 0);
}

// Whether launches of the streaming on-chip solver may take the separable product on chip (mgk_pcg_sep.hip).
bool separable_on_chip(const mgk_ctx* ctx) {
    return mgk_launch_pcg_sep_rk5 && (ctx->edge_kernel == MGK_EK_SE || ctx->edge_kernel == MGK_EK_CONST) && ctx->tile_path == MGK_TILE_AUTO &&
           ctx->product_cache != 0 && ctx->waves == 0;
}

// Fewest wavefronts of its pairs.  Two do less work for a pair whose inner graph fits one chunk, but make a launch of their
// own: 5050 molecule-like pairs (2679 of them with two) 95 us, all with four 111; with fewer than a launch should have
// (kMinJobsPerLaunch) a launch more costs more.
int reduced_waves(int64_t n_pairs) { return n_pairs >= 4096 ? 2 : 4; }

bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) {   // the default stream while another one records
        (void)hipGetLastError();
        return true;
    }
    return status != hipStreamCaptureStatusNone;
}

// Calls that stage their lists in pinned memory are refused while a graph is recorded: a replay would
// copy what later calls have put there.
mgk_status refuse_capture(mgk_ctx* ctx, hipStream_t stream) {
    if (!capturing(stream)) return MGK_OK;
    return fail(ctx, MGK_EDEVICE, "operation not permitted when stream is capturing");
}

// While it lives the thread may allocate, and wait for streams that take no part in a recording, while a graph is recorded.
class RelaxedCapture {
public:
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }

private:
    hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

// What a call reads.  done() records its end, one event a call (4 us; a second one, behind the copies of the
// lists, took as long again); a batch of a call that fails on the way, that is part of a recorded graph, or
// that has too many calls under way, is waited for with the whole device.
class BatchReads {
public:
    BatchReads(mgk_batch* X, mgk_batch* Y) : b_{X, Y}, was_{X->untracked, Y->untracked} { X->untracked = Y->untracked = true; }
    // may_create: else the event is one that an earlier call has left
    void done(Staging& staging, hipStream_t stream, bool may_create, bool idle) {
        if (idle) {   // the call has waited for its kernels
            for (Staging::Slot& s : staging.slot)
                if (s.stream == stream) s.open = false;
            for (int k = 0; k < 2; ++k) b_[k]->untracked = was_[k];
            return;
        }
        const bool staged = std::any_of(std::begin(staging.slot), std::end(staging.slot), [](const Staging::Slot& s) { return s.open; });
        // nothing to gain: freeing waits already, or the batch is compared with itself, hardly just once
        if (!staged && ((was_[0] && was_[1]) || b_[0] == b_[1])) return;
        try {
            auto end = std::make_shared<CallEnd>();
            end->memory = b_[0]->memory;
            for (mgk_batch* b : b_) {     // calls end in the order they were made, or are kept a little longer
                auto first = std::find_if(b->reads.begin(), b->reads.end(), [](const std::shared_ptr<CallEnd>& r) { return !r->over(); });
                b->reads.erase(b->reads.begin(), first);
            }
            {
                std::lock_guard<std::mutex> lock(end->memory->m);
                std::vector<hipEvent_t>& spare = end->memory->events;
                if (!spare.empty()) { end->event = spare.back(); spare.pop_back(); }
            }
            if (!end->event && (!may_create || hipEventCreateWithFlags(&end->event, hipEventDisableTiming) != hipSuccess)) return;
            if (hipEventRecord(end->event, stream) != hipSuccess) { (void)hipGetLastError(); return; }
            for (Staging::Slot& s : staging.slot)
                if (s.open && s.stream == stream) {
                    s.open = false;
                    s.end = end;
                }
            for (int k = 0; k < (b_[0] == b_[1] ? 1 : 2); ++k)
                if (b_[k]->reads.size() < kMaxReads) {
                    b_[k]->reads.push_back(end);
                    b_[k]->untracked = was_[k];
                }
        } catch (...) {   // out of memory: untracked
        }
    }

private:
    mgk_batch* b_[2];
    const bool was_[2];
};

// the batches must carry the number of label attributes the edge kernel reads
mgk_status check_label_dim(mgk_ctx* ctx, const mgk_batch* X, const mgk_batch* Y) {
    if (attr_dim_of(ctx) == 0) return MGK_OK;
    if (X->label_dim != ctx->label_dim || Y->label_dim != ctx->label_dim)
        return fail(ctx, MGK_ESTATE, "edge kernel reads %d label attributes, the batches hold %d and %d",
                    ctx->label_dim, X->label_dim, Y->label_dim);
    return MGK_OK;
}

MgkParams make_params(const mgk_ctx* ctx, const mgk_batch* X) {
    MgkParams p{};
    p.q = ctx->q;
    p.h = ctx->h;
    const double log2e = 1.4426950408889634;
    const double alpha = 1.0 / (2.0 * (double)ctx->length_scale * (double)ctx->length_scale);
    p.e_scale = (float)std::sqrt(alpha * log2e);  // exp(-a d^2) = exp2(-(d sqrt(a log2 e))^2)
    p.e_shift = (float)X->label_mean;
    if (ctx->edge_kernel == MGK_EK_POLY) p.e_scale = 1.0f / ctx->poly_rho;
    p.label_dim = ctx->edge_kernel == MGK_EK_KRON_SE || ctx->edge_kernel == MGK_EK_RCONV_SE ? ctx->label_dim : 1;
    for (int a = 0; a < MGK_MAX_LABEL_DIM; ++a) {
        const double l = ctx->attr_ls[ctx->edge_kernel == MGK_EK_RCONV_SE ? 0 : a];
        p.attr_scale[a] = (float)std::sqrt(log2e / (2.0 * l * l));
    }
    for (int i = 0; i < MGK_POLY_MAX_COEF; ++i) p.poly_c[i] = ctx->poly_c[i];
    p.ke_const = ctx->ke_const;
    p.rtol2 = ctx->rtol * ctx->rtol;
    p.max_iter = ctx->max_iter;
    p.edge_kernel = ctx->edge_kernel;
    return p;
}

// Launch shapes of the on-chip solver: `waves` wavefronts per pair, `ept`
// vector elements per thread; a pair fits when n n' <= waves * 64 * ept.
struct SmallConfig { int waves, ept; };
const SmallConfig kAutoConfigs[] = {{1, 4}, {2, 4}, {4, 4}, {4, 6}, {4, 8}, {4, 10}, {4, 12}, {4, 14}, {4, 16}, {8, 12}, {8, 16}, {16, 10}, {16, 12}, {16, 16}};
const int kEpts[] = {4, 8, 12, 16};

// Orientation, launch shape and cost of one pair for the on-chip solver.  The
// inner graph's nonzeros are spread over lanes in chunks of 64, the outer
// graph's are streamed, so the work is z_outer * ceil(z_inner / 64) wave
// iterations.
struct PairPlan {
    bool swap = false;   // true: Y's graph is the outer one
    bool atomic_rows = false;
    int64_t cost = 0;
    int64_t lds_words = 0;
    int waves = 0, ept = 0;  // 0: does not fit
    int chunks = 0;          // > 0: register-resident solver
    bool reduced = false;    // of the reduced system
    int sell_regs = 0;       // > 0: owner-computes solver
    int eliminated = 0;      // elements of the reduced system's black vertices
};

// Register-resident solver for (outer o, inner i) with `waves` wavefronts: every
// wavefront's run of outer rows must fit the unrolled loop, the inner layout the
// chunk registers, the vectors the register blocks.  Returns the cost in wave
// instructions of one iteration, or -1 if the pair does not fit.
int64_t regs_cost(const MgkGraphDesc& o, const MgkGraphDesc& i, int waves) {
    const int chunks = std::max(1, i.lane_len / 64);
    if (chunks > MGK_REGS_MAX_CHUNKS || i.max_deg > MGK_REGS_MAX_DEG) return -1;
    const int smax = waves == 4 ? MGK_REGS_SMAX_W4 : MGK_REGS_SMAX_W8;
    const int run = waves == 4 ? (o.regs_runs & 0xffff) : (int)((uint32_t)o.regs_runs >> 16);
    if (run > smax) return -1;
    const int64_t N = (int64_t)o.n * i.n;
    const int64_t ept = std::max<int64_t>(1, (N + waves * 64 - 1) >> (waves == 4 ? 8 : 9));
    // register blocks that keep four wavefronts per SIMD resident
    if (ept > MGK_REGS_MAX_EPT) return -1;
    return (int64_t)o.nnz * (2 * chunks) + (int64_t)o.n * (1 + 4 * chunks) +
           (int64_t)waves * (8 * ept + 45);
}

// The same for the solver of the reduced system, both orientations and `fewest` to 8 wavefronts: the cheapest (the first of
// equal ones, fewer wavefronts before more).  Returns false if the pair does not fit.
bool plan_reduced(PairPlan& pl, const MgkGraphDesc& a, const MgkGraphDesc& b, bool may_swap, int fewest) {
    struct Side {
        const MgkGraphDesc *o, *i;
        bool swap;
        int chunks, left, eliminated;   // elements
        int64_t cost;
    } side[2];
    int sides = 0;
    for (int sw = 0; sw < (may_swap ? 2 : 1); ++sw) {
        const MgkGraphDesc &o = sw ? b : a, &i = sw ? a : b;
        const int chunks = std::max(1, i.lane_len / 64);
        const int64_t left = (int64_t)o.n_red * i.n, all = (int64_t)o.n * i.n;   // on chip: 16384 at most
        if (chunks > MGK_REGS_MAX_CHUNKS || i.max_deg > MGK_REGS_MAX_DEG || left > 8 * 64 * MGK_REGS_MAX_EPT) continue;
        side[sides++] = {&o, &i, sw != 0, chunks, (int)left, (int)(all - left), (int64_t)o.nnz * (2 * chunks) + (int64_t)o.n * (1 + 4 * chunks)};
    }
    int64_t best = INT64_MAX;
    const Side* of_best = nullptr;
    for (int which = fewest == 2 ? 0 : fewest == 4 ? 1 : 2; which < 3; ++which)
        for (int k = 0; k < sides; ++k) {
            const Side& s = side[k];
            const int waves = 2 << which, ept = std::max(1, (s.left + waves * 64 - 1) >> (7 + which));
            const int64_t cost = s.cost + waves * (9 * ept + 90);
            const uint8_t* need = s.o->red_need + 2 * which;
            if (cost >= best || ept > MGK_REGS_MAX_EPT || need[0] > MGK_RED_BLACK(waves) || need[1] > MGK_RED_RED(waves) ||
                (waves == 2 && s.chunks > 1) || waves * 64 * ept + s.eliminated > MGK_RED_MAX_P)
                continue;
            const int32_t words = mgk_reduced_plan(s.o->n, s.o->n_red, s.i->n, waves, ept).total;
            if (words * 4 > MGK_LDS_LIMIT_BYTES) continue;   // many isolated vertices
            best = cost;
            of_best = &s;
            pl.waves = waves;
            pl.ept = ept;
            pl.lds_words = words;
        }
    if (!of_best) return false;
    pl.reduced = true;
    pl.swap = of_best->swap;
    pl.chunks = of_best->chunks;
    pl.cost = best * 16;
    pl.eliminated = of_best->eliminated;
    return true;
}

// Owner-computes solver for (outer o, inner i): the cheapest launch shape that holds the
// pair.  Cost in wave instructions of one iteration: the entries of the most loaded
// wavefront (a gather, weighted by its bank conflicts, and a multiply-add each), the
// vector part per slot, the three workgroup sums, and the share of the compute unit the
// workgroup occupies.  Returns -1 when no shape fits.
int64_t sell_cost(const MgkSellDesc& o, const MgkSellDesc& i, int* waves, int* ept, int* regs) {
    int64_t best = -1;
    for (int w = 4; w <= 16; w *= 2) {
        int32_t slots = 0, executed = 0;
        const int32_t need = mgk_sell_need(o, i, w, &slots, &executed);
        for (const MgkSellShape& sh : kMgkSellShapes)
            if (sh.waves == w && sh.ept >= slots && sh.regs >= need) {
                const int64_t c = (int64_t)executed * 4 + (int64_t)w * (13 * slots + 45);
                if (best < 0 || c < best) {
                    best = c;
                    *waves = w;
                    *ept = sh.ept;
                    *regs = sh.regs;
                }
                break;   // shapes of a workgroup size are listed smallest first
            }
    }
    return best;
}

// cache: 0 entries regenerated in every product; 1 (and 2) kept in registers by the kernel
// in which a wavefront owns rows of the outer graph; 3 by the owner-computes kernel where
// a pair fits it, else as 1.  reduced: fewest wavefronts for the solver of the reduced system, 0: the full one
PairPlan plan_pair(const MgkGraphDesc& a, const MgkGraphDesc& b, const MgkSellDesc* sa, const MgkSellDesc* sb,
                   bool may_swap, int forced_waves, int onchip_limit, int cache, int attr_dim, int reduced) {
    const bool product_cache = cache != 0;
    const int64_t N = (int64_t)a.n * b.n;
    const bool fits = N <= MGK_SMALL_MAX_N && N <= onchip_limit;
    PairPlan pl;
    if (fits && cache == 3 && forced_waves == 0 && attr_dim == 0 && sa && sb &&
        mgk_sell_ok(*sa) && mgk_sell_ok(*sb)) {
        int64_t best = -1;
        for (int sw = 0; sw < (may_swap ? 2 : 1); ++sw) {
            int w = 0, ept = 0, regs = 0;
            const int64_t c = sw ? sell_cost(*sb, *sa, &w, &ept, &regs) : sell_cost(*sa, *sb, &w, &ept, &regs);
            if (c >= 0 && (best < 0 || c < best)) {
                best = c;
                pl.waves = w;
                pl.ept = ept;
                pl.sell_regs = regs;
                pl.swap = sw != 0;
            }
        }
        if (best >= 0) {
            const MgkGraphDesc& o = pl.swap ? b : a;
            const MgkGraphDesc& i = pl.swap ? a : b;
            pl.atomic_rows = false;
            pl.chunks = 0;
            pl.cost = best * 16 + 16 * N;
            pl.lds_words = mgk_sell_plan(o.n, i.n, pl.waves, pl.ept).total;
            return pl;
        }
    }
    // the reduced system first; pairs that fit the full one only are solved with that
    if (fits && reduced && product_cache && forced_waves == 0 && plan_reduced(pl, a, b, may_swap, reduced)) return pl;
    // wave iterations of one XMV: outer nonzeros x 64-lane chunks of the inner layout
    auto passes = [](const MgkGraphDesc& o, const MgkGraphDesc& i) {
        return (int64_t)o.nnz * (i.lane_len / 64) + 2 * (int64_t)o.n * (i.lane_len / 64);
    };
    const int64_t keep = passes(a, b), swp = passes(b, a);
    const bool keep_atomic = b.max_deg > MGK_LANE_GROUP, swp_atomic = a.max_deg > MGK_LANE_GROUP;
    pl.swap = may_swap && (keep_atomic != swp_atomic ? keep_atomic : swp < keep);
    pl.atomic_rows = pl.swap ? swp_atomic : keep_atomic;
    pl.cost = (pl.swap ? swp : keep) * 64 + 16 * N;
    if (!fits) return pl;
    if (product_cache && forced_waves == 0) {
        int64_t best = -1;
        for (int w = 4; w <= 8; w *= 2)
            for (int sw = 0; sw < (may_swap ? 2 : 1); ++sw) {
                const int64_t c = sw ? regs_cost(b, a, w) : regs_cost(a, b, w);
                if (c >= 0 && (best < 0 || c < best)) { best = c; pl.waves = w; pl.swap = sw != 0; }
            }
        if (best >= 0) {
            const MgkGraphDesc& o = pl.swap ? b : a;
            const MgkGraphDesc& i = pl.swap ? a : b;
            pl.atomic_rows = false;
            pl.ept = (int)std::max<int64_t>(1, (N + pl.waves * 64 - 1) / (pl.waves * 64));
            pl.chunks = std::max(1, i.lane_len / 64);
            pl.cost = best * 16 + 16 * N;
            pl.lds_words = mgk_regs_plan(o.n, i.n, pl.waves, pl.ept).total;
            return pl;
        }
    }
    if (forced_waves > 0) {  // requested workgroup size, doubled until the pair fits
        for (int w = forced_waves; w <= 16 && pl.waves == 0; w *= 2)
            for (int e : kEpts)
                if ((int64_t)w * 64 * e >= N) { pl.waves = w; pl.ept = e; break; }
    } else {
        for (const SmallConfig& c : kAutoConfigs)
            if ((int64_t)c.waves * 64 * c.ept >= N) { pl.waves = c.waves; pl.ept = c.ept; break; }
    }
    if (pl.waves == 0) return pl;
    const MgkGraphDesc& o = pl.swap ? b : a;
    const MgkGraphDesc& i = pl.swap ? a : b;
    pl.lds_words = mgk_small_plan(o.n, i.n, o.nnz, i.lane_len, o.n_tiles, i.n_tiles, pl.waves, pl.ept, attr_dim).total;
    if (pl.lds_words * 4 > MGK_LDS_LIMIT_BYTES) pl.waves = pl.ept = 0;
    return pl;
}

// Launches of a call follow each other, and one with a few pairs takes as long as a pair does.  Where one of a few
// pairs needs the streaming solver with one wavefront (n n' <= 256), those of the reduced one go there too if they are
// as small: 36 + 9 pairs of 8 or 9 vertices 40.8 us in two launches, 25.0 in one.  Not where the caller has asked for
// the reduced system, whose iterations are then counted.  graphs(k): the two graphs of pair k.
constexpr size_t kFewPairs = 256;
template <class Graphs>
bool join_few(std::vector<PairPlan>& plans, const Graphs& graphs, int onchip_limit, int attr_dim) {   // whether any pair is moved
    if (plans.size() > kFewPairs) return false;
    bool one_wave[2] = {};   // [atomic rows]
    for (const PairPlan& pl : plans)
        if (pl.waves == 1) one_wave[pl.atomic_rows] = true;
    if (!one_wave[0] && !one_wave[1]) return false;
    bool any = false;
    std::vector<PairPlan> moved(plans);
    for (size_t k = 0; k < plans.size(); ++k) {
        if (!plans[k].reduced) continue;
        const auto g = graphs(k);
        moved[k] = plan_pair(*g.first, *g.second, nullptr, nullptr, true, 0, onchip_limit, 0, attr_dim, 0);
        if (moved[k].waves != 1 || !one_wave[moved[k].atomic_rows]) return false;
        any = true;
    }
    plans.swap(moved);
    return any;
}

// Pairs that the reduced solver does not take and the register-resident one of the full system does have a launch of their own.
// Where a few pairs need the streaming solver anyway, up to kFewFull of them go there too if that needs no other
// workgroup size: 60 ladders of 16 to 50 vertices (1830 pairs, 696 of that kind) 159 us in four launches, 118 in three; by
// themselves they are better off where their entries are kept (100 000 of them 4.68 and 5.26 ms, 250 50 and 74 us).
constexpr int kFewFull = 1024;
struct PlanKinds {   // of the pairs of a call
    std::atomic<int> full{0};
    std::atomic<uint32_t> streaming{0};   // launches of the streaming solver, see launch()
    static uint32_t launch(const PairPlan& pl, bool two_batches) {
        int size = 0;
        while (1 << size < pl.waves) ++size;
        return 1u << (4 * size + 2 * pl.atomic_rows + (pl.swap && two_batches));
    }
    struct Part {   // counted by one task
        int full = 0;
        uint32_t streaming = 0;
        void add(const PairPlan& pl, bool two_batches) {
            if (pl.reduced || pl.sell_regs > 0 || pl.waves == 0) return;
            if (pl.chunks > 0) ++full;
            else streaming |= launch(pl, two_batches);
        }
    };
    void add(const Part& p) {
        full += p.full;
        streaming |= p.streaming;
    }
};
template <class Graphs>
void join_full(std::vector<PairPlan>& plans, const PlanKinds& kinds, bool two_batches, const Graphs& graphs, int onchip_limit, int attr_dim) {
    if (kinds.full == 0 || kinds.full > kFewFull || kinds.streaming == 0 || plans.size() > 65536) return;   // more pairs: a launch does not count
    std::vector<std::pair<size_t, PairPlan>> moved;
    for (size_t k = 0; k < plans.size(); ++k) {
        if (plans[k].reduced || plans[k].chunks == 0) continue;
        const auto g = graphs(k);
        moved.emplace_back(k, plan_pair(*g.first, *g.second, nullptr, nullptr, true, 0, onchip_limit, 0, attr_dim, 0));
        if (moved.back().second.waves == 0 || !(kinds.streaming & PlanKinds::launch(moved.back().second, two_batches))) return;
    }
    for (const auto& m : moved) plans[m.first] = m.second;
}

// A launch shape: jobs of one shape go into one kernel launch.
struct Shape {
    uint32_t key = 0;          // of the six below, and big
    int16_t waves = 0, ept = 0, chunks = 0, sell_regs = 0;
    bool atomic_rows = false, swapped = false, reduced = false;
    bool big = false;          // too large for the separable product on chip, where that may be taken
    SepWork sep;
    int64_t count = 0;
    int64_t base_words = 0;    // largest LDS need of its jobs without the padded vectors
    int32_t eliminated = 0;    // most of a job
    int64_t min_cost = INT64_MAX, max_cost = 0;
    // padded vectors in the LDS plan of each solver (the owner-computes one also has a
    // schedule word per wavefront and slot; 4 words of alignment slack)
    int64_t vector_words() const {
        const int vectors = sell_regs > 0 ? 3 : chunks > 0 && !reduced ? 4 : 2;
        return (int64_t)vectors * waves * 64 * ept + (sell_regs > 0 ? waves * ept + 4 : 0);
    }
    int64_t lds_bytes() const { return (base_words + vector_words()) * 4; }
};

struct HostJob {
    MgkJob job;
    int64_t cost;
    int32_t shape;   // index into the list of shapes
};

// The jobs of a call, planned: every job with its launch shape.
struct JobPlan {
    std::vector<HostJob> jobs;
    std::vector<Shape> shapes;
    const bool separable;      // separable_on_chip()
    bool any_big = false;      // streaming pairs beyond it
    explicit JobPlan(bool sep) : separable(sep) { std::fill(table, table + kTable, (int16_t)-1); }
    // index of the shape of a planned pair of graphs a and b; counts the pair in (16 ns; 31 with a Shape made for every pair)
    int shape_of(const PairPlan& pl, bool swapped, const MgkGraphDesc& a, const MgkGraphDesc& b) {
        const bool streaming = pl.chunks == 0 && pl.sell_regs == 0;
        const bool beyond = streaming && (int64_t)a.n * b.n > MGK_PCG_SEP_MAX_N, big = beyond && separable;
        any_big = any_big || beyond;
        const uint32_t key = (uint32_t)pl.waves | (uint32_t)pl.ept << 5 | (uint32_t)pl.chunks << 10 | (uint32_t)pl.sell_regs << 13 |
                             (uint32_t)pl.atomic_rows << 20 | (uint32_t)swapped << 21 | (uint32_t)pl.reduced << 22 | (uint32_t)big << 23;
        uint32_t slot = (key * 2654435761u) >> 20;   // open addressing: there are far fewer shapes than slots
        while (table[slot] >= 0 && shapes[(size_t)table[slot]].key != key) slot = (slot + 1) % kTable;
        if (table[slot] < 0) {
            Shape s;
            s.key = key;
            s.waves = (int16_t)pl.waves;
            s.ept = (int16_t)pl.ept;
            s.chunks = (int16_t)pl.chunks;
            s.sell_regs = (int16_t)pl.sell_regs;
            s.atomic_rows = pl.atomic_rows;
            s.swapped = swapped;
            s.reduced = pl.reduced;
            s.big = big;
            table[slot] = (int16_t)shapes.size();
            shapes.push_back(s);
        }
        Shape& t = shapes[(size_t)table[slot]];
        t.count++;
        if (streaming) t.sep.add(sep_work(a, b));
        t.base_words = std::max(t.base_words, pl.lds_words - t.vector_words());
        t.eliminated = std::max(t.eliminated, pl.eliminated);
        t.min_cost = std::min(t.min_cost, pl.cost);
        t.max_cost = std::max(t.max_cost, pl.cost);
        return table[slot];
    }

private:
    static constexpr int kTable = 4096;
    int16_t table[kTable];
};

constexpr int64_t kMinJobsPerLaunch = 4096;
// A launch shape with few jobs costs more in launch and drain time than its pairs
// gain from the exact fit: such jobs move to the closest larger shape that can run
// them (same solver and workgroup size, at least as many elements per thread and
// inner chunks).  Only the vector blocks grow, so the LDS need grows by the
// difference of the padded vector lengths.  Returns the shape each shape's jobs end up in.

std::vector<int> merge_small_shapes(std::vector<Shape>& shapes) {
    std::vector<int> into(shapes.size());
    std::iota(into.begin(), into.end(), 0);
    std::vector<char> frozen(shapes.size(), 0);   // shapes whose jobs would outgrow LDS in the larger shape
    while (true) {
        // smallest shape below the threshold that has somewhere to go
        int from = -1, to = -1;
        for (size_t k = 0; k < shapes.size(); ++k) {
            const Shape& a = shapes[k];
            if (a.count == 0 || a.count >= kMinJobsPerLaunch || frozen[k]) continue;
            int best = -1;
            auto size = [&](int q) { return shapes[q].ept * 4 + shapes[q].chunks + shapes[q].sell_regs; };
            for (size_t q = 0; q < shapes.size(); ++q) {
                const Shape& b = shapes[q];
                if (q == k || b.count == 0 || a.waves != b.waves || a.atomic_rows != b.atomic_rows || a.swapped != b.swapped ||
                    a.reduced != b.reduced || a.big != b.big || (a.chunks > 0) != (b.chunks > 0) || b.chunks < a.chunks || b.ept < a.ept ||
                    (a.sell_regs > 0) != (b.sell_regs > 0) || b.sell_regs < a.sell_regs)
                    continue;
                if (best < 0 || size((int)q) < size(best)) best = (int)q;
            }
            if (best >= 0 && (from < 0 || a.ept * 4 + a.chunks < shapes[from].ept * 4 + shapes[from].chunks)) {
                from = (int)k;
                to = best;
            }
        }
        if (from < 0) break;
        Shape &a = shapes[from], &b = shapes[to];
        if ((a.base_words + b.vector_words()) * 4 > MGK_LDS_LIMIT_BYTES ||
            (a.reduced && b.waves * 64 * b.ept + a.eliminated > MGK_RED_MAX_P)) {   // of which the kernel keeps 16-bit offsets
            frozen[from] = 1;
            continue;
        }
        b.count += a.count;
        b.sep.add(a.sep);
        b.base_words = std::max(b.base_words, a.base_words);
        b.eliminated = std::max(b.eliminated, a.eliminated);
        b.min_cost = std::min(b.min_cost, a.min_cost);
        b.max_cost = std::max(b.max_cost, a.max_cost);
        a.count = 0;
        for (int& k : into)
            if (k == from) k = to;
    }
    return into;
}

mgk_status staging_slot(mgk_ctx* ctx, size_t bytes, bool may_allocate, hipStream_t stream, Staging::Slot** out);
void staging_copied(Staging::Slot* slot, hipStream_t stream);
hipError_t device_alloc(mgk_ctx* ctx, void** p, size_t bytes);
constexpr size_t kMaxStagedBytes = (size_t)4 << 20;

// Launch shapes largest first, inside a shape the expensive pairs first (in 256 steps of
// cost: near enough for balance, and one counting sort).  `fixed`: the job array is storage the
// caller provides (`out.dev` set, *capacity jobs); nothing is allocated or freed then.
mgk_status build_job_list(mgk_ctx* ctx, JobPlan& plan, JobList& out,
                          hipStream_t stream, int64_t* capacity, bool fixed = false) {
    std::vector<Shape>& shapes = plan.shapes;
    const std::vector<int> into = merge_small_shapes(shapes);
    std::vector<int> order;
    for (size_t k = 0; k < shapes.size(); ++k)
        if (shapes[k].count > 0) order.push_back((int)k);
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
        const Shape &a = shapes[x], &b = shapes[y];
        const int ka = a.waves * 64 * a.ept, kb = b.waves * 64 * b.ept;
        if (ka != kb) return ka > kb;
        if (a.waves != b.waves) return a.waves > b.waves;
        if (a.chunks != b.chunks) return a.chunks > b.chunks;
        if (a.sell_regs != b.sell_regs) return a.sell_regs > b.sell_regs;
        if (a.atomic_rows != b.atomic_rows) return a.atomic_rows;
        return !a.swapped && b.swapped;
    });
    out.bins.clear();
    out.n = (int64_t)plan.jobs.size();
    std::vector<int> rank(shapes.size(), 0);
    int64_t first = 0;
    for (size_t r = 0; r < order.size(); ++r) {
        const Shape& s = shapes[order[r]];
        rank[order[r]] = (int)r;
        JobBin b;
        b.first = first;
        b.count = s.count;
        b.lds_bytes = (size_t)s.lds_bytes();
        b.waves = s.waves;
        b.ept = s.ept;
        b.chunks = s.chunks;
        b.reduced = s.reduced;
        b.sell_regs = s.sell_regs;
        b.atomic_rows = s.atomic_rows;
        b.swapped = s.swapped;
        b.sep = s.sep;
        out.bins.push_back(b);
        first += s.count;
    }
    if (fixed) {
        if (out.n > *capacity) return fail(ctx, MGK_ELIMIT, "job list of %lld pairs exceeds the fixed storage of %lld",
                                           (long long)out.n, (long long)*capacity);
    } else if (capacity == nullptr || *capacity < out.n) {
        if (out.dev) MGK_HIP(ctx, hipFree(out.dev));
        out.dev = nullptr;
        const int64_t cap = std::max<int64_t>(out.n, 1);
        MGK_HIP(ctx, device_alloc(ctx, (void**)&out.dev, (size_t)cap * sizeof(MgkJob)));
        if (capacity) *capacity = cap;
    }
    if (out.n == 0) return MGK_OK;
    constexpr int kSteps = 256;
    std::vector<int32_t> at((size_t)order.size() * kSteps + 1, 0);
    auto bucket = [&](const HostJob& j) {
        const int k = into[j.shape];
        const Shape& s = shapes[k];
        int q = 0;
        if (ctx->cost_sorted && s.max_cost > s.min_cost)
            q = (int)((s.max_cost - j.cost) * (kSteps - 1) / (s.max_cost - s.min_cost));
        return (size_t)rank[k] * kSteps + (size_t)q;
    };
    std::vector<int32_t> where(plan.jobs.size());
    for (size_t k = 0; k < plan.jobs.size(); ++k) at[(size_t)(where[k] = (int32_t)bucket(plan.jobs[k])) + 1]++;
    for (size_t k = 1; k < at.size(); ++k) at[k] += at[k - 1];
    const size_t bytes = (size_t)out.n * sizeof(MgkJob);
    Staging::Slot* slot = nullptr;
    if (bytes <= kMaxStagedBytes && capacity)   // lists kept with a batch are made once
        if (mgk_status st = staging_slot(ctx, bytes, !fixed, stream, &slot)) return st;
    std::vector<MgkJob> pageable(slot ? 0 : plan.jobs.size());
    MgkJob* flat = slot ? static_cast<MgkJob*>(slot->p) : pageable.data();
    for (size_t k = 0; k < plan.jobs.size(); ++k) flat[at[(size_t)where[k]]++] = plan.jobs[k].job;
    MGK_HIP(ctx, hipMemcpyAsync(out.dev, flat, bytes, hipMemcpyHostToDevice, stream));
    if (slot) staging_copied(slot, stream);
    else MGK_HIP(ctx, hipStreamSynchronize(stream));  // `pageable` dies here
    return MGK_OK;
}

// Gives back what the context keeps for later calls: features and blocks of freed batches.
bool release_spare(mgk_ctx* ctx) {
    bool any = false;
    for (DevBuf* b : {&ctx->sep_packets[0], &ctx->sep_packets[1], &ctx->sep_dense[0], &ctx->sep_dense[1], &ctx->wide_outer, &ctx->wide_inner, &ctx->onchip_packets})
        if (b->p && !ctx->features_in_use) {
            (void)hipFree(b->p);   // waits for the work that reads it
            *b = DevBuf{};
            any = true;
        }
    for (void* p : ctx->old_packets) {
        (void)hipFree(p);
        any = true;
    }
    ctx->old_packets.clear();
    std::vector<FreeBlob> blobs;
    {
        std::lock_guard<std::mutex> lock(ctx->memory->m);
        blobs.swap(ctx->memory->blobs);
    }
    for (FreeBlob& f : blobs) (void)hipFree(f.p);
    return any || !blobs.empty();
}

// hipMalloc; where memory has run out, again without what the context keeps for later calls.
hipError_t device_alloc(mgk_ctx* ctx, void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();   // no error of a later launch
        if (release_spare(ctx) && (e = hipMalloc(p, bytes)) != hipSuccess) (void)hipGetLastError();
    }
    return e;
}

mgk_status ensure(mgk_ctx* ctx, DevBuf& b, size_t bytes) {
    if (bytes <= b.cap) return MGK_OK;
    if (b.p) MGK_HIP(ctx, hipFree(b.p));
    b.p = nullptr;
    b.cap = 0;
    hipError_t e = device_alloc(ctx, &b.p, bytes);
    if (e != hipSuccess)
        return fail(ctx, MGK_ENOMEM, "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    b.cap = bytes;
    return MGK_OK;
}

// Tile-pair primitive for a pair in the global-memory solver (Section IV-B,
// "hybrid dense-sparse"): the dense primitive evaluates all 4096 products of a
// tile pair, the sparse one only nnz * nnz' of them but pays gathers and row
// sums; the dense one wins when both graphs' tiles are well filled.
constexpr int kDenseMinNnzPerTile = 53;   // measured crossover on 256-vertex graphs: density 0.82

bool use_dense_tiles(const mgk_ctx* ctx, const MgkGraphDesc& a, const MgkGraphDesc& b) {
    if (ctx->edge_kernel == MGK_EK_KRON_SE || ctx->edge_kernel == MGK_EK_RCONV_SE) return false;
    if (ctx->tile_path == MGK_TILE_DENSE) return true;
    if (ctx->tile_path == MGK_TILE_SPARSE || ctx->tile_path == MGK_TILE_SPARSE_GATHER) return false;
    return a.n_tiles > 0 && b.n_tiles > 0 &&
           (int64_t)a.nnz >= (int64_t)kDenseMinNnzPerTile * a.n_tiles &&
           (int64_t)b.nnz >= (int64_t)kDenseMinNnzPerTile * b.n_tiles;
}

// Numbers of sep_basis that do not depend on the kernel.
struct SepTables {
    static constexpr int N = 48, H = N / 2, D = 2 * MGK_SEP_MAX_TERMS, E = 33;
    double node[H];       // Chebyshev nodes in (0, 1); the other half are their negatives
    double cosm[H][D];    // T_m(node) times the weight of the transform
    double mono[D][D];    // monomial coefficients of T_m
    double grid[E];
    SepTables() : mono{} {
        const double pi = 3.14159265358979323846;
        for (int i = 0; i < H; ++i) {
            node[i] = std::cos(pi * (i + 0.5) / N);
            for (int m = 0; m < D; ++m) cosm[i][m] = std::cos(pi * m * (i + 0.5) / N) * (m ? 2.0 : 1.0) / N;
        }
        mono[0][0] = mono[1][1] = 1.0;
        for (int m = 2; m < D; ++m)
            for (int j = 0; j <= m; ++j) mono[m][j] = (j ? 2.0 * mono[m - 1][j - 1] : 0.0) - mono[m - 2][j];
        for (int e = 0; e < E; ++e) grid[e] = std::cos(pi * e / (E - 1));
    }
};

// Separable form of the square-exponential kernel for labels within R of `center`, t = (R / l)^2; rank 0
// where it has none of at most MGK_SEP_MAX_RANK terms.  Functions are even or odd, so half of every
// grid does.  It is formed on the calling thread before the first launch: 31 us at rank 5, 45 at 12; with
// whole grids, tables made each time and the error taken anew for every rank it was 122 and 213.
MgkSepBasis sep_basis_se(double center, double R, double t) {
    static const SepTables T;
    constexpr int H = T.H, D = T.D, E = T.E, MaxR = MGK_SEP_MAX_RANK;
    MgkSepBasis S{};
    S.center = center;
    S.inv_r = R > 0.0 ? 1.0 / R : 0.0;
    // |exp(t s s') - its Chebyshev sum of rank r| falls like 4 (t / 4)^r / r!: hopeless beyond this
    if (!(t <= 8.0)) return S;
    // Chebyshev coefficients of exp(t s s') from its values on a grid of nodes, both variables
    double half[H][D] = {}, C[D][D] = {};
    for (int i = 0; i < H; ++i)
        for (int j = 0; j < H; ++j) {
            const double u = std::exp(t * T.node[i] * T.node[j]), v = std::exp(-t * T.node[i] * T.node[j]);
            const double sum = u + v, dif = u - v;
            for (int m = 0; m < D; m += 2) {
                half[i][m] += sum * T.cosm[j][m];
                half[i][m + 1] += dif * T.cosm[j][m + 1];
            }
        }
    for (int i = 0; i < H; ++i)   // the function is even in (s, s') together
        for (int m = 0; m < D; ++m)
            for (int n = m & 1; n <= m; n += 2) C[m][n] += 2.0 * half[i][m] * T.cosm[i][n];
    for (int m = 0; m < D; ++m)
        for (int n = m & 1; n < m; n += 2) C[n][m] = C[m][n];
    double gauss[H], left[E][E];   // what the columns so far leave of the kernel
    for (int i = 0; i < H; ++i) gauss[i] = std::exp(-0.5 * t * T.node[i] * T.node[i]);
    for (int e = 0; e < E; ++e)
        for (int f = 0; f <= e; ++f) left[e][f] = std::exp(-0.5 * t * (T.grid[e] - T.grid[f]) * (T.grid[e] - T.grid[f]));
    for (int k = 0; k < MaxR; ++k) {
        // column k of the Cholesky factor, as a function times the Gaussian, as a polynomial
        const int odd = k & 1;
        const double d = C[k][k];
        if (!(d > 0.0)) return S;   // no further degree can be resolved in double
        double col[D], cheb[D] = {}, poly[D] = {};
        for (int m = 0; m < D; ++m) col[m] = C[m][k] / std::sqrt(d);
        for (int m = odd; m < D; m += 2)
            for (int n = odd; n < D; n += 2) C[m][n] -= col[m] * col[n];
        for (int i = 0; i < H; ++i) {
            double v = 0.0;
            for (int m = odd; m < D; m += 2) v += col[m] * T.cosm[i][m] * (m ? 0.5 * T.N : T.N);
            v *= 2.0 * gauss[i];
            for (int m = odd; m < D; m += 2) cheb[m] += v * T.cosm[i][m];
        }
        int last = D - 1;   // what is left above is rounding noise, which the monomials would amplify
        while (last > 0 && std::fabs(cheb[last]) < 1e-12) --last;
        for (int m = odd; m <= last; m += 2)
            for (int j = odd; j <= m; j += 2) poly[j] += cheb[m] * T.mono[m][j];
        for (int m = 0; m < MGK_SEP_MAX_TERMS; ++m) S.coef[m * MaxR + k] = poly[2 * m + odd];
        double feat[E], err = 0.0;
        for (int e = 0; e < E; ++e) {
            double v = 0.0;
            for (int m = MGK_SEP_MAX_TERMS - 1; m >= 0; --m) v = v * T.grid[e] * T.grid[e] + S.coef[m * MaxR + k];
            feat[e] = odd ? v * T.grid[e] : v;
        }
        for (int e = 0; e < E; ++e)
            for (int f = 0; f <= e; ++f) {
                left[e][f] -= feat[e] * feat[f];
                err = std::max(err, std::fabs(left[e][f]));
            }
        if (err > MGK_SEP_TOLERANCE) continue;
        S.rank = k + 1;
        S.terms = 1;
        for (int m = 0; m < MGK_SEP_MAX_TERMS; ++m)
            for (int q = 0; q <= k; ++q)
                if (S.coef[m * MaxR + q] != 0.0) S.terms = m + 1;
        return S;
    }
    return S;
}

// The same in powers of the second label (see MgkWideBasis).  kappa_e / g at a Chebyshev node s has in s' the Chebyshev
// coefficients c_n(s); those below the rank, as powers of s', are the functions, each even or odd.  The exponent of g is
// free: a little below t / 2 balances what the sum leaves at the middle and at the ends of the range, one to three terms fewer than t / 2
// itself (t = 0.5, 1.3, 2.3, 5: 6, 9, 10, 13 terms where that needs 7, 10, 12, 16).  35 to 60 us, when pairs first may take it.
MgkWideBasis wide_basis_se(double center, double R, double t) {
    static const SepTables T;
    constexpr int H = T.H, D = T.D, E = T.E, MaxR = MGK_SEP_MAX_RANK;
    MgkWideBasis S{};
    S.outer.center = center;
    S.outer.inv_r = R > 0.0 ? 1.0 / R : 0.0;
    S.half_t = 0.5 * t * (t <= 1.0 ? 0.95 : t <= 2.5 ? 0.9 : 0.85);
    if (!(t <= 8.0)) return S;
    double c[H][D] = {};
    for (int i = 0; i < H; ++i)
        for (int j = 0; j < H; ++j) {
            const double s = T.node[i], r = T.node[j], weight = S.half_t * r * r;
            const double u = std::exp(weight - 0.5 * t * (s - r) * (s - r)), v = std::exp(weight - 0.5 * t * (s + r) * (s + r));
            for (int m = 0; m < D; m += 2) {
                c[i][m] += (u + v) * T.cosm[j][m];
                c[i][m + 1] += (u - v) * T.cosm[j][m + 1];
            }
        }
    double inner[E][MaxR];   // g(s') s'^l
    for (int e = 0; e < E; ++e) {
        inner[e][0] = std::exp(-S.half_t * T.grid[e] * T.grid[e]);
        for (int l = 1; l < MaxR; ++l) inner[e][l] = inner[e][l - 1] * T.grid[e];
    }
    int first = 1;   // exp(t s s') has c_r of about 2 (t / 2)^r / r!
    for (double left = t; first < MaxR && left > (t <= 2.0 ? 32.0 : t <= 4.0 ? 1000.0 : 4000.0) * MGK_SEP_TOLERANCE; left *= 0.5 * t / ++first) {}
    for (int rank = first; rank <= MaxR; ++rank) {
        std::fill(std::begin(S.outer.coef), std::end(S.outer.coef), 0.0);
        double feat[E][MaxR];
        for (int l = 0; l < rank; ++l) {
            const int odd = l & 1;
            double cheb[D] = {}, poly[D] = {};
            for (int i = 0; i < H; ++i) {
                double v = 0.0;
                for (int n = l; n < rank; n += 2) v += c[i][n] * T.mono[n][l];
                for (int m = odd; m < D; m += 2) cheb[m] += 2.0 * v * T.cosm[i][m];
            }
            int last = D - 1;   // what is left above is rounding noise, which the monomials would amplify
            while (last > 0 && std::fabs(cheb[last]) < 1e-12) --last;
            for (int m = odd; m <= last; m += 2)
                for (int j = odd; j <= m; j += 2) poly[j] += cheb[m] * T.mono[m][j];
            for (int m = 0; m < MGK_SEP_MAX_TERMS; ++m) S.outer.coef[m * MaxR + l] = poly[2 * m + odd];
            for (int e = 0; e < E; ++e) {
                double v = 0.0;
                for (int m = MGK_SEP_MAX_TERMS - 1; m >= 0; --m) v = v * T.grid[e] * T.grid[e] + S.outer.coef[m * MaxR + l];
                feat[e][l] = odd ? v * T.grid[e] : v;
            }
        }
        double err = 0.0;
        for (int e = 0; e < E; ++e)
            for (int f = 0; f < E; ++f) {
                double v = std::exp(-0.5 * t * (T.grid[e] - T.grid[f]) * (T.grid[e] - T.grid[f]));
                for (int l = 0; l < rank; ++l) v -= feat[e][l] * inner[f][l];
                err = std::max(err, std::fabs(v));
            }
        if (err > MGK_SEP_TOLERANCE) continue;
        S.outer.rank = rank;
        S.outer.terms = 1;
        for (int m = 0; m < MGK_SEP_MAX_TERMS; ++m)
            for (int l = 0; l < rank; ++l)
                if (S.outer.coef[m * MaxR + l] != 0.0) S.outer.terms = m + 1;
        return S;
    }
    return S;
}

// Separable form of the edge kernel on the label range [lo, hi] (see MgkSepBasis).  rank 0: the kernel
// has none (short length scale against the range, or a kernel that is not smooth).  The last few are kept
// with the context: batches compared in turn have ranges of their own.
const MgkSepBasis* kept_basis(const mgk_ctx* ctx, float lo, float hi) {
    const float param = ctx->edge_kernel == MGK_EK_SE ? ctx->length_scale : ctx->ke_const;
    for (const KeptBasis& b : ctx->bases)
        if (b.kernel == ctx->edge_kernel && b.param == param && b.lo == lo && b.hi == hi) return &b.basis;
    return nullptr;
}
const MgkSepBasis* make_basis(mgk_ctx* ctx, float lo, float hi) {
    const float param = ctx->edge_kernel == MGK_EK_SE ? ctx->length_scale : ctx->ke_const;
    KeptBasis& b = ctx->bases[ctx->next_basis];
    ctx->next_basis = (ctx->next_basis + 1) % (int)(sizeof(ctx->bases) / sizeof(ctx->bases[0]));
    b = KeptBasis{};
    b.kernel = ctx->edge_kernel;
    b.param = param;
    b.lo = lo;
    b.hi = hi;
    if (ctx->edge_kernel == MGK_EK_CONST) {
        b.basis.rank = b.basis.terms = 1;
        b.basis.coef[0] = std::sqrt((double)ctx->ke_const);
    } else if (ctx->edge_kernel == MGK_EK_SE) {
        const double center = 0.5 * ((double)lo + (double)hi), R = std::max((double)hi - center, center - (double)lo);
        const double l = (double)ctx->length_scale;
        b.basis = sep_basis_se(center, R, R * R / (l * l));
    }
    return &b.basis;
}

// How the sparse separable product of a pair with n2 columns divides its rank: the fewest
// features executed, then the fewest passes; rk = 0 when no column count fits in LDS.
MgkSepLayout sep_layout(int rank, int n2) {
    MgkSepLayout L{};
    for (int rk : {7, 6, 5, 4, 1}) {
        if (mgk_sep_lds_bytes(rk, n2) > MGK_LDS_LIMIT_BYTES || (rk == 1) != (rank == 1)) continue;
        const int passes = (rank + rk - 1) / rk;
        if (L.rk == 0 || passes * rk < L.passes * L.rk || (passes * rk == L.passes * L.rk && passes < L.passes))
            L = MgkSepLayout{rk, passes, mgk_sep_per_packet(rk), MGK_SEP_SLAB(rk) * 4, 0};
    }
    return L;
}

// The same for graphs of many vertices: one pass with 8 rows where two workgroups share a compute unit with it (contact graphs of 256 and 300
// vertices, rank 9, 64 pairs: one pass 993 and 1584 us, two 1080 and 1429), else the fewest features executed, then the
// fewest passes, with 8 rows where two workgroups share a compute unit; rows = 0 where no division fits.
MgkWideLayout wide_layout(int rank, int n2) {
    MgkWideLayout best{};
    static const struct { int hi, lo; } kForms[] = {{4, 4}, {5, 5}, {6, 6}, {8, 8}, {9, 9}, {10, 10}, {4, 5}};   // single passes by size
    for (const auto& f : kForms) {
        MgkWideLayout L{8, f.hi, f.lo, 1 + std::max(0, (rank - f.hi + f.lo - 1) / f.lo)};
        if (rank <= 0 || (f.hi > 6 && L.passes > 1) || (f.hi != f.lo && L.passes == 1)) continue;
        if (!mgk_wide_two(L, n2)) {
            L.rows = 4;
            if (f.hi > 6 || L.rows * n2 > MGK_WIDE_MAX_ELEMENTS || mgk_wide_lds_bytes(L, n2) > MGK_LDS_LIMIT_BYTES) continue;
        }
        if (L.passes == 1 && L.rows == 8) return L;
        const int all = f.hi + (L.passes - 1) * f.lo, least = best.hi + (best.passes - 1) * best.lo;
        if (best.rows == 0 || all < least || (all == least && L.passes < best.passes)) best = L;
    }
    return best;
}

// Product of the global-memory solver for one pair.
enum { kPathSparse = 0, kPathDenseTiles = 1, kPathSep = 2, kPathSepDense = 3, kPathWide = 4, kPathSepParts = 5, kPaths = 6 };
bool is_sep_dense(int path) { return path == kPathSepDense || path == kPathSepParts; }   // the same features, two kernels
bool is_sep(int path) { return path == kPathSep || path == kPathWide || is_sep_dense(path); }

// Estimated clocks of one compute unit for one product of a pair on every path, infinite where it cannot run.
// Throughput of a full chip, fitted to iterations of 64 pairs of random graphs (n = 128 to 256, densities 0.01
// to 1, ranks 1 to 8) and of contact graphs: the row-staged product evaluates 7 entries per clk, stages the
// rows of p and pays 6 clk per element in dependent loads, and takes a third longer for entries of rows of up
// to 14 nonzeros (5 to 64 pairs of n = 256 to 480), less for longer ones; the sparse separable product does 20
// multiply-adds per clk and writes and reads T; the dense one does 42 per clk and has work for all four of its
// wavefronts from 256 columns on.  A few pairs leave the chip idle: then the time of a workgroup counts, as
// many times as workgroups follow each other on a compute unit.  It is a row of the outer graph (row-staged:
// 5000 clk and 1.6 times its share of the work, behind the rest), 16 rows (sparse: 45 clk per column and pass
// and 1.05 times its share), 32 rows (dense: 60 multiply-adds per clk).  The direct products expand the lists
// of both batches, whichever graphs the pairs have: 0.4 ns per nonzero or 1.2 per octile, over about 12
// iterations.
// The form for graphs of many vertices does 33 multiply-adds per clk, 5 clk per element go to the vectors and 6000 to a
// workgroup's trips to memory and barriers a pass, more than half of a small one's time; a workgroup alone takes 8 clk per element of T and 1000 per nonzero of a row.
// Us per call, row-staged or sparse / that, contact graphs of rank 9, 1, 4, 16 and 64 pairs: n = 132 225 / 244, 240 / 256, 328 / 313, 571 / 590;
// 256 264 / 274, 371 / 280, 416 / 391, 1121 / 956; 300 282 / 314, 413 / 341, 564 / 580, 1367 / 1453; 480 388 / 372, 575 / 425, 986 / 982, 2928 / 2924;
// 600 522 / 395, 1230 / 610, 3796 / 1379; 1000 1107 / 537, 3086 / 1081, 9940 / 3100; 2048 3347 / 1303, 11149 / 3821, 40577 / 13426.  Random graphs of
// n = 256, rank 6, 1, 8 and 64 pairs: density 0.01 307 / 304, 514 / 465, 1360 / 1225; 0.12 326 / 253, 338 / 290, 1004 / 859.
// Measured, us per call, row-staged / sparse / dense, rank 5, one batch of 128 graphs: 1 pair of n = 256
// density 0.01 420 / 478 / 3432, 0.03 388 / 296 / 1686, 0.2 660 / 375 / 1011, 1 3467 / 872 / 893; 64 pairs
// 2090 / 1842 / 7344, 1899 / 1094 / 3630, 13540 / 1311 / 2215, 189182 / 2944 / 1677.  8 graphs of n = 600
// density 0.1, 1, 2, 4, 16 pairs, row-staged / dense: 2515 / 5206, 4112 / 5264, 7394 / 5294, 26957 / 10472; n
// = 1000 density 0.05: 4592 / 11290, 8246 / 11366, 15217 / 11569, 56425 / 25971.  Geometric graphs of degree
// 12, row-staged / sparse, 2, 4, 8, 16 pairs: n = 140 rank 9 220 / 305, 233 / 311, 281 / 319, 352 / 327; n =
// 300 rank 5 358 / 439, 454 / 454, 622 / 486, 934 / 686, rank 13 307 / 569, 381 / 583, 515 / 616, 741 / 816; n
// = 480 rank 11 516 / 704, 773 / 744, 1207 / 913, 2091 / 1403.  Constant kernel, 37 pairs of n = 146 to 162,
// density 0.011: 711 / 798, whence its 10 clk per element of the sparse form where others have 8.
struct LargeCost {
    double clk[kPaths] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    int best = kPathSparse;
    struct { double share, workgroup; } fp32{}, parts{};   // of the dense forms: all compute units busy; one workgroup
};
// Bytes the features of a graph take at most, whatever the layout.
constexpr int64_t kMaxFeatureBytes = (int64_t)8 << 30;   // of the pairs solved together
constexpr int64_t kWideMaxDegree = 32;   // mean; beyond, stage 1 was not measured, and from 50 on the dense form is near
// An absent nonzero may point at columns 0 to 3.  Below 24 columns the row-staged product takes the less time: outer graphs of 4000 vertices, degree 8, 1,
// 8 and 64 pairs, row-staged / this: n = 20 403 / 285, 447 / 704, 1633 / 4063 us; n = 10 349 / 269, 418 / 745, 906 / 3650.
constexpr int kWideMinColumns = 24;
int64_t wide_feature_bytes(const mgk_batch* b, int32_t g) {   // as outer and as inner graph
    constexpr int kPasses = MGK_SEP_MAX_RANK / 4;
    return (int64_t)kPasses * 32 * b->graphs[(size_t)g].nnz + 4 * mgk_wide_inner_words(b->graphs[(size_t)g], kPasses);
}
int64_t feature_bytes(const mgk_batch* b, int32_t g, int rank, bool dense) {
    const int64_t np = (b->graphs[(size_t)g].n + 63) & ~63;
    const auto& off = b->packet_off[rank == 1 ? 1 : 0];
    return dense ? 4 * np * np * rank : 256 * (int64_t)((rank + 3) / 4) * (off[(size_t)g + 1] - off[(size_t)g]);
}

// The form for graphs of many vertices, made once for every kept one; without `make` what there is, or null.
const MgkWideBasis* wide_basis(mgk_ctx* ctx, const MgkSepBasis* kept, bool make) {
    for (KeptBasis& b : ctx->bases)
        if (&b.basis == kept) {
            if (!b.has_wide && !make) return nullptr;
            if (!b.has_wide) {
                const double R = kept->inv_r > 0.0 ? 1.0 / kept->inv_r : 0.0, l = (double)ctx->length_scale;
                b.wide = wide_basis_se(kept->center, R, R * R / (l * l));
                b.has_wide = true;
            }
            return &b.wide;
        }
    return nullptr;
}

// rank 0: no separable form.  L, W: the division of the pairs that are solved together.  n_pairs: pairs of the call that may run beside this one.  n_tiles: octiles of
// both batches, or a third of the nonzeros where that is less.  Forming the features is left out: only the graphs of the pairs get them, which takes 1 % of
// what the products of a pair take.
LargeCost large_cost(const mgk_ctx* ctx, int rank, const MgkSepLayout& L, const MgkWideLayout& W, const mgk_batch* A, int32_t ga, const mgk_batch* B, int32_t gb,
                     int64_t n_pairs, int64_t n_tiles) {
    constexpr double kUnits = 256;   // compute units
    const MgkGraphDesc &o = A->graphs[(size_t)ga], &i = B->graphs[(size_t)gb];
    auto fits = [&](bool dense) { return feature_bytes(A, ga, rank, dense) + feature_bytes(B, gb, rank, dense) <= kMaxFeatureBytes; };
    LargeCost C;
    C.best = use_dense_tiles(ctx, o, i) ? kPathDenseTiles : kPathSparse;
    if (ctx->tile_path != MGK_TILE_AUTO || rank == 0) {
        C.clk[C.best] = 0.0;   // no choice
        return C;
    }
    // Pairs small enough for the on-chip solver come here where the caller has lowered its limit; their
    // workgroups take less time than the launches of an iteration: throughput alone decides.
    const double pairs = o.n * (int64_t)i.n <= MGK_SMALL_MAX_N && ctx->onchip_limit < MGK_SMALL_MAX_N ? INFINITY : (double)n_pairs;
    const double N = (double)o.n * i.n, one_sided = (double)o.nnz * i.n + (double)o.n * i.nnz;
    const double entries = (double)o.nnz * i.nnz * (1.0 / 7.0) + 0.5 * (double)o.nnz * i.n;
    const double short_rows = std::isinf(pairs) ? 0.0 : std::min(0.35, 5.0 * o.n / std::max(o.nnz, 1));
    C.clk[C.best] = (1.0 + short_rows) * entries + 6.0 * N + 61.0 * (double)n_tiles / pairs + kUnits / pairs * (5000.0 + 1.6 * entries / o.n);
    // clocks of a pair's share of all compute units while the workgroups of all pairs run
    auto workgroups = [&](double blocks, int64_t lds_bytes, int64_t most, double clk) {
        const double side_by_side = kUnits * (double)std::min<int64_t>(most, MGK_LDS_LIMIT_BYTES / std::max<int64_t>(lds_bytes, 1));
        const double rounds = blocks * pairs / side_by_side;   // the last blocks of a pair have its rows of lowest degree
        return std::isinf(pairs) ? 0.0 : kUnits / pairs * std::max(1.0, 0.5 * (rounds + std::ceil(rounds))) * clk;
    };
    const double op = (o.n + 31) & ~31, ip = (i.n + 255) & ~255, np = (i.n + 63) & ~63;
    const double sparse = (double)L.rk * L.passes * one_sided * (1.0 / 20.0), dense = rank * op * ip * ((double)o.n + i.n);
    const double elements = (ctx->edge_kernel == MGK_EK_CONST ? 10.0 : 8.0) * N;   // rank 1 stays a bound of higher ones
    const bool may_sparse = L.rk > 0 && fits(false), may_dense = ip <= MGK_SEP_DENSE_MAX_N && fits(true);
    // With operands in 16-bit parts (64 columns to a workgroup, one to a compute unit) 145 multiply-adds per clk.  Us per call, sparse / fp32 / parts: 64 pairs
    // of n = 256, density 0.2 1179 / 2215 / 985, 1 2944 / 1668 / 819; n = 150, density 0.3, 0.5, 1 611 / 1041 / 592, 849 / 1051 / 609, 982 / 886 /
    // 513; n = 130 548 / 1094 / 624, 668 / 944 / 555, 796 / 801 / 482; 8 pairs of n = 150 266 / 661 / 462, 347 / 666 / 461, 390 / 554 / 385.
    // Never slower than the fp32 kernel, down to n = 40.
    const bool in_parts = may_dense && mgk_sep_in_parts(o.n, i.n);
    if (may_sparse) {
        const double blocks = (o.n + MGK_SEP_ROWS - 1) / MGK_SEP_ROWS;
        C.clk[kPathSep] = std::max(sparse + elements + (std::isinf(pairs) ? 0.0 : 6000.0 * blocks * (L.passes - 1)),
                                   workgroups(blocks, mgk_sep_lds_bytes(L.rk, i.n), 2048 / MGK_SEP_THREADS, 45.0 * i.n * L.passes + 1.05 * sparse / blocks));
    }
    if (may_dense) {
        const double blocks = op / MGK_SEP_DENSE_ROWS;
        C.fp32 = {dense * (1.0 / 42.0), dense / 60.0 / blocks};
        C.clk[kPathSepDense] = std::max(C.fp32.share, workgroups(blocks, (int64_t)(4 * MGK_SEP_DENSE_ROWS * (np + 1)), 2, C.fp32.workgroup));
    }
    if (in_parts) {
        C.parts = {rank * op * np * ((double)o.n + i.n) * (1.0 / 145.0) + elements, rank * (15700.0 + 63.0 * ((double)o.n + i.n))};
        // of small pairs (n = 40 to 100 at density 0.5) the sparse form takes less time by throughput too: the rate of the fp32 kernel
        C.clk[kPathSepParts] = std::isinf(pairs) ? C.clk[kPathSepDense] : std::max(C.parts.share, workgroups(np / 64, MGK_SEP_PARTS_LDS, 1, C.parts.workgroup));
    }
    if (W.rows > 0 && !std::isinf(pairs) && i.n >= kWideMinColumns && o.nnz <= kWideMaxDegree * (int64_t)o.n && i.nnz <= kWideMaxDegree * (int64_t)i.n) {
        const double blocks = (o.n + W.rows - 1) / W.rows, products = (W.hi + (W.passes - 1) * W.lo) * one_sided * (1.0 / 33.0);
        C.clk[kPathWide] = std::max(products + 5.0 * N + 6000.0 * blocks * W.passes,
                                    workgroups(blocks, mgk_wide_lds_bytes(W, i.n), 2, 8.0 * W.rows * i.n + products / blocks + 1000.0 * W.passes * o.nnz / o.n));
        if (C.clk[kPathWide] < C.clk[C.best]) C.best = kPathWide;
    }
    if (!may_sparse && !may_dense) return C;
    // of the two forms the one with the higher throughput, or, with a few pairs in 16-bit parts, the sooner end
    const bool denser = in_parts && !std::isinf(pairs) ? C.clk[kPathSepParts] < C.clk[kPathSep] : C.fp32.share < sparse + elements;
    const int form = may_dense && (!may_sparse || denser) ? in_parts ? kPathSepParts : kPathSepDense : kPathSep;
    if (C.clk[form] < C.clk[C.best]) C.best = form;
    return C;
}

// Every path in use is a sequence of launches of its own with a wait at its end: 300 us for a path of
// half of 64 pairs of 256-vertex graphs at density 0.01, whose products take the same time either way,
// or 1e7 clk per iteration.  A path that saves less than that goes to the next best one in use.
void merge_paths(std::vector<LargeCost>& costs) {
    constexpr double kPathClk = 1e7;
    while (true) {
        double move[kPaths][kPaths] = {};
        bool used[kPaths] = {};
        for (const LargeCost& C : costs) {
            used[C.best] = true;
            for (int to = 0; to < kPaths; ++to)
                if (to != C.best) move[C.best][to] += C.clk[to] - C.clk[C.best];
        }
        int from = -1, into = -1;
        for (int a = 0; a < kPaths; ++a)
            for (int b = 0; b < kPaths; ++b)
                if (a != b && used[a] && used[b] && move[a][b] < kPathClk && (from < 0 || move[a][b] < move[from][into])) {
                    from = a;
                    into = b;
                }
        if (from < 0) return;
        for (LargeCost& C : costs)
            if (C.best == from) C.best = into;
    }
}

// The two dense forms in one call: pairs on parts run beside the others in the fp32 kernel unless launches of their own take less
// time.  A launch takes what its longest workgroup takes, or its work on all compute units, or rather more than either where they are alike.  Us per
// call, joined / apart, complete graphs, one pair of n = 290 and 8, 20, 60, 128 and 256 of n = 250: 2160 / 2620, 2318 / 2723, 3098 / 2967, 5444 /
// 3991, 9570 / 5891; n = 500 and 250: 3312 / 3349, 3700 / 3435, 4256 / 3679, 5942 / 4743, 10101 / 6618; n = 270 and 140, 60, 128 and 256: 2175 /
// 2278, 2584 / 2711, 3548 / 3432.
void join_dense(std::vector<LargeCost>& costs) {
    constexpr double kUnits = 256, kPathClk = 1e7 / kUnits;
    double fp32 = 0.0, also = 0.0, parts = 0.0, longest = 0.0, longest_parts = 0.0;
    for (const LargeCost& C : costs) {
        if (C.best == kPathSepDense) {
            fp32 += C.fp32.share / kUnits;
            longest = std::max(longest, C.fp32.workgroup);
        } else if (C.best == kPathSepParts) {
            also += C.fp32.share / kUnits;
            parts += C.parts.share / kUnits;
            longest_parts = std::max(longest_parts, C.parts.workgroup);
        }
    }
    if (fp32 == 0.0 || parts == 0.0) return;
    if (std::hypot(fp32 + also, longest) < std::hypot(fp32, longest) + 0.7 * std::hypot(parts, longest_parts) + kPathClk)
        for (LargeCost& C : costs)
            if (C.best == kPathSepParts) C.best = kPathSepDense;
}

// Plan of one pair for the global-memory solver (any size).
MgkLargePair plan_large(const MgkGraphDesc& a, const MgkGraphDesc& b, int32_t ia, int32_t ib, bool* swap,
                        int max_iter_param) {
    auto passes = [](const MgkGraphDesc& o, const MgkGraphDesc& i) {
        return (int64_t)o.nnz * (i.lane_len / 64) + 2 * (int64_t)o.n * (i.lane_len / 64);
    };
    const bool keep_atomic = b.max_deg > MGK_LANE_GROUP, swp_atomic = a.max_deg > MGK_LANE_GROUP;
    *swap = keep_atomic != swp_atomic ? keep_atomic : passes(b, a) < passes(a, b);
    const MgkGraphDesc& o = *swap ? b : a;
    const MgkGraphDesc& i = *swap ? a : b;
    MgkLargePair P{};
    P.g1 = *swap ? ib : ia;
    P.g2 = *swap ? ia : ib;
    P.n1 = o.n;
    P.n2 = i.n;
    const int64_t N = (int64_t)o.n * i.n;
    P.npad = (int32_t)((N + 63) & ~(int64_t)63);
    P.max_iter = max_iter_param > 0 ? max_iter_param : (int32_t)std::min<int64_t>(2 * N, 1000);
    P.nsteps = i.max_deg <= 1 ? 0 : i.max_deg <= 2 ? 1 : i.max_deg <= 4 ? 2 : i.max_deg <= 8 ? 3 : 4;
    P.atomic_rows = i.max_deg > MGK_LANE_GROUP ? 1 : 0;
    return P;
}

// A slot of pinned memory, of at least `bytes`, for copies on `stream`: the next one, grown where it is too
// small; while its last call is under way another one that is large enough and idle.  Without may_allocate one
// that is large enough, waited for if need be, or none (*out is null).
mgk_status staging_slot(mgk_ctx* ctx, size_t bytes, bool may_allocate, hipStream_t stream, Staging::Slot** out) {
    Staging& S = ctx->staging;
    constexpr int kSlots = sizeof(S.slot) / sizeof(S.slot[0]);
    *out = nullptr;
    if (!S.block && may_allocate) {
        MGK_HIP(ctx, hipHostMalloc(&S.block, kSlots * kSlotBytes, hipHostMallocDefault));
        for (Staging::Slot& s : S.slot) {
            s.p = (char*)S.block + (size_t)(&s - S.slot) * kSlotBytes;
            s.cap = kSlotBytes;
        }
    }
    int pick = S.next, large = -1;
    for (int k = 0; k < kSlots; ++k) {
        const int at = (S.next + k) % kSlots;
        Staging::Slot& s = S.slot[at];
        const bool fits = s.cap >= bytes;
        if (!fits && !(may_allocate && k == 0)) continue;
        if (fits && large < 0) large = at;
        if (!s.open && (!s.end || s.end->over())) { pick = at; large = -1; break; }
    }
    if (!may_allocate && large >= 0) pick = large;   // all that are large enough are in use
    Staging::Slot& s = S.slot[pick];
    if (bytes > s.cap && !may_allocate) return MGK_OK;
    S.next = (pick + 1) % kSlots;
    if (s.open) {   // by a call that failed, or by this one, which has used all slots
        if (s.stream == stream) MGK_HIP(ctx, hipStreamSynchronize(stream));
        MGK_HIP(ctx, hipDeviceSynchronize());
        s.open = false;
    } else if (s.end && !s.end->over()) {
        MGK_HIP(ctx, hipEventSynchronize(s.end->event));
    }
    s.end.reset();
    if (bytes > s.cap) {
        if (s.own) MGK_HIP(ctx, hipHostFree(s.p));
        s.p = nullptr;
        s.cap = 0;
        s.own = true;
        const size_t cap = std::max(bytes + bytes / 4, kSlotBytes);
        MGK_HIP(ctx, hipHostMalloc(&s.p, cap, hipHostMallocDefault));
        s.cap = cap;
    }
    *out = &s;
    return MGK_OK;
}

void staging_copied(Staging::Slot* slot, hipStream_t stream) {   // a copy out of it is on the stream
    slot->open = true;
    slot->stream = stream;
}

// Device memory for a batch: a freed batch's block that nothing reads any more, or a new one.
mgk_status take_blob(mgk_ctx* ctx, size_t bytes, void** p, size_t* cap) {
    std::vector<std::shared_ptr<CallEnd>> ended;
    std::unique_lock<std::mutex> lock(ctx->memory->m);
    std::vector<FreeBlob>& blobs = ctx->memory->blobs;
    for (size_t k = 0; k < blobs.size(); ++k) {
        FreeBlob& f = blobs[k];
        if (f.cap < bytes || f.cap > 4 * bytes + 65536) continue;
        if (!std::all_of(f.reads.begin(), f.reads.end(), [](const std::shared_ptr<CallEnd>& r) { return r->over(); })) continue;
        *p = f.p;
        *cap = f.cap;
        ended.swap(f.reads);   // given back when the lock is
        blobs.erase(blobs.begin() + (std::ptrdiff_t)k);
        return MGK_OK;
    }
    lock.unlock();
    *cap = bytes <= kMaxBlobBytes ? (bytes + bytes / 4 + 65535) & ~(size_t)65535 : bytes;   // room for others, later
    if (*cap > bytes && device_alloc(ctx, p, *cap) == hipSuccess) return MGK_OK;
    *cap = bytes;
    MGK_HIP(ctx, device_alloc(ctx, p, bytes));
    return MGK_OK;
}

// Keeps the block of a batch that is being freed, unless there are enough or it is large.
bool keep_blob(mgk_batch* b) {
    std::lock_guard<std::mutex> lock(b->memory->m);
    std::vector<FreeBlob>& blobs = b->memory->blobs;
    if (!b->memory->open || blobs.size() >= kMaxBlobs || b->blob_cap > kMaxBlobBytes || b->untracked) return false;
    blobs.push_back(FreeBlob{b->blob, b->blob_cap, b->reads});
    return true;
}

// Run Alg. 1 with global-memory vectors for a list of pairs (outer graphs from
// A, inner from B).  Synchronises the stream: the host watches the number of
// pairs still iterating.
mgk_status solve_large(mgk_ctx* ctx, const mgk_batch* A, const mgk_batch* Bb, int ia, int ib,
                       std::vector<MgkLargePair> pairs, bool dense, const MgkOutputs& out,
                       hipStream_t stream, const MgkParams& prm, bool weighted) {
    const int n_pairs = (int)pairs.size();
    if (n_pairs == 0) return MGK_OK;
    int64_t total = 0;
    int max_npad = 0, max_iter = 0, xmv_blocks = 1;
    int max_n1 = 1, max_n2 = 1, max_deg1 = 1, max_chunks = 1, min_chunks = 1 << 30;
    constexpr int CPB = MGK_LARGE_WAVES * MGK_LARGE_CHUNKS_PER_WAVE;
    for (MgkLargePair& P : pairs) {
        max_n1 = std::max(max_n1, P.n1);
        max_n2 = std::max(max_n2, P.n2);
        max_deg1 = std::max(max_deg1, A->graphs[P.g1].max_deg);
        max_chunks = std::max(max_chunks, Bb->graphs[P.g2].lane_len / 64);
        min_chunks = std::min(min_chunks, Bb->graphs[P.g2].lane_len / 64);
        P.vec = total;
        total += 5 * (int64_t)P.npad;
        max_npad = std::max(max_npad, P.npad);
        max_iter = std::max(max_iter, P.max_iter);
        const int chunks = Bb->graphs[P.g2].lane_len / 64;
        const int rb = (P.n1 + MGK_LARGE_ROWS_PER_BLOCK - 1) / MGK_LARGE_ROWS_PER_BLOCK;
        if (dense)
            xmv_blocks = std::max(xmv_blocks, (A->graphs[P.g1].n_tile_rows * Bb->graphs[P.g2].n_tile_rows + 3) / 4);
        else
            xmv_blocks = std::max(xmv_blocks, rb * ((chunks + CPB - 1) / CPB));
    }
    // Sparse product: stage the rows of p a row of the outer graph needs in LDS when a row
    // fits (one workgroup per outer row), else gather p from global memory.
    // Up to 60 KB of LDS per workgroup of at most 8 wavefronts (two or more workgroups per
    // CU); when the rows of p are so long that the neighbours of one outer row need more,
    // one workgroup of 16 wavefronts per CU with up to 120 KB.
    constexpr int kRowsLdsSmall = 60 * 1024, kRowsLdsLarge = 120 * 1024;
    int rows_threads = 0, rows_lds_bytes = 0, rows_chunks = 1;
    if (!dense && ctx->row_staging && (int64_t)max_n2 * 4 <= kRowsLdsLarge) {
        const int64_t need = (int64_t)max_deg1 * max_n2 * 4;
        const bool large = need > kRowsLdsSmall;
        const int budget = large ? kRowsLdsLarge : kRowsLdsSmall;
        const int rows = std::max(1, std::min(std::min(max_deg1, MGK_ROWS_MAX_BATCH), budget / (max_n2 * 4)));
        rows_lds_bytes = rows * max_n2 * 4;   // + the batch's outer entries and attributes, added by the launcher
        rows_threads = 64 * std::max(1, std::min(large ? 16 : 8, (max_chunks + 1) / 2));
        xmv_blocks = max_n1;
        // Chunks of the inner layout per pass of a wavefront: every outer entry read from LDS
        // then serves that many gathers.  Four need about 110 registers per lane, which only
        // the single large workgroup per CU affords; two where every wavefront still gets a
        // pass on the smallest pair.
        const int waves = rows_threads / 64;
        rows_chunks = large && min_chunks >= 4 * waves ? 4 : min_chunks >= 2 * waves ? 2 : 1;
    }
    const int vec_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(2048, ((int64_t)max_npad + 1023) / 1024));
    mgk_status st;
    if ((st = ensure(ctx, ctx->vec, (size_t)total * sizeof(float))) != MGK_OK) return st;
    if ((st = ensure(ctx, ctx->lpairs, (size_t)n_pairs * sizeof(MgkLargePair))) != MGK_OK) return st;
    if ((st = ensure(ctx, ctx->lstate, (size_t)n_pairs * sizeof(MgkPairState))) != MGK_OK) return st;
    if ((st = ensure(ctx, ctx->lactive, 64)) != MGK_OK) return st;
    if (!ctx->active_host) MGK_HIP(ctx, hipHostMalloc((void**)&ctx->active_host, 64, hipHostMallocDefault));

    // expanded entry lists of the batches involved (label scaling depends on the parameters)
    const mgk_batch* bt[2] = {A, Bb};
    const int slot[2] = {ia, ib};
    MgkExpanded ex[2] = {};
    MgkDenseTiles dt[2] = {};
    for (int k = 0; k < 2 && dense; ++k) {
        if (k == 1 && Bb == A) { dt[1] = dt[0]; break; }
        const size_t bytes = std::max<size_t>(16, (size_t)bt[k]->dev.n_tiles_total * 64 * sizeof(float));
        for (int a = 0; a < 3; ++a)
            if ((st = ensure(ctx, ctx->dense_tiles[slot[k]][a], bytes)) != MGK_OK) return st;
        float* dw = (float*)ctx->dense_tiles[slot[k]][0].p;
        float* de = (float*)ctx->dense_tiles[slot[k]][1].p;
        float* dlw = (float*)ctx->dense_tiles[slot[k]][2].p;
        hipError_t e = mgk_launch_expand_dense(bt[k]->dev, prm, dw, de, dlw, stream);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "expand launch failed: %s", hipGetErrorString(e));
        dt[k].w = dw; dt[k].e = de; dt[k].lw = dlw;
    }
    for (int k = 0; k < 2 && !dense; ++k) {
        if (k == 1 && Bb == A) { ex[1] = ex[0]; break; }
        DevBuf& bo = ctx->exp_outer[slot[k]];
        DevBuf& bi = ctx->exp_inner[slot[k]];
        if ((st = ensure(ctx, bo, std::max<size_t>(16, (size_t)bt[k]->dev.nnz_total * sizeof(MgkEntry)))) != MGK_OK) return st;
        if ((st = ensure(ctx, bi, std::max<size_t>(16, (size_t)bt[k]->dev.lanes_total * sizeof(MgkEntry)))) != MGK_OK) return st;
        hipError_t e = mgk_launch_expand(bt[k]->dev, prm, (MgkEntry*)bo.p, (MgkEntry*)bi.p, stream);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "expand launch failed: %s", hipGetErrorString(e));
        ex[k].outer = (const MgkEntry*)bo.p;
        ex[k].inner = (const MgkEntry*)bi.p;
    }

    MgkLargePair* dpairs = (MgkLargePair*)ctx->lpairs.p;
    MgkPairState* dstate = (MgkPairState*)ctx->lstate.p;
    int* dactive = (int*)ctx->lactive.p;
    float* vec = (float*)ctx->vec.p;
    // The pair records go through pinned memory owned by the context, so that the copy needs
    // no wait.
    Staging::Slot* slot_p;
    {
        const size_t bytes = (size_t)n_pairs * sizeof(MgkLargePair);
        if ((st = staging_slot(ctx, bytes, true, stream, &slot_p)) != MGK_OK) return st;
        memcpy(slot_p->p, pairs.data(), bytes);
        MGK_HIP(ctx, hipMemcpyAsync(dpairs, slot_p->p, bytes, hipMemcpyHostToDevice, stream));
        staging_copied(slot_p, stream);
    }
    MGK_HIP(ctx, hipMemsetAsync(dstate, 0, (size_t)n_pairs * sizeof(MgkPairState), stream));
    ctx->active_host[0] = n_pairs;   // pairs still iterating
    ctx->active_host[1] = 0;         // most iterations any pair needed
    MGK_HIP(ctx, hipMemcpyAsync(dactive, ctx->active_host, 2 * sizeof(int), hipMemcpyHostToDevice, stream));
    hipError_t e = mgk_launch_large_init(A->dev, Bb->dev, dpairs, dstate, vec, prm, false, n_pairs, vec_blocks, stream);
    if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "init launch failed: %s", hipGetErrorString(e));
    // The kernels of an iteration return at once for pairs that have stopped, so iterations
    // are enqueued without waiting: as many as the previous call of this kind needed, then
    // the host reads how many pairs still iterate, and goes on four at a time if any do.
    int it = 0;
    const int first_batch = std::max(1, std::min(max_iter, ctx->large_iter_guess));
    while (it < max_iter) {
        const int upto = it == 0 ? first_batch : std::min(max_iter, it + 4);
        for (; it < upto; ++it) {
            e = mgk_launch_large_iteration(A->dev, Bb->dev, ex[0], ex[1], dpairs, dstate, vec, prm, weighted,
                                           n_pairs, xmv_blocks, vec_blocks, dactive, it,
                                           dense ? &dt[0] : nullptr, dense ? &dt[1] : nullptr, rows_threads,
                                           rows_lds_bytes, rows_chunks, stream);
            if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "iteration launch failed: %s", hipGetErrorString(e));
        }
        MGK_HIP(ctx, hipMemcpyAsync(ctx->active_host, dactive, 2 * sizeof(int), hipMemcpyDeviceToHost, stream));
        MGK_HIP(ctx, hipStreamSynchronize(stream));
        slot_p->open = false;
        if (ctx->active_host[0] <= 0) break;
    }
    if (ctx->active_host[0] <= 0) ctx->large_iter_guess = std::max(1, ctx->active_host[1]);
    log_launch(ctx, "%s pairs=%d iterations_enqueued=%d entries_cached=0 (+ mgk_large_dot / update / pupdate per iteration)",
               dense ? "mgk_large_xmv_dense_kernel" : rows_threads > 0 ? "mgk_large_xmv_rows_kernel" : "mgk_large_xmv_kernel",
               n_pairs, it);
    e = mgk_launch_large_final(A->dev, Bb->dev, ex[0], ex[1], dpairs, dstate, vec, prm, weighted, n_pairs, xmv_blocks,
                               vec_blocks, dense ? &dt[0] : nullptr, dense ? &dt[1] : nullptr, rows_threads,
                               rows_lds_bytes, rows_chunks, out, stream);
    if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "final launch failed: %s", hipGetErrorString(e));
    ctx->idle = false;
    return MGK_OK;
}

// Alg. 1 with global-memory vectors and the separable product (mgk_sep.hip) for a list of pairs
// (outer graphs from A, inner from Bb).  Three launches per iteration (product with p^T a, update,
// new direction); the outputs are formed behind the iterations the last such call needed, before
// the host looks whether any pair still iterates, so that the GPU does not wait for that.  If any does,
// they are formed once more when none does.
mgk_status solve_sep(mgk_ctx* ctx, const mgk_batch* A, const mgk_batch* Bb, std::vector<MgkLargePair> pairs, int path, const MgkSepBasis& S,
                     const MgkSepLayout& L, const MgkWideBasis& SW, const MgkWideLayout& W, const MgkOutputs& out, hipStream_t stream, const MgkParams& prm) {
    const bool dense = is_sep_dense(path), parts = path == kPathSepParts, wide = path == kPathWide;
    const int n_pairs = (int)pairs.size();
    if (n_pairs == 0) return MGK_OK;
    if (!mgk_launch_sep_xmv) return fail(ctx, MGK_ESTATE, "the library was linked without the kernels of the separable product");
    int64_t total = 0;
    int max_npad = 0, max_iter = 0, max_n1 = 1, max_n2 = 1;
    for (MgkLargePair& P : pairs) {
        max_n1 = std::max(max_n1, P.n1);
        max_n2 = std::max(max_n2, P.n2);
        P.vec = total;
        total += 5 * (int64_t)P.npad;
        max_npad = std::max(max_npad, P.npad);
        max_iter = std::max(max_iter, P.max_iter);
        P.voff1 = A->graphs[(size_t)P.g1].voff;
        P.voff2 = Bb->graphs[(size_t)P.g2].voff;
    }
    const int vec_blocks = mgk_lean_blocks(n_pairs, max_npad);
    // the graphs in use and where their features go, from A and from Bb (the same list when it is A)
    const int gi = L.per_packet == 8 ? 1 : 0, sides = Bb == A ? 1 : 2;
    const mgk_batch* bt[2] = {A, Bb};
    std::vector<MgkSepGraph> used[2];
    std::vector<int64_t> place[2];   // of the features of each graph, -1: not in use
    int64_t size[2] = {0, 0};        // floats of dense F_k by the rank, or packet steps of a pass
    int32_t max_n[2] = {1, 1};
    for (int k = 0; k < sides; ++k) place[k].assign((size_t)bt[k]->n_graphs, -1);
    for (const MgkLargePair& P : pairs) {
        place[0][(size_t)P.g1] = 0;
        place[sides - 1][(size_t)P.g2] = 0;
    }
    if (wide) {   // by the part a graph has in the pairs: records of the nonzeros of outer ones, steps of inner ones
        if (max_n2 > MGK_WIDE_MAX_N) return fail(ctx, MGK_ESTATE, "an inner graph of %d vertices", max_n2);   // the limit is theirs alone
        for (int k = 0; k < 2; ++k) place[k].assign((size_t)bt[k]->n_graphs, -1);
        for (const MgkLargePair& P : pairs) place[0][(size_t)P.g1] = place[1][(size_t)P.g2] = 0;
        for (int k = 0; k < 2; ++k)
            for (int32_t g = 0; g < bt[k]->n_graphs; ++g) {
                if (place[k][(size_t)g] < 0) continue;
                const MgkGraphDesc& desc = bt[k]->graphs[(size_t)g];
                place[k][(size_t)g] = size[k];
                used[k].push_back({size[k], g, 0});
                size[k] += k == 0 ? desc.nnz : mgk_wide_inner_words(desc, W.passes);
                max_n[k] = std::max(max_n[k], desc.n);
            }
    }
    for (int k = 0; k < sides && !wide; ++k)
        for (int32_t g = 0; g < bt[k]->n_graphs; ++g) {
            int64_t& at = place[k][(size_t)g];
            if (at < 0) continue;
            const int32_t n = bt[k]->graphs[(size_t)g].n;
            const int64_t np = (n + 63) & ~63, steps0 = bt[k]->packet_off[gi][(size_t)g], steps1 = bt[k]->packet_off[gi][(size_t)g + 1];
            at = dense ? size[k] * S.rank : size[k] - steps0;
            used[k].push_back({dense ? size[k] : at, g, 0});
            size[k] += dense ? np * np : steps1 - steps0;
            max_n[k] = std::max(max_n[k], n);
        }
    std::vector<MgkSepAt> feat;
    std::vector<MgkWidePair> wide_pairs;
    feat.reserve(wide ? 0 : pairs.size());
    wide_pairs.reserve(wide ? pairs.size() : 0);
    for (const MgkLargePair& P : pairs) {
        const MgkGraphDesc &o = A->graphs[(size_t)P.g1], &i = Bb->graphs[(size_t)P.g2];
        if (wide)
            wide_pairs.push_back({P.vec, place[0][(size_t)P.g1], place[1][(size_t)P.g2], P.n1, P.n2, P.npad, o.nnz, o.voff, i.voff, mgk_wide_steps(i), {}});
        else
            feat.push_back({place[0][(size_t)P.g1], place[sides - 1][(size_t)P.g2]});
    }
    const void* const feat_data = wide ? (const void*)wide_pairs.data() : feat.data();
    const size_t feat_bytes = wide ? wide_pairs.size() * sizeof(MgkWidePair) : feat.size() * sizeof(MgkSepAt);
    // pair records, their zeroed states, the counters and the places of the features are one block and one copy;
    // the graph lists follow them in pinned memory
    const size_t state_at = ((size_t)n_pairs * sizeof(MgkLargePair) + 63) & ~(size_t)63;
    const size_t active_at = (state_at + (size_t)n_pairs * sizeof(MgkPairState) + 63) & ~(size_t)63;
    const size_t env_at = active_at + MGK_COUNTERS_BYTES, feat_at = (env_at + sizeof(MgkVectorEnv) + 63) & ~(size_t)63, copied = feat_at + feat_bytes;
    const size_t used_at[2] = {copied, copied + used[0].size() * sizeof(MgkSepGraph)};
    const size_t rec_bytes = used_at[1] + used[1].size() * sizeof(MgkSepGraph);
    mgk_status st;
    if ((st = ensure(ctx, ctx->vec, (size_t)total * sizeof(float))) != MGK_OK) return st;
    if ((st = ensure(ctx, ctx->lpairs, copied)) != MGK_OK) return st;
    if (!ctx->active_host) MGK_HIP(ctx, hipHostMalloc((void**)&ctx->active_host, 64, hipHostMallocDefault));
    struct InUse {
        bool& flag;
        ~InUse() { flag = false; }
    } in_use{ctx->features_in_use};
    ctx->features_in_use = true;
    MgkSepList sl[2] = {};
    MgkWideFeatures wf{};
    if (wide) {
        if ((st = ensure(ctx, ctx->wide_outer, std::max<size_t>(256, (size_t)W.passes * size[0] * 4 * mgk_wide_record(W.hi)))) != MGK_OK) return st;
        if ((st = ensure(ctx, ctx->wide_inner, std::max<size_t>(256, (size_t)size[1] * 4))) != MGK_OK) return st;
        wf = MgkWideFeatures{(const float*)ctx->wide_outer.p, (const float*)ctx->wide_inner.p, Bb->sep[0].deg_order, size[0]};
    }
    for (int k = 0; k < sides && !wide; ++k) {
        sl[k] = bt[k]->sep[gi];
        sl[k].total = dense ? 0 : (int32_t)size[k];
        DevBuf& buf = dense ? ctx->sep_dense[k] : ctx->sep_packets[k];
        const size_t floats = dense ? (size_t)size[k] * S.rank : ((size_t)L.passes * size[k] + 1) * 64;   // stage 2 may load one step past the last
        if ((st = ensure(ctx, buf, std::max<size_t>(256, floats * sizeof(float)))) != MGK_OK) return st;
        (dense ? sl[k].dense : sl[k].packets) = (const float*)buf.p;
    }
    if (sides == 1) sl[1] = sl[0];

    Staging::Slot* slot;
    if ((st = staging_slot(ctx, rec_bytes, true, stream, &slot)) != MGK_OK) return st;
    char* rec = static_cast<char*>(slot->p);
    for (int k = 0; k < 2; ++k) memcpy(rec + used_at[k], used[k].data(), used[k].size() * sizeof(MgkSepGraph));
    staging_copied(slot, stream);
    // features of the graphs' nonzeros (they depend on the edge kernel's parameters).  The kernels do not wait
    // for the copy: they read the list of all graphs from the batch, or one of some of them from pinned memory
    // (for all 128 graphs of 64 pairs that took 15 us more).
    if (wide) {
        const MgkSepGraph *outer = (const MgkSepGraph*)(rec + used_at[0]), *inner = (const MgkSepGraph*)(rec + used_at[1]);
        hipError_t e = mgk_launch_wide_pack(A->dev, SW, W, A->sep[0].deg_order, outer, (int)used[0].size(), inner, 0, max_n[0], size[0],
                                            (float*)ctx->wide_outer.p, (float*)ctx->wide_inner.p, stream);
        if (e == hipSuccess)
            e = mgk_launch_wide_pack(Bb->dev, SW, W, Bb->sep[0].deg_order, outer, 0, inner, (int)used[1].size(), max_n[1], size[0],
                                     (float*)ctx->wide_outer.p, (float*)ctx->wide_inner.p, stream);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "feature launch failed: %s", hipGetErrorString(e));
    }
    for (int k = 0; k < sides && !wide; ++k) {
        const bool whole = (int32_t)used[k].size() == bt[k]->n_graphs;
        const MgkSepGraph* list = whole ? sl[k].whole : (const MgkSepGraph*)(rec + used_at[k]);
        hipError_t e = dense ? mgk_launch_sep_dense_pack(bt[k]->dev, S, list, (int)used[k].size(), max_n[k], (float*)ctx->sep_dense[k].p, stream)
                             : mgk_launch_sep_pack(bt[k]->dev, S, L, sl[k], list, (int)used[k].size(), max_n[k], (float*)ctx->sep_packets[k].p, stream);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "feature launch failed: %s", hipGetErrorString(e));
    }
    memset(rec, 0, feat_at);
    memcpy(rec, pairs.data(), (size_t)n_pairs * sizeof(MgkLargePair));
    memcpy(rec + feat_at, feat_data, feat_bytes);
    const MgkVectorEnv env{A->dev.rowsum, Bb->dev.rowsum, A->dev.vlabel, Bb->dev.vlabel, prm.q, prm.h};
    memcpy(rec + env_at, &env, sizeof env);
    reinterpret_cast<int*>(rec + active_at)[0] = n_pairs;   // pairs still iterating, then the most iterations any needed
    MGK_HIP(ctx, hipMemcpyAsync(ctx->lpairs.p, rec, copied, hipMemcpyHostToDevice, stream));
    MgkLargePair* dpairs = (MgkLargePair*)ctx->lpairs.p;
    MgkPairState* dstate = (MgkPairState*)((char*)ctx->lpairs.p + state_at);
    int* dactive = (int*)((char*)ctx->lpairs.p + active_at);
    float* vec = (float*)ctx->vec.p;

    const MgkSepAt* dfeat = (const MgkSepAt*)((char*)ctx->lpairs.p + feat_at);
    auto product = [&](int it, bool check_only) {
        return wide  ? mgk_launch_wide_xmv(A->dev, Bb->dev, wf, W, (const MgkWidePair*)dfeat, dstate, vec, prm, n_pairs, max_n1, max_n2, it, check_only, stream)
             : dense ? mgk_launch_sep_dense(A->dev, Bb->dev, sl[0], sl[1], S.rank, parts, dpairs, dfeat, dstate, vec, prm, n_pairs,
                                            max_n1, max_n2, it, check_only, stream)
                     : mgk_launch_sep_xmv(A->dev, Bb->dev, sl[0], sl[1], L, dpairs, dfeat, dstate, vec, prm, n_pairs,
                                          max_n1, max_n2, it, check_only, stream);
    };
    hipError_t e = mgk_launch_large_init(A->dev, Bb->dev, dpairs, dstate, vec, prm, true, n_pairs, vec_blocks, stream);
    if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "init launch failed: %s", hipGetErrorString(e));
    int it = 0;
    const int first_batch = std::max(1, std::min(max_iter, ctx->large_iter_guess));
    ctx->active_host[0] = n_pairs;
    auto outputs = [&] {
        hipError_t f = mgk_launch_large_outputs(A->dev, Bb->dev, dpairs, dstate, vec, prm, n_pairs, vec_blocks, out, 0, stream);
        if (f == hipSuccess) f = product(0, true);
        return f != hipSuccess ? f : mgk_launch_large_outputs(A->dev, Bb->dev, dpairs, dstate, vec, prm, n_pairs, vec_blocks, out, 1, stream);
    };
    while (it < max_iter && ctx->active_host[0] > 0) {
        const bool foreseen = it == 0;
        const int upto = foreseen ? first_batch : std::min(max_iter, it + 4);
        for (; it < upto; ++it) {
            if ((e = product(it, false)) == hipSuccess)
                e = mgk_launch_large_vectors(dpairs, dstate, vec, n_pairs, vec_blocks, it, prm.rtol2, dactive, stream);
            if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "iteration launch failed: %s", hipGetErrorString(e));
        }
        if (foreseen && (e = outputs()) != hipSuccess) return fail(ctx, MGK_EDEVICE, "final launch failed: %s", hipGetErrorString(e));
        MGK_HIP(ctx, hipMemcpyAsync(ctx->active_host, dactive, 2 * sizeof(int), hipMemcpyDeviceToHost, stream));
        MGK_HIP(ctx, hipStreamSynchronize(stream));
        slot->open = false;
    }
    if (it > first_batch) {   // more iterations than foreseen
        if ((e = outputs()) != hipSuccess) return fail(ctx, MGK_EDEVICE, "final launch failed: %s", hipGetErrorString(e));
        MGK_HIP(ctx, hipStreamSynchronize(stream));
    }
    ctx->idle = true;
    if (ctx->active_host[0] <= 0) ctx->large_iter_guess = std::max(1, ctx->active_host[1]);
    char form[64];
    if (wide) snprintf(form, sizeof form, "mgk_wide_xmv_kernel<%d, %d, %d> rank=%d passes=%d", W.rows, W.hi, W.lo, SW.outer.rank, W.passes);
    else if (parts) snprintf(form, sizeof form, "mgk_sep_dense_parts_kernel rank=%d", S.rank);
    else if (dense) snprintf(form, sizeof form, "mgk_sep_dense_kernel<%d> rank=%d", mgk_sep_dense_tiles(max_n2), S.rank);
    else snprintf(form, sizeof form, "mgk_sep_xmv_kernel<%d> rank=%d passes=%d", L.rk, S.rank, L.passes);
    log_launch(ctx, "%s pairs=%d iterations_enqueued=%d entries_cached=0 (+ mgk_lean_update / pupdate per iteration)", form, n_pairs, it);
    return MGK_OK;
}

// Launch shape of the separable product for a bin of the streaming on-chip solver; waves 0: its pairs do not fit.
// Eight wavefronts for pairs of which two workgroups share a compute unit, else sixteen.
struct OnchipSep {
    int waves = 0, ept = 0, rb = 0;
    size_t lds_bytes = 0;
};
OnchipSep onchip_sep_shape(const JobBin& b, int rk) {
    static const struct { int waves, ept; } kShapes[] = {{8, 4}, {8, 8}, {16, 6}, {16, 8}, {16, 10}, {16, 12}, {16, 14}};
    OnchipSep s;
    for (const auto& c : kShapes) {
        const int np = c.waves * 64 * c.ept;
        if (np < b.sep.elements) continue;
        // most words over its pairs: p and y have a word per element and row at most, the rest grows with either graph
        const int64_t base = mgk_pcg_sep_plan(b.sep.rows, b.sep.cols, rk, 0).total +
                             2 * ((int64_t)b.sep.elements + b.sep.rows - (int64_t)b.sep.rows * (b.sep.cols | 1)) + 8;
        const int64_t slab = (int64_t)MGK_PCG_SEP_SLAB(rk) * b.sep.cols;
        const int64_t limit = (c.waves == 8 ? MGK_LDS_LIMIT_BYTES / 2 : MGK_LDS_LIMIT_BYTES) / 4;
        const int rb = (int)std::min<int64_t>((limit - base) / slab, c.waves == 8 ? 2 : 4);
        if (base + slab > limit) continue;
        s.waves = c.waves;
        s.ept = c.ept;
        s.rb = std::min(rb, (b.sep.rows + 15) / 16);
        s.lds_bytes = (size_t)(base + slab * s.rb) * 4;
        return s;
    }
    return s;
}

// Clocks of a compute unit that the separable product saves the pairs of a bin of the streaming on-chip solver in eight
// iterations.  The streaming solver evaluates 6 to 7 entries a clock, the separable one does 18 multiply-adds and waits
// about 300 clocks for a block of 16 rows (160 scale-free graphs of 96 vertices, 1080 nonzeros: 169 000 and 59 000
// clocks an iteration).
double onchip_sep_gain(const JobBin& b, int rank_executed, int passes) {
    const double rounds = (double)((b.count + 255) / 256) / (double)b.count;
    return 8.0 * rounds * ((double)b.sep.entries / 6.0 - (double)b.sep.halves * rank_executed / 18.0 - 300.0 * passes * (double)b.sep.blocks);
}

// Memory for the packets of calls that read this batch, and another one no larger: reserved when it is loaded, so that solve
// calls, also those that may not allocate, find it.  Not where every pair fits the register-resident solver.  Sizes are
// powers of two, a smaller block stays (loading waits for no call); without memory the solve calls do without.
void reserve_packets(mgk_ctx* ctx, const mgk_batch* b) {
    if (!mgk_launch_pcg_sep_rk5 || std::none_of(b->graphs.begin(), b->graphs.end(), [](const MgkGraphDesc& g) {
            return g.n > 64 || g.max_deg > MGK_REGS_MAX_DEG || g.lane_len > 64 * MGK_REGS_MAX_CHUNKS || (int)((uint32_t)g.regs_runs >> 16) > MGK_REGS_SMAX_W8;
        }))
        return;
    static_assert(64 * 64 <= 8 * 64 * MGK_REGS_MAX_EPT, "two graphs of 64 vertices");
    constexpr int kPasses = MGK_SEP_MAX_RANK / 4;   // at most, of four features
    const int64_t need = std::min<int64_t>(MGK_ONCHIP_PACKET_BYTES, 2 * ((int64_t)kPasses * b->packet_off[0].back() + 8) * 256);
    if (!ctx->onchip_packets_end && hipEventCreateWithFlags(&ctx->onchip_packets_end, hipEventDisableTiming) != hipSuccess) {
        ctx->onchip_packets_end = nullptr;
        (void)hipGetLastError();
        return;
    }
    if ((int64_t)ctx->onchip_packets.cap >= need) return;
    size_t size = (size_t)64 << 10;
    while ((int64_t)size < need) size *= 2;
    ctx->old_packets.reserve(ctx->old_packets.size() + 1);
    void* p = nullptr;
    if (hipMalloc(&p, size) != hipSuccess) {
        (void)hipGetLastError();   // no error of a later launch
        return;
    }
    if (ctx->onchip_packets.p) ctx->old_packets.push_back(ctx->onchip_packets.p);
    ctx->onchip_packets = DevBuf{p, size};
}

// Writing and reading the packets of a call: its end is recorded on every way out once something may be enqueued.
struct PacketUse {
    mgk_ctx* ctx;
    hipStream_t stream;
    bool open = false;
    hipError_t end() {
        open = false;
        return hipEventRecord(ctx->onchip_packets_end, stream);
    }
    ~PacketUse() {
        if (!open || end() == hipSuccess) return;
        (void)hipGetLastError();
        (void)hipStreamSynchronize(stream);   // nothing to wait for is left, then
    }
};

// The bins of a call that take the separable product on chip (use[k].waves > 0), and its packets in sl[].
// Not while a graph is recorded (the packets belong to the context), nor where the caller asked for
// the streaming solver.  A call that may not allocate takes the same kernels: the memory is there (reserve_packets).
mgk_status prepare_onchip_sep(mgk_ctx* ctx, const mgk_batch* X, const mgk_batch* Y, const JobList& jl, bool may_allocate, hipStream_t stream,
                              std::vector<OnchipSep>& use, MgkSepLayout& L, MgkSepList (&sl)[2], PacketUse& packets) {
    if (!separable_on_chip(ctx)) return MGK_OK;
    // Features of all graphs of the batches, formed before the kernels: 20 us with the basis and the launch, and 6 clocks of
    // a unit per nonzero and feature (23 us for 160 graphs of 1080 nonzeros).  At the lowest rank first: the basis takes time.
    auto total_gain = [&](int rank) {
        double gain = 0.0;
        for (const JobBin& b : jl.bins)
            if (b.chunks == 0 && b.sell_regs == 0 && b.sep.elements > 0 && b.sep.elements <= MGK_PCG_SEP_MAX_N)
                gain += std::max(0.0, onchip_sep_gain(b, rank, 1));
        return gain;
    };
    const int64_t nnz = X->nnz + (X == Y ? 0 : Y->nnz);
    auto cost = [&](int rank) { return 50e3 + (double)nnz * rank * 6.0 / 256.0; };
    if (total_gain(1) <= cost(1) || capturing(stream)) return MGK_OK;
    const float lo = std::min(X->label_lo, Y->label_lo), hi = std::max(X->label_hi, Y->label_hi);
    const MgkSepBasis* basis = kept_basis(ctx, lo, hi);
    if (!basis) basis = make_basis(ctx, lo, hi);
    if (basis->rank <= 0) return MGK_OK;
    const MgkSepBasis S = *basis;
    L = MgkSepLayout{};
    for (int rk : {7, 6, 5, 4, 1}) {
        if ((rk == 1) != (S.rank == 1)) continue;
        const int passes = (S.rank + rk - 1) / rk;
        if (L.rk == 0 || passes * rk < L.passes * L.rk || (passes * rk == L.passes * L.rk && passes < L.passes))
            L = mgk_pcg_sep_numbers(rk) ? MgkSepLayout{rk, passes, mgk_sep_per_packet(rk), MGK_PCG_SEP_SLAB(rk) * 4, 1}
                                        : MgkSepLayout{rk, passes, mgk_sep_per_packet(rk), 1, 0};
    }
    double gain = 0.0;
    for (size_t k = 0; k < jl.bins.size(); ++k) {
        const JobBin& b = jl.bins[k];
        if (b.chunks > 0 || b.sell_regs > 0 || b.sep.elements == 0) continue;
        const double g = onchip_sep_gain(b, L.rk * L.passes, L.passes);
        if (g <= 0.0) continue;
        use[k] = onchip_sep_shape(b, L.rk);
        if (use[k].waves > 0) gain += g;
    }
    const int gi = L.per_packet == 8 ? 1 : 0, sides = X == Y ? 1 : 2;
    const mgk_batch* bt[2] = {X, Y};
    int64_t bytes = 0;
    for (int k = 0; k < sides; ++k) bytes += ((int64_t)L.passes * bt[k]->packet_off[gi].back() + 8) * 256;
    if (gain <= cost(L.rk * L.passes) || bytes > MGK_ONCHIP_PACKET_BYTES) {
        std::fill(use.begin(), use.end(), OnchipSep{});
        return MGK_OK;
    }
    // Reserved when the graphs were loaded; a call that may allocate makes up for what was not to be had then.
    if (ctx->onchip_packets.cap < (size_t)bytes && (!may_allocate || ensure(ctx, ctx->onchip_packets, (size_t)bytes) != MGK_OK)) {
        std::fill(use.begin(), use.end(), OnchipSep{});   // short memory: the streaming solver
        return MGK_OK;
    }
    if (!ctx->onchip_packets_end) MGK_HIP(ctx, hipEventCreateWithFlags(&ctx->onchip_packets_end, hipEventDisableTiming));
    // An earlier call may still read the packets, also one on a stream of the same handle: destroyed since, or the
    // per-thread stream of another thread.  The stream waits, not the host.
    MGK_HIP(ctx, hipStreamWaitEvent(stream, ctx->onchip_packets_end, 0));
    float* to = (float*)ctx->onchip_packets.p;
    for (int k = 0; k < sides; ++k) {
        const mgk_batch* b = bt[k];
        sl[k] = b->sep[gi];
        sl[k].total = b->packet_off[gi].back();
        sl[k].packets = to;
        int32_t max_n = 1;
        for (const MgkGraphDesc& g : b->graphs) max_n = std::max(max_n, g.n);
        packets.open = true;
        hipError_t e = mgk_launch_sep_pack(b->dev, S, L, sl[k], sl[k].whole, b->n_graphs, max_n, to, stream);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "feature launch failed: %s", hipGetErrorString(e));
        to += ((size_t)L.passes * sl[k].total + 8) * 64;   // a stage loads eight steps at a time
    }
    if (sides == 1) sl[1] = sl[0];
    return MGK_OK;
}

mgk_status launch_jobs(mgk_ctx* ctx, const mgk_batch* X, const mgk_batch* Y, const JobList& jl,
                       const MgkOutputs& out, hipStream_t stream, bool may_allocate = true) {
    const MgkParams prm = make_params(ctx, X);
    const bool weighted = X->weighted || Y->weighted;
    const bool any_large = !jl.large[0].empty() || !jl.large[1].empty();
    if (any_large)   // before anything is recorded
        if (mgk_status st = refuse_capture(ctx, stream)) return st;
    ctx->calls++;
    ctx->idle = false;
    ctx->launch_log.clear();
    std::vector<OnchipSep> sep(jl.bins.size());
    MgkSepLayout onchip_layout{};
    MgkSepList onchip_lists[2] = {};
    PacketUse packets{ctx, stream};
    if (mgk_status st = prepare_onchip_sep(ctx, X, Y, jl, may_allocate, stream, sep, onchip_layout, onchip_lists, packets)) return st;
    for (const JobBin& b : jl.bins) {
        const OnchipSep& s = sep[(size_t)(&b - jl.bins.data())];
        if (s.waves > 0)
            log_launch(ctx, "mgk_pcg_sep<%d, %d, %d> passes=%d pairs=%lld entries_cached=0", onchip_layout.rk, s.ept, s.waves, onchip_layout.passes,
                       (long long)b.count);
        else if (b.sell_regs > 0)
            log_launch(ctx, "mgk_pcg_sell<%d, %d, %d> pairs=%lld entries_cached=1", b.waves, b.ept, b.sell_regs, (long long)b.count);
        else if (b.reduced)
            log_launch(ctx, "mgk_pcg_reduced<%d, %d, %d> pairs=%lld entries_cached=1", b.waves, b.ept, b.chunks, (long long)b.count);
        else if (b.chunks > 0)
            log_launch(ctx, "mgk_pcg_regs<%d, %d, %d, %d> pairs=%lld entries_cached=1", b.waves,
                       b.waves == 4 ? MGK_REGS_SMAX_W4 : MGK_REGS_SMAX_W8, b.ept, b.chunks, (long long)b.count);
        else
            log_launch(ctx, "mgk_pcg_small<%d, %d%s> pairs=%lld entries_cached=0", b.waves, b.ept,
                       b.atomic_rows ? ", atomic rows" : "", (long long)b.count);
        int64_t done = 0;
        while (done < b.count) {  // grid dimension limit
            const int64_t chunk = std::min<int64_t>(b.count - done, (int64_t)1 << 30);
            const MgkBatchDev& o = b.swapped ? Y->dev : X->dev;
            const MgkBatchDev& i = b.swapped ? X->dev : Y->dev;
            hipError_t e = s.waves > 0
                ? mgk_launch_pcg_sep(onchip_layout.rk, s.waves, s.ept, onchip_layout.passes, o, i, onchip_lists[b.swapped ? 1 : 0],
                                     onchip_lists[b.swapped ? 0 : 1], jl.dev + b.first + done, (int)chunk, prm, s.rb, s.lds_bytes, out, stream)
                : b.sell_regs > 0
                ? mgk_launch_sell(b.waves, b.ept, b.sell_regs, o, i, jl.dev + b.first + done, (int)chunk, prm,
                                  b.lds_bytes, out, stream)
                : b.reduced
                ? mgk_launch_reduced(b.waves, b.chunks, b.ept, weighted, o, i, jl.dev + b.first + done, (int)chunk,
                                     prm, b.lds_bytes, out, stream)
                : b.chunks > 0
                ? mgk_launch_regs(b.waves, b.chunks, b.ept, weighted, o, i, jl.dev + b.first + done, (int)chunk,
                                  prm, b.lds_bytes, out, stream)
                : mgk_launch_small(b.waves, b.ept, weighted, b.atomic_rows, o, i,
                                   jl.dev + b.first + done, (int)chunk, prm, b.lds_bytes, out, stream);
            if (e != hipSuccess)
                return fail(ctx, MGK_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
            done += chunk;
        }
    }
    if (packets.open) MGK_HIP(ctx, packets.end());
    if (!any_large) return MGK_OK;
    // ---- pairs with vectors in global memory: the product of each from the current edge kernel
    const bool may_sep = ctx->tile_path == MGK_TILE_AUTO && (ctx->edge_kernel == MGK_EK_SE || ctx->edge_kernel == MGK_EK_CONST);
    struct Choice {
        MgkLargePair asked, sep;   // the pair as the direct product takes it, and the separable one
        int swapped, sep_swapped;
    };
    std::vector<Choice> choices;
    choices.reserve(jl.large[0].size() + jl.large[1].size());
    for (int swapped = 0; swapped < 2; ++swapped)
        for (const MgkLargePair& asked : jl.large[swapped]) {
            Choice c{asked, asked, swapped, swapped};
            MgkLargePair& P = c.sep;
            if (may_sep && P.n2 > P.n1) {   // separable product: T has a column per inner vertex
                std::swap(P.g1, P.g2);
                std::swap(P.n1, P.n2);
                if (P.out1 < 0) P.out1 = P.out1 == MGK_OUT1_SWAPPED ? MGK_OUT1_NONE : MGK_OUT1_SWAPPED;
                if (X != Y) c.sep_swapped = 1 - swapped;
            }
            choices.push_back(c);
        }
    const int64_t n_tiles = std::min(X->n_tiles, X->nnz / 3) + (X == Y ? 0 : std::min(Y->n_tiles, Y->nnz / 3));
    // What the products of all pairs take, and the paths that they take then.  The pairs of a path are solved with the division of the largest
    // inner graph among them: once it is known which that is they are priced with it, and again while that changes.  first_look: each for
    // itself.
    auto costs_at = [&](int rank, int wide_rank, bool first_look) {
        std::vector<LargeCost> costs(choices.size());
        int32_t sep_n2 = 0, wide_n2 = 0, least = INT32_MAX;   // at first every pair has its own
        for (const Choice& c : choices) least = std::min(least, c.sep.n2);
        for (int round = 0; round < 3; ++round) {
            MgkSepLayout L{};
            MgkWideLayout W{};
            int32_t sep_at = -1, wide_at = -1;   // the inner graphs that L and W are for
            for (size_t k = 0; k < choices.size(); ++k) {
                const Choice& c = choices[k];
                if (rank > 0 && sep_at != std::max(sep_n2, c.sep.n2)) L = sep_layout(rank, sep_at = std::max(sep_n2, c.sep.n2));
                if (wide_rank > 0 && wide_at != std::max(wide_n2, c.sep.n2)) W = wide_layout(wide_rank, wide_at = std::max(wide_n2, c.sep.n2));
                costs[k] = large_cost(ctx, rank, L, W, c.sep_swapped ? Y : X, c.sep.g1, c.sep_swapped ? X : Y, c.sep.g2, (int64_t)choices.size(), n_tiles);
            }
            if (first_look) break;
            merge_paths(costs);
            join_dense(costs);
            int32_t sep_now = 0, wide_now = 0;
            for (size_t k = 0; k < choices.size(); ++k) {
                if (costs[k].best == kPathSep) sep_now = std::max(sep_now, choices[k].sep.n2);
                if (costs[k].best == kPathWide) wide_now = std::max(wide_now, choices[k].sep.n2);
            }
            if (sep_now == sep_n2 && wide_now == wide_n2) break;
            if (round == 0) {   // often all have the same: fewer divisions fit more columns, so none between has another
                const MgkSepLayout a = sep_layout(rank, least), b = sep_layout(rank, sep_now);
                const MgkWideLayout c = wide_layout(wide_rank, least), d = wide_layout(wide_rank, wide_now);
                if ((sep_now == 0 || (a.rk == b.rk && a.passes == b.passes)) &&
                    (wide_now == 0 || (c.rows == d.rows && c.hi == d.hi && c.lo == d.lo && c.passes == d.passes)))
                    break;
            }
            sep_n2 = sep_now;
            wide_n2 = wide_now;
        }
        return costs;
    };
    const bool may_wide = may_sep && ctx->edge_kernel == MGK_EK_SE && mgk_launch_wide_xmv &&
                          std::any_of(choices.begin(), choices.end(), [](const Choice& c) { return c.sep.n2 >= kWideMinColumns; });
    const MgkSepBasis none{}, *basis = &none;
    std::vector<LargeCost> costs;
    if (may_sep) {
        const float lo = std::min(X->label_lo, Y->label_lo), hi = std::max(X->label_hi, Y->label_hi);
        basis = kept_basis(ctx, lo, hi);
        if (!basis) {   // it takes time: made if any pair would take the separable product at the lowest rank
            costs = costs_at(1, may_wide ? 1 : 0, true);
            basis = std::any_of(costs.begin(), costs.end(), [](const LargeCost& C) { return is_sep(C.best); }) ? make_basis(ctx, lo, hi) : &none;
        }
    }
    // The form for graphs of many vertices takes as long to make again: only if a pair would take it with as many terms as the other form
    // has (over 120 length scales it had as many or one more).  Another length scale every call: 64 pairs of n = 256, density 0.3, 927 -> 914 us.
    static const MgkWideBasis no_wide{};
    const bool any_wide = may_wide && basis->rank > 0;
    const MgkWideBasis* made = any_wide ? wide_basis(ctx, basis, false) : &no_wide;
    costs = costs_at(basis->rank, made ? made->outer.rank : basis->rank, false);
    if (!made) {
        const bool taken = std::any_of(costs.begin(), costs.end(), [](const LargeCost& C) { return C.best == kPathWide; });
        made = taken ? wide_basis(ctx, basis, true) : &no_wide;
        if (taken) costs = costs_at(basis->rank, made->outer.rank, false);
    }
    const MgkWideBasis& wide = *made;
    const MgkSepBasis& S = *basis;
    std::vector<const Choice*> lists[2][kPaths];
    for (size_t k = 0; k < choices.size(); ++k) {
        const Choice& c = choices[k];
        const int path = costs[k].best;
        std::vector<const Choice*>& list = lists[is_sep(path) ? c.sep_swapped : c.swapped][path];
        if (list.empty()) list.reserve(choices.size() - k);
        list.push_back(&c);
    }
    auto direct = [&](const std::vector<MgkLargePair>& pairs, int swapped, bool dense) {
        return swapped ? solve_large(ctx, Y, X, 1, 0, pairs, dense, out, stream, prm, weighted)
                       : solve_large(ctx, X, Y, 0, 1, pairs, dense, out, stream, prm, weighted);
    };
    // In groups: the pair index is a grid dimension (at most 65535) and every pair of a group
    // holds 5 vectors of scratch at the same time.  The separable products put pairs and blocks of
    // outer rows into one dimension, as many blocks for every pair as the largest one has.
    constexpr size_t kMaxPairsPerGroup = 4096;
    constexpr int64_t kMaxScratchFloats = (int64_t)1 << 31;   // 8 GiB
    constexpr int64_t kMaxGridThreads = (int64_t)1 << 32;     // of a grid dimension, exclusive
    for (int path = 0; path < kPaths; ++path)
        for (int swapped = 0; swapped < 2; ++swapped) {
            auto grid_threads = [&](int64_t n_pairs, int max_n1) {
                return path == kPathWide ? mgk_wide_grid(n_pairs, max_n1, 4) * MGK_WIDE_THREADS
                     : path == kPathSep ? mgk_sep_grid(n_pairs, max_n1, MGK_SEP_ROWS) * MGK_SEP_THREADS
                     : path == kPathSepParts ? mgk_sep_grid(n_pairs, MGK_SEP_PARTS_MAX_N, 64) * MGK_SEP_PARTS_THREADS
                     : path == kPathSepDense ? mgk_sep_grid(n_pairs, max_n1, MGK_SEP_DENSE_ROWS) * MGK_SEP_DENSE_THREADS : 0;
            };
            const std::vector<const Choice*>& all = lists[swapped][path];
            auto pair = [&](size_t k) -> const MgkLargePair& { return is_sep(path) ? all[k]->sep : all[k]->asked; };
            const mgk_batch* A = swapped ? Y : X;
            const mgk_batch* B = swapped ? X : Y;
            size_t first = 0;
            while (first < all.size()) {
                std::vector<MgkLargePair> group;
                group.reserve(std::min(all.size() - first, kMaxPairsPerGroup));
                size_t last = first;
                int64_t floats = 0, features = 0;
                int max_n1 = 1, max_n2 = 1;
                for (; last < all.size() && last - first < kMaxPairsPerGroup; ++last) {
                    const MgkLargePair& P = pair(last);
                    floats += 5 * (int64_t)P.npad;
                    if (is_sep(path))   // graphs that pairs share are counted for each
                        features += path == kPathWide ? wide_feature_bytes(A, P.g1) + wide_feature_bytes(B, P.g2)
                                    : feature_bytes(A, P.g1, S.rank, is_sep_dense(path)) + feature_bytes(B, P.g2, S.rank, is_sep_dense(path));
                    max_n1 = std::max(max_n1, P.n1);
                    if (last > first && (floats > kMaxScratchFloats || features > kMaxFeatureBytes ||
                                         grid_threads((int64_t)(last - first) + 1, max_n1) >= kMaxGridThreads))
                        break;
                    max_n2 = std::max(max_n2, P.n2);
                    group.push_back(P);
                }
                mgk_status st;
                if (is_sep(path)) {
                    st = solve_sep(ctx, A, B, std::move(group), path, S, sep_layout(S.rank, max_n2), wide, wide_layout(wide.outer.rank, max_n2), out,
                                   stream, prm);
                    if (st == MGK_ENOMEM) {   // the direct product needs less
                        std::vector<MgkLargePair> again[2][2];
                        for (size_t k = first; k < last; ++k) {
                            const MgkLargePair& P = all[k]->asked;
                            const bool s = all[k]->swapped != 0;
                            again[s][use_dense_tiles(ctx, (s ? Y : X)->graphs[P.g1], (s ? X : Y)->graphs[P.g2])].push_back(P);
                        }
                        st = MGK_OK;
                        for (int s = 0; s < 2; ++s)
                            for (int d = 0; d < 2 && st == MGK_OK; ++d) st = direct(again[s][d], s, d != 0);
                    }
                } else {
                    st = direct(group, swapped, path == kPathDenseTiles);
                }
                if (st != MGK_OK) return st;
                first = last;
            }
        }
    constexpr size_t kKeptFeatureBytes = (size_t)1 << 30;   // of each buffer; forming more takes longer than allocating it
    for (DevBuf* b : {&ctx->sep_packets[0], &ctx->sep_packets[1], &ctx->sep_dense[0], &ctx->sep_dense[1], &ctx->wide_outer, &ctx->wide_inner})
        if (b->cap > kKeptFeatureBytes) {
            (void)hipFree(b->p);
            *b = DevBuf{};
        }
    return MGK_OK;
}

}  // namespace

// ============================================================================
extern "C" {

mgk_status mgk_create(mgk_ctx** out, int device) {
    if (!out) return MGK_EINVAL;
    *out = nullptr;
    if (device < -1) return MGK_EINVAL;
    if (device >= 0) {
        int count = 0;
        if (hipGetDeviceCount(&count) != hipSuccess || device >= count) return MGK_EDEVICE;
    }
    mgk_ctx* ctx = new (std::nothrow) mgk_ctx();
    if (!ctx) return MGK_ENOMEM;
    ctx->device = device;
    try {
        ctx->err.reserve(512);
        ctx->memory = std::make_shared<BatchMemory>();
        ctx->memory->events.reserve(4 * kMaxReads);
    } catch (...) { delete ctx; return MGK_ENOMEM; }
    if (device >= 0 && hipSetDevice(device) != hipSuccess) { delete ctx; return MGK_EDEVICE; }
    for (int k = 0; device >= 0 && k < 4; ++k) {   // for calls that may not create any; 1 us each
        hipEvent_t e = nullptr;
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess) ctx->memory->events.push_back(e);
    }
    *out = ctx;
    return MGK_OK;
}

void mgk_destroy(mgk_ctx* ctx) {
    if (!ctx) return;
    if (ctx->pair_jobs.dev) (void)hipFree(ctx->pair_jobs.dev);
    for (DevBuf* b : {&ctx->exp_outer[0], &ctx->exp_outer[1], &ctx->exp_inner[0], &ctx->exp_inner[1],
                      &ctx->sep_packets[0], &ctx->sep_packets[1], &ctx->sep_dense[0], &ctx->sep_dense[1], &ctx->wide_outer, &ctx->wide_inner, &ctx->onchip_packets, &ctx->vec, &ctx->lpairs, &ctx->lstate, &ctx->lactive, &ctx->nodal_off, &ctx->diag,
                      &ctx->dense_tiles[0][0], &ctx->dense_tiles[0][1], &ctx->dense_tiles[0][2],
                      &ctx->dense_tiles[1][0], &ctx->dense_tiles[1][1], &ctx->dense_tiles[1][2]})
        if (b->p) (void)hipFree(b->p);
    for (void* p : ctx->old_packets) (void)hipFree(p);
    if (ctx->active_host) (void)hipHostFree(ctx->active_host);
    if (ctx->onchip_packets_end) (void)hipEventDestroy(ctx->onchip_packets_end);
    for (Staging::Slot& s : ctx->staging.slot) {
        if (s.open) (void)hipDeviceSynchronize();
        if (s.end) (void)hipEventSynchronize(s.end->event);
        s.end.reset();
        if (s.own && s.p) (void)hipHostFree(s.p);
    }
    if (ctx->staging.block) (void)hipHostFree(ctx->staging.block);
    std::vector<FreeBlob> blobs;
    {
        std::lock_guard<std::mutex> lock(ctx->memory->m);
        ctx->memory->open = false;
        blobs.swap(ctx->memory->blobs);
    }
    for (FreeBlob& f : blobs) (void)hipFree(f.p);   // waits for the work that reads it
    blobs.clear();
    if (ctx->upload) (void)hipStreamDestroy(ctx->upload);
    delete ctx;
}

const char* mgk_last_error(const mgk_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

mgk_status mgk_set_vertex_kernel_delta(mgk_ctx* ctx, float h) {
    if (!ctx) return MGK_EINVAL;
    if (!(h > 0.f && h <= 1.f)) return fail(ctx, MGK_EINVAL, "vertex kernel h must be in (0, 1], got %g", h);
    ctx->h = h;
    return MGK_OK;
}

mgk_status mgk_set_edge_kernel_se(mgk_ctx* ctx, float length_scale) {
    if (!ctx) return MGK_EINVAL;
    if (!(length_scale > 0.f) || !std::isfinite(length_scale))
        return fail(ctx, MGK_EINVAL, "length scale must be positive and finite, got %g", length_scale);
    ctx->length_scale = length_scale;
    ctx->edge_kernel = MGK_EK_SE;
    ctx->label_dim = 1;
    return MGK_OK;
}

mgk_status mgk_set_edge_kernel_const(mgk_ctx* ctx, float c) {
    if (!ctx) return MGK_EINVAL;
    if (!(c >= 0.f && c <= 1.f)) return fail(ctx, MGK_EINVAL, "constant edge kernel must be in [0, 1], got %g", c);
    ctx->ke_const = c;
    ctx->edge_kernel = MGK_EK_CONST;
    ctx->label_dim = 1;
    return MGK_OK;
}

mgk_status mgk_set_edge_kernel_poly(mgk_ctx* ctx, int32_t n_coef, const float* coef, float rho) {
    if (!ctx) return MGK_EINVAL;
    if (n_coef < 1 || n_coef > MGK_POLY_MAX_COEF || !coef)
        return fail(ctx, MGK_EINVAL, "polynomial needs 1 to %d coefficients", MGK_POLY_MAX_COEF);
    if (!(rho > 0.f) || !std::isfinite(rho)) return fail(ctx, MGK_EINVAL, "support radius must be positive and finite, got %g", rho);
    for (int i = 0; i < n_coef; ++i)
        if (!std::isfinite(coef[i])) return fail(ctx, MGK_EINVAL, "coefficient %d is not finite", i);
    for (int k = 0; k <= 4096; ++k) {  // range of a base kernel (Section II-B)
        const double r = k / 4096.0;
        double v = 0.0;
        for (int i = n_coef - 1; i >= 0; --i) v = v * r + coef[i];
        if (v < -1e-6 || v > 1.0 + 1e-6)
            return fail(ctx, MGK_EINVAL, "polynomial is %g at r = %g, outside [0, 1]", v, r);
    }
    for (int i = 0; i < MGK_POLY_MAX_COEF; ++i) ctx->poly_c[i] = i < n_coef ? coef[i] : 0.f;
    ctx->poly_rho = rho;
    ctx->edge_kernel = MGK_EK_POLY;
    ctx->label_dim = 1;
    return MGK_OK;
}

static mgk_status set_attr_kernel(mgk_ctx* ctx, int kind, int32_t dim, const float* ls, int n_ls) {
    if (!ctx) return MGK_EINVAL;
    if (dim < 1 || dim > MGK_MAX_LABEL_DIM) return fail(ctx, MGK_EINVAL, "label attributes must be 1 to %d, got %d", MGK_MAX_LABEL_DIM, dim);
    if (!ls) return fail(ctx, MGK_EINVAL, "null length scales");
    for (int a = 0; a < n_ls; ++a)
        if (!(ls[a] > 0.f) || !std::isfinite(ls[a]))
            return fail(ctx, MGK_EINVAL, "length scale %d must be positive and finite, got %g", a, ls[a]);
    for (int a = 0; a < MGK_MAX_LABEL_DIM; ++a) ctx->attr_ls[a] = a < n_ls ? ls[a] : 1.f;
    ctx->edge_kernel = kind;
    ctx->label_dim = dim;
    return MGK_OK;
}

mgk_status mgk_set_edge_kernel_kron_se(mgk_ctx* ctx, int32_t dim, const float* length_scale) {
    return set_attr_kernel(ctx, MGK_EK_KRON_SE, dim, length_scale, dim);
}

mgk_status mgk_set_edge_kernel_rconv_se(mgk_ctx* ctx, int32_t dim, float length_scale) {
    return set_attr_kernel(ctx, MGK_EK_RCONV_SE, dim, &length_scale, 1);
}

mgk_status mgk_set_stop_prob(mgk_ctx* ctx, float q) {
    if (!ctx) return MGK_EINVAL;
    if (!(q > 0.f) || !std::isfinite(q)) return fail(ctx, MGK_EINVAL, "stopping probability must be > 0, got %g", q);
    ctx->q = q;
    return MGK_OK;
}

mgk_status mgk_set_solver(mgk_ctx* ctx, float rtol, int32_t max_iter) {
    if (!ctx) return MGK_EINVAL;
    if (!(rtol > 0.f) || !std::isfinite(rtol)) return fail(ctx, MGK_EINVAL, "rtol must be > 0, got %g", rtol);
    ctx->rtol = rtol;
    ctx->max_iter = max_iter;
    return MGK_OK;
}

mgk_status mgk_set_tile_path(mgk_ctx* ctx, int32_t mode) {
    if (!ctx) return MGK_EINVAL;
    if (mode < MGK_TILE_AUTO || mode > MGK_TILE_SPARSE_GATHER) return fail(ctx, MGK_EINVAL, "unknown tile path %d", mode);
    ctx->tile_path = mode;
    ctx->row_staging = mode == MGK_TILE_SPARSE_GATHER ? 0 : 1;
    return MGK_OK;
}

mgk_status mgk_set_onchip_limit(mgk_ctx* ctx, int32_t max_product) {
    if (!ctx) return MGK_EINVAL;
    if (max_product < 0) return fail(ctx, MGK_EINVAL, "on-chip limit must be >= 0, got %d", max_product);
    ctx->onchip_limit = std::min<int32_t>(max_product, MGK_SMALL_MAX_N);
    return MGK_OK;
}

mgk_status mgk_set_product_cache(mgk_ctx* ctx, int32_t enable) {
    if (!ctx) return MGK_EINVAL;
    if (enable < 0 || enable > 3) return fail(ctx, MGK_EINVAL, "product cache must be 0 to 3, got %d", enable);
    ctx->product_cache = enable;
    return MGK_OK;
}

mgk_status mgk_set_reduced_system(mgk_ctx* ctx, int32_t mode) {
    if (!ctx) return MGK_EINVAL;
    if (mode < 0 || mode > 2) return fail(ctx, MGK_EINVAL, "reduced system must be 0 to 2, got %d", mode);
    ctx->reduced_system = mode;
    return MGK_OK;
}

mgk_status mgk_set_schedule(mgk_ctx* ctx, int32_t cost_sorted) {
    if (!ctx) return MGK_EINVAL;
    if (cost_sorted != 0 && cost_sorted != 1) return fail(ctx, MGK_EINVAL, "schedule must be 0 or 1, got %d", cost_sorted);
    ctx->cost_sorted = cost_sorted;
    return MGK_OK;
}

mgk_status mgk_set_launch(mgk_ctx* ctx, int32_t waves_per_pair) {
    if (!ctx) return MGK_EINVAL;
    const int w = waves_per_pair;
    if (!(w == 0 || w == 1 || w == 2 || w == 4 || w == 8 || w == 16))
        return fail(ctx, MGK_EINVAL, "waves_per_pair must be 0, 1, 2, 4, 8 or 16, got %d", w);
    ctx->waves = w;
    return MGK_OK;
}

// ----------------------------------------------------------------------------
mgk_status mgk_load_graphs(mgk_ctx* ctx, int32_t n_graphs, const int64_t* vtx_off,
                           const int32_t* vtx_label, const float* start_prob,
                           const int64_t* edge_off, const int32_t* src, const int32_t* dst,
                           const float* weight, const float* edge_label, int32_t reorder,
                           mgk_batch** out) {
    return mgk_load_graphs_attr(ctx, n_graphs, vtx_off, vtx_label, start_prob, edge_off, src, dst, weight,
                                1, edge_label, reorder, out);
}

static mgk_status load_graphs_body(mgk_ctx* ctx, int32_t n_graphs, const int64_t* vtx_off,
                                   const int32_t* vtx_label, const float* start_prob,
                                   const int64_t* edge_off, const int32_t* src, const int32_t* dst,
                                   const float* weight, int32_t label_dim, const float* edge_label,
                                   int32_t reorder, int32_t coord_dim, const float* coords, mgk_batch** out);

mgk_status mgk_load_graphs_attr(mgk_ctx* ctx, int32_t n_graphs, const int64_t* vtx_off,
                                const int32_t* vtx_label, const float* start_prob,
                                const int64_t* edge_off, const int32_t* src, const int32_t* dst,
                                const float* weight, int32_t label_dim, const float* edge_label,
                                int32_t reorder, mgk_batch** out) {
    return guarded(ctx, [&] {
        return load_graphs_body(ctx, n_graphs, vtx_off, vtx_label, start_prob, edge_off, src, dst, weight,
                                label_dim, edge_label, reorder, 0, nullptr, out);
    });
}

mgk_status mgk_load_graphs_embedded(mgk_ctx* ctx, int32_t n_graphs, const int64_t* vtx_off,
                                    const int32_t* vtx_label, const float* start_prob,
                                    const int64_t* edge_off, const int32_t* src, const int32_t* dst,
                                    const float* weight, const float* edge_label, int32_t coord_dim,
                                    const float* coords, mgk_batch** out) {
    return guarded(ctx, [&]() -> mgk_status {
        if (!ctx) return MGK_EINVAL;
        if (coord_dim < 1 || coord_dim > 3) return fail(ctx, MGK_EINVAL, "coordinates must have 1 to 3 dimensions, got %d", coord_dim);
        if (!coords) return fail(ctx, MGK_EINVAL, "coords is null");
        return load_graphs_body(ctx, n_graphs, vtx_off, vtx_label, start_prob, edge_off, src, dst, weight, 1,
                                edge_label, MGK_REORDER_MORTON, coord_dim, coords, out);
    });
}

static mgk_status load_graphs_body(mgk_ctx* ctx, int32_t n_graphs, const int64_t* vtx_off,
                                   const int32_t* vtx_label, const float* start_prob,
                                   const int64_t* edge_off, const int32_t* src, const int32_t* dst,
                                   const float* weight, int32_t label_dim, const float* edge_label,
                                   int32_t reorder, int32_t coord_dim, const float* coords, mgk_batch** out) {
    if (!ctx || !out) return MGK_EINVAL;
    *out = nullptr;
    if (label_dim < 1 || label_dim > MGK_MAX_LABEL_DIM)
        return fail(ctx, MGK_EINVAL, "label attributes must be 1 to %d, got %d", MGK_MAX_LABEL_DIM, label_dim);
    const int D = label_dim;
    if (n_graphs < 0 || !vtx_off || !edge_off) return fail(ctx, MGK_EINVAL, "null offsets or negative graph count");
    if (reorder < MGK_REORDER_NONE || reorder > MGK_REORDER_MORTON || (reorder == MGK_REORDER_MORTON && !coords))
        return fail(ctx, MGK_EINVAL, "unknown reorder mode %d (the space-filling-curve order needs mgk_load_graphs_embedded)", reorder);
    if (vtx_off[0] != 0 || edge_off[0] != 0) return fail(ctx, MGK_EINVAL, "offset arrays must start at 0");
    // every array below is sized by the last offsets: they must bound all the others
    for (int32_t g = 0; g < n_graphs; ++g) {
        if (vtx_off[g + 1] <= vtx_off[g]) return fail(ctx, MGK_EINVAL, "graph %d has no vertices", g);
        if (edge_off[g + 1] < edge_off[g]) return fail(ctx, MGK_EINVAL, "graph %d: edge offsets decrease", g);
    }
    const int64_t tot_v = vtx_off[n_graphs], tot_e = edge_off[n_graphs];
    if (tot_v > 0 && !vtx_label) return fail(ctx, MGK_EINVAL, "vtx_label is null");
    if (tot_e > 0 && (!src || !dst)) return fail(ctx, MGK_EINVAL, "src/dst is null");
    if (tot_v >= (int64_t)1 << 31 || 2 * tot_e >= (int64_t)1 << 31)
        return fail(ctx, MGK_ELIMIT, "batch too large for 32-bit offsets");

    mgk_batch* B = new (std::nothrow) mgk_batch();
    if (!B) return fail(ctx, MGK_ENOMEM, "out of host memory");
    struct Guard {
        mgk_batch* b;
        ~Guard() { if (b) { if (b->blob) (void)hipFree(b->blob); delete b; } }
    } guard{B};

    B->owner = ctx;
    B->memory = ctx->memory;
    B->n_graphs = n_graphs;
    B->graphs.resize(n_graphs);
    B->vtx_off.assign(vtx_off, vtx_off + n_graphs + 1);
    B->perm.resize((size_t)tot_v);
    std::vector<int32_t> vlabel((size_t)tot_v), rowptr((size_t)tot_v), lanepos((size_t)tot_v), iperm((size_t)tot_v), trow_ptr, tile_graph;
    std::vector<MgkSellVertex> sell_vtx;            // records of the owner-computes solver
    std::vector<MgkSellNbr> sell_nbr;
    B->sell_desc.reserve((size_t)n_graphs);
    std::vector<MgkEntry> list_outer, list_inner;   // nonzero lists for the register-resident solver
    std::vector<int32_t> gptr[2], deg_order;       // packets of the separable product, rows by degree
    std::vector<int32_t> qoff((size_t)n_graphs);
    std::vector<MgkSepGraph> whole;
    whole.reserve((size_t)n_graphs);
    int64_t dense_floats = 0;
    constexpr int kPerPacket[2] = {2, 8};
    for (auto& v : gptr) v.reserve((size_t)(tot_v / 4 + 2 * (int64_t)n_graphs));
    for (auto& v : B->packet_off) v.assign((size_t)n_graphs + 1, 0);
    int32_t packets[2] = {0, 0};
    deg_order.resize((size_t)tot_v);
    B->label_lo = INFINITY;
    B->label_hi = -INFINITY;
    std::vector<int32_t> regs_split;                // its division of every graph's rows among wavefronts
    size_t list_sched_size = 0;
    list_outer.reserve((size_t)(2 * tot_e));
    // label attributes in the order of the two lists, attribute-major; filled after the loop
    // (the plane stride is the batch total): (position, edge) pairs collected meanwhile
    std::vector<std::pair<int64_t, int64_t>> attr_pos_outer, attr_pos_inner;
    B->label_dim = D;
    int64_t lanes_total = 0;
    std::vector<float> rowsum((size_t)tot_v), start((size_t)tot_v);
    B->w.reserve((size_t)(2 * tot_e));
    B->e.reserve((size_t)(2 * tot_e));
    double label_sum = 0.0;

    struct Nz { uint32_t i, j; float w, e; int64_t edge; };
    std::vector<Nz> nz, given;
    std::vector<int32_t> sorted[2], bucket, deg, filled;
    std::vector<double> rs;
    MgkAdj adj;
    std::vector<int32_t> cursor;

    // The vertex orders are by far the most expensive part of loading and independent per
    // graph: they are computed first, on several threads, for every graph whose edge list is
    // sound.  The loop below validates each graph in full (so errors are reported as before,
    // for the first bad graph) and only then takes the order computed here.  Few graphs: the
    // starting partitions of a graph are tasks of their own.
    std::vector<std::vector<int32_t>> pre_perm((size_t)n_graphs);
    if (reorder == MGK_REORDER_PBR || reorder == MGK_REORDER_RCM) {
        auto adjacency = [&](int32_t g, MgkAdj& a, std::vector<int32_t>& cur) {
            const int64_t v0 = vtx_off[g], v1 = vtx_off[g + 1], e0 = edge_off[g], e1 = edge_off[g + 1];
            if (v1 <= v0 || e1 < e0 || v1 - v0 > 65535 * (int64_t)kTile) return false;
            const int n = (int)(v1 - v0);
            a.n = n;
            a.ptr.assign(n + 1, 0);
            for (int64_t k = e0; k < e1; ++k) {
                const int32_t sv = src[k], dv = dst[k];
                if (sv < 0 || sv >= n || dv < 0 || dv >= n || sv == dv) return false;
                a.ptr[sv + 1]++;
                a.ptr[dv + 1]++;
            }
            for (int i = 0; i < n; ++i) a.ptr[i + 1] += a.ptr[i];
            a.idx.assign((size_t)(2 * (e1 - e0)), 0);
            cur.assign(a.ptr.begin(), a.ptr.end() - 1);
            for (int64_t k = e0; k < e1; ++k) {
                a.idx[cur[src[k]]++] = dst[k];
                a.idx[cur[dst[k]]++] = src[k];
            }
            for (int i = 0; i < n; ++i) std::sort(a.idx.begin() + a.ptr[i], a.idx.begin() + a.ptr[i + 1]);
            return true;
        };
        const int parts = reorder == MGK_REORDER_PBR && n_graphs < 16 ? MGK_PBR_STARTS : 1;
        std::vector<MgkPbrCandidate> cand((size_t)(parts > 1 ? n_graphs * parts : 0));
        const int T = parts > 1 ? n_graphs * parts : std::min(n_graphs, 64);
        ctx->workers.run(T, [&](int t) {
            try {   // a worker that runs out of memory stops; the loop below orders what it left
                MgkAdj a;
                std::vector<int32_t> cur;
                if (parts > 1) {
                    if (adjacency(t % n_graphs, a, cur))
                        cand[(size_t)((t % n_graphs) * parts + t / n_graphs)] = mgk_pbr_candidate(a, kTile, t / n_graphs);
                    return;
                }
                for (int32_t g = t; g < n_graphs; g += T)
                    if (adjacency(g, a, cur))
                        pre_perm[(size_t)g] = reorder == MGK_REORDER_PBR ? mgk_order_pbr(a, kTile) : mgk_order_rcm(a);
            } catch (...) {
            }
        }, (int)std::min<int64_t>(64, tot_e / 24));   // an edge takes about 3 us, starting a thread 20
        for (int32_t g = 0; parts > 1 && g < n_graphs; ++g) pre_perm[(size_t)g] = mgk_pbr_best(&cand[(size_t)g * parts]);
    }

    for (int32_t g = 0; g < n_graphs; ++g) {
        const int64_t v0 = vtx_off[g], v1 = vtx_off[g + 1], e0 = edge_off[g], e1 = edge_off[g + 1];
        if (v1 <= v0) return fail(ctx, MGK_EINVAL, "graph %d has no vertices", g);
        if (e1 < e0) return fail(ctx, MGK_EINVAL, "graph %d: edge offsets decrease", g);
        const int64_t n64 = v1 - v0, m = e1 - e0;
        if (n64 > 65535 * (int64_t)kTile) return fail(ctx, MGK_ELIMIT, "graph %d has too many vertices", g);
        const int n = (int)n64;

        // ---- validate edges
        for (int64_t k = e0; k < e1; ++k) {
            const int32_t s = src[k], d = dst[k];
            if (s < 0 || s >= n || d < 0 || d >= n)
                return fail(ctx, MGK_EINVAL, "graph %d edge %lld: endpoint out of range", g, (long long)(k - e0));
            if (s == d) return fail(ctx, MGK_EINVAL, "graph %d edge %lld: self loop", g, (long long)(k - e0));
            const float wv = weight ? weight[k] : 1.f;
            if (!(wv > 0.f) || !std::isfinite(wv))
                return fail(ctx, MGK_EINVAL, "graph %d edge %lld: weight must be finite and > 0", g, (long long)(k - e0));
            for (int a = 0; edge_label && a < D; ++a)
                if (!std::isfinite(edge_label[k * D + a]))
                    return fail(ctx, MGK_EINVAL, "graph %d edge %lld: label is not finite", g, (long long)(k - e0));
        }
        // Adjacency (both directions) and the first vertex with an edge given twice.  A graph whose order is there does without: an edge given
        // twice shows among the sorted nonzeros below.
        auto first_twice = [&] {
            adj.n = n;
            adj.ptr.assign(n + 1, 0);
            for (int64_t k = e0; k < e1; ++k) {
                adj.ptr[src[k] + 1]++;
                adj.ptr[dst[k] + 1]++;
            }
            for (int i = 0; i < n; ++i) adj.ptr[i + 1] += adj.ptr[i];
            adj.idx.assign((size_t)(2 * m), 0);
            cursor.assign(adj.ptr.begin(), adj.ptr.end() - 1);
            for (int64_t k = e0; k < e1; ++k) {
                adj.idx[cursor[src[k]]++] = dst[k];
                adj.idx[cursor[dst[k]]++] = src[k];
            }
            int first = -1;
            for (int i = n - 1; i >= 0; --i) {
                std::sort(adj.idx.begin() + adj.ptr[i], adj.idx.begin() + adj.ptr[i + 1]);
                if (std::adjacent_find(adj.idx.begin() + adj.ptr[i], adj.idx.begin() + adj.ptr[i + 1]) != adj.idx.begin() + adj.ptr[i + 1]) first = i;
            }
            return first;
        };
        int bad_prob = -1;
        for (int i = n - 1; start_prob && i >= 0; --i)
            if (!std::isfinite(start_prob[v0 + i]) || start_prob[v0 + i] < 0.f) bad_prob = i;
        bool bad_coord = false;
        for (int64_t k = v0 * coord_dim; reorder == MGK_REORDER_MORTON && k < v1 * coord_dim; ++k) bad_coord = bad_coord || !std::isfinite(coords[k]);
        const bool has_order = !pre_perm[(size_t)g].empty();
        if (bad_prob >= 0 || bad_coord || (!has_order && (reorder == MGK_REORDER_PBR || reorder == MGK_REORDER_RCM))) {
            const int i = first_twice();
            if (i >= 0) return fail(ctx, MGK_EINVAL, "graph %d: duplicate edge at vertex %d", g, i);
        }
        if (bad_prob >= 0) return fail(ctx, MGK_EINVAL, "graph %d vertex %d: bad starting probability", g, bad_prob);
        if (bad_coord) return fail(ctx, MGK_EINVAL, "graph %d: coordinate is not finite", g);

        // ---- a2: vertex order
        std::vector<int32_t> perm;
        if (has_order) perm = std::move(pre_perm[(size_t)g]);
        else if (reorder == MGK_REORDER_PBR) perm = mgk_order_pbr(adj, kTile);
        else if (reorder == MGK_REORDER_RCM) perm = mgk_order_rcm(adj);
        else if (reorder == MGK_REORDER_MORTON) perm = mgk_order_morton(n, coord_dim, coords + v0 * coord_dim);
        else perm = mgk_order_identity(n);
        std::copy(perm.begin(), perm.end(), B->perm.begin() + v0);

        // ---- per-vertex data in stored order; a1: row sums for d_i = sum_j A_ij + q
        rs.assign((size_t)n, 0.0);
        for (int64_t k = e0; k < e1; ++k) {
            const double wv = weight ? weight[k] : 1.0;
            rs[perm[src[k]]] += wv;
            rs[perm[dst[k]]] += wv;
        }
        for (int i = 0; i < n; ++i) {
            const int ni = perm[i];
            vlabel[v0 + ni] = vtx_label[v0 + i];
            iperm[v0 + ni] = i;
            start[v0 + ni] = start_prob ? start_prob[v0 + i] : 1.0f / (float)n;
            rowsum[v0 + ni] = (float)rs[ni];
        }

        // ---- a3: cut into octiles, drop empty ones, bitmap-pack
        const int ntr = (n + kTile - 1) / kTile;
        given.clear();
        given.reserve((size_t)(2 * m));
        for (int64_t k = e0; k < e1; ++k) {
            const float wv = weight ? weight[k] : 1.f;
            const float ev = edge_label ? edge_label[k * D] : 0.f;
            if (wv != 1.f) B->weighted = true;
            label_sum += 2.0 * ev;
            B->label_lo = std::min(B->label_lo, ev);
            B->label_hi = std::max(B->label_hi, ev);
            const int a = perm[src[k]], b = perm[dst[k]];
            for (int dir = 0; dir < 2; ++dir) {
                const int i = dir ? b : a, j = dir ? a : b;
                given.push_back({(uint32_t)i, (uint32_t)j, wv, ev, k});
            }
        }
        // by octile, then by bit of its bitmap: counting sorts by the bit, the octile's column and its row
        {
            auto by = [&](int buckets, const int32_t* from, std::vector<int32_t>& to, const auto& key) {
                bucket.assign((size_t)buckets + 1, 0);
                to.resize(given.size());
                for (const Nz& z : given) bucket[key(z) + 1]++;
                for (int q = 0; q < buckets; ++q) bucket[(size_t)q + 1] += bucket[(size_t)q];
                for (size_t k = 0; k < given.size(); ++k) {
                    const int32_t z = from ? from[k] : (int32_t)k;
                    to[(size_t)bucket[key(given[(size_t)z])]++] = z;
                }
            };
            by(64, nullptr, sorted[0], [](const Nz& z) { return (size_t)(z.i % kTile * kTile + z.j % kTile); });
            by(ntr, sorted[0].data(), sorted[1], [](const Nz& z) { return (size_t)(z.j / kTile); });
            by(ntr, sorted[1].data(), sorted[0], [](const Nz& z) { return (size_t)(z.i / kTile); });
            nz.resize(given.size());
            bool twice = false;
            for (size_t k = 0; k < nz.size(); ++k) {
                nz[k] = given[(size_t)sorted[0][k]];
                twice |= k > 0 && nz[k].i == nz[k - 1].i && nz[k].j == nz[k - 1].j;
            }
            if (twice) return fail(ctx, MGK_EINVAL, "graph %d: duplicate edge at vertex %d", g, first_twice());
        }

        MgkGraphDesc& gd = B->graphs[g];
        gd.n = n;
        gd.nnz = (int32_t)nz.size();
        gd.n_tile_rows = ntr;
        gd.voff = (int32_t)v0;
        gd.zoff = (int32_t)B->w.size();
        gd.toff = (int32_t)B->tiles.size();
        gd.roff = (int32_t)trow_ptr.size();
        deg.assign((size_t)n, 0);
        trow_ptr.resize(trow_ptr.size() + ntr + 1, 0);
        int32_t* trp = trow_ptr.data() + gd.roff;
        for (size_t k = 0; k < nz.size(); ++k) {
            const int tr = (int)(nz[k].i / kTile), tc = (int)(nz[k].j / kTile), bit = (int)(nz[k].i % kTile * kTile + nz[k].j % kTile);
            if (k == 0 || (int)(nz[k - 1].i / kTile) != tr || (int)(nz[k - 1].j / kTile) != tc) {
                MgkTile t;
                t.tr = (uint16_t)tr;
                t.tc = (uint16_t)tc;
                t.nzoff = (uint32_t)k;
                t.bitmap = 0;
                B->tiles.push_back(t);
                trp[tr + 1]++;
                if (tr != tc) B->n_offdiag++;
            }
            B->tiles.back().bitmap |= 1ull << bit;
            B->w.push_back(nz[k].w);
            B->e.push_back(nz[k].e);
            deg[nz[k].i]++;
        }
        for (int r = 0; r < ntr; ++r) trp[r + 1] += trp[r];
        gd.n_tiles = (int32_t)B->tiles.size() - gd.toff;
        int32_t run = 0;
        for (int i = 0; i < n; ++i) { rowptr[v0 + i] = run; run += deg[i]; }
        // lane layout as inner operand: rows packed into groups of 16 lanes
        int32_t slot = 0, max_deg = 0;
        for (int i = 0; i < n; ++i) max_deg = std::max(max_deg, deg[i]);
        const bool packed = max_deg > MGK_LANE_GROUP;   // long rows: atomic adds anyway, no gaps
        for (int i = 0; i < n; ++i) {
            const int dg = deg[i];
            const int room = MGK_LANE_GROUP - slot % MGK_LANE_GROUP;
            if (!packed && dg > room && room != MGK_LANE_GROUP) slot += room;  // start a new group
            lanepos[v0 + i] = slot;
            slot += dg;
        }
        gd.max_deg = max_deg;
        gd.lane_len = (slot + 63) & ~63;
        // rows by descending degree (counting sort), packets per row
        {
            cursor.assign((size_t)max_deg + 2, 0);
            for (int i = 0; i < n; ++i) cursor[(size_t)(max_deg - deg[i]) + 1]++;
            for (int d = 0; d <= max_deg; ++d) cursor[(size_t)d + 1] += cursor[(size_t)d];
            for (int i = 0; i < n; ++i) deg_order[(size_t)v0 + cursor[(size_t)(max_deg - deg[i])]++] = i;
            qoff[(size_t)g] = (int32_t)gptr[0].size();
            for (int i = 0; i < n; i += 4) {   // four rows of adjacent degrees: the first has the most packets
                const int d = deg[deg_order[(size_t)v0 + i]];
                for (int q = 0; q < 2; ++q) {
                    gptr[q].push_back(packets[q]);
                    packets[q] += (d + kPerPacket[q] - 1) / kPerPacket[q];
                }
            }
            for (int q = 0; q < 2; ++q) {
                gptr[q].push_back(packets[q]);
                B->packet_off[q][(size_t)g + 1] = packets[q];
            }
            const int64_t np = (n + 63) & ~63;
            whole.push_back({dense_floats, g, 0});
            dense_floats += np * np;
        }
        gd.loff = (int32_t)lanes_total;
        {
            int32_t bounds[MGK_REGS_SPLIT_STRIDE];
            const int run4 = balanced_split(deg, n, 4, bounds);
            const int run8 = balanced_split(deg, n, 8, bounds + MGK_REGS_SPLIT_W8);
            regs_split.insert(regs_split.end(), bounds, bounds + MGK_REGS_SPLIT_STRIDE);
            gd.regs_runs = (int32_t)((uint32_t)std::min(run4, 0xffff) | ((uint32_t)std::min(run8, 0xffff) << 16));
        }
        lanes_total += gd.lane_len;
        if (lanes_total >= (int64_t)1 << 31) return fail(ctx, MGK_ELIMIT, "batch too large for 32-bit offsets");
        // the same nonzeros as plain lists: CSR order (columns ascending inside a row, which is
        // the order the octiles hold them in) and lane order
        list_outer.resize((size_t)gd.zoff + nz.size());
        list_inner.resize((size_t)gd.loff + gd.lane_len, MgkEntry{0u, 0u, 0u, 0u});
        filled.assign((size_t)n, 0);
        for (size_t k = 0; k < nz.size(); ++k) {
            const uint32_t i = nz[k].i, j = nz[k].j;
            const int rank = filled[i]++;
            uint32_t wbits, ebits;
            memcpy(&wbits, &nz[k].w, 4);
            memcpy(&ebits, &nz[k].e, 4);
            const bool row_end = rank + 1 == deg[i];
            list_outer[(size_t)gd.zoff + rowptr[v0 + i] + rank] =
                MgkEntry{i, j, ebits, wbits | (row_end ? 0x80000000u : 0u)};
            const MgkRunPos rp = mgk_run_pos(lanepos[v0 + i], rank, deg[i]);
            list_inner[(size_t)gd.loff + lanepos[v0 + i] + rank] =
                MgkEntry{i | (rp.rank << 20) | (rp.cut << 30) | (rp.last << 31), j, ebits, wbits};
            if (D > 1) {
                attr_pos_outer.push_back({(int64_t)gd.zoff + rowptr[v0 + i] + rank, nz[k].edge});
                attr_pos_inner.push_back({(int64_t)gd.loff + lanepos[v0 + i] + rank, nz[k].edge});
            }
        }
        tile_graph.resize(B->tiles.size(), g);

        // ---- place of the schedule as outer operand of the reduced solver
        gd.n_red = n;
        memset(gd.red_need, 255, sizeof gd.red_need);
        gd.soff = ReducedSchedule::makes(gd) && list_sched_size < ((size_t)1 << 31) - 3 * MGK_RED_MAX_NNZ ? (int32_t)list_sched_size : -1;
        if (gd.soff >= 0) list_sched_size += 3 * (size_t)gd.nnz;

        // ---- records of the owner-computes solver: vertices sorted by degree (descending),
        //      four neighbour records per vertex
        {
            MgkSellDesc sd{};
            sd.voff = (int32_t)sell_vtx.size();
            if (n <= MGK_SELL_MAX_N && max_deg <= MGK_SELL_MAX_DEG) {
                const int32_t* order = deg_order.data() + v0;
                int32_t pos[MGK_SELL_MAX_N];
                for (int k = 0; k < n; ++k) pos[order[k]] = k;
                const int r8 = (n + 7) & ~7;
                for (int k = 0; k < r8; ++k) {
                    MgkSellVertex sv{0.f, 0.f, -1, 0xffffu};
                    MgkSellNbr sn[MGK_SELL_MAX_DEG] = {};   // weight 0, position 0: no entry
                    if (k < n) {
                        const int v = order[k];
                        sv.rowsum = rowsum[v0 + v];
                        sv.start = start[v0 + v];
                        sv.label = vlabel[v0 + v];
                        sv.id_deg = (uint32_t)v | ((uint32_t)deg[v] << 16);
                        for (int a = 0; a < deg[v]; ++a) {
                            const MgkEntry& en = list_outer[(size_t)gd.zoff + rowptr[v0 + v] + a];
                            const uint32_t wbits = en.w & 0x7fffffffu;
                            sn[a].pos = (uint32_t)pos[en.y];
                            memcpy(&sn[a].w, &wbits, 4);
                            memcpy(&sn[a].e, &en.z, 4);
                        }
                    }
                    sell_vtx.push_back(sv);
                    sell_nbr.insert(sell_nbr.end(), sn, sn + MGK_SELL_MAX_DEG);
                }
                uint32_t ga[MGK_SELL_MAX_DEG + 1] = {}, gb[MGK_SELL_MAX_DEG + 1] = {};
                for (int k = 0; k < n; k += MGK_SELL_OUTER_GROUP) ga[deg[order[k]]]++;
                for (int k = 0; k < n; k += MGK_SELL_INNER_GROUP) gb[deg[order[k]]]++;
                sd.ga03 = ga[0] | (ga[1] << 8) | (ga[2] << 16) | (ga[3] << 24);
                sd.gb03 = gb[0] | (gb[1] << 8) | (gb[2] << 16) | (gb[3] << 24);
                sd.hi = ga[4] | (gb[4] << 8) | (1u << 16);
            }
            B->sell_desc.push_back(sd);
        }
    }
    std::vector<uint16_t> red_split((size_t)n_graphs * MGK_RED_SPLIT_STRIDE), red_order((size_t)(3 * tot_v));
    std::vector<uint32_t> list_sched(list_sched_size);
    {
        constexpr int kPerTask = 16;   // graphs; 40 us
        std::atomic<bool> failed{false};
        // waking the threads a second time takes as long as the schedules of some 30 graphs
        const int tasks = (n_graphs + kPerTask - 1) / kPerTask, helpers = n_graphs < 64 ? 0 : tasks - 1;
        ctx->workers.run(tasks, [&](int t) {
            try {
                ReducedSchedule schedule;
                for (int32_t g = t * kPerTask; g < std::min(n_graphs, (t + 1) * kPerTask); ++g) {
                    MgkGraphDesc& gd = B->graphs[(size_t)g];
                    if (gd.soff >= 0)
                        schedule.make(gd, rowptr.data() + gd.voff, list_outer.data() + gd.zoff, deg_order.data() + gd.voff, list_sched.data() + gd.soff,
                                      red_split.data() + (int64_t)g * MGK_RED_SPLIT_STRIDE, red_order.data() + 3 * (int64_t)gd.voff);
                }
            } catch (...) {
                failed = true;
            }
        }, helpers);
        if (failed) return fail(ctx, MGK_ENOMEM, "out of host memory");
    }
    if (!(B->label_lo <= B->label_hi)) B->label_lo = B->label_hi = 0.f;   // no edges
    B->n_vertices = tot_v;
    B->nnz = (int64_t)B->w.size();
    B->n_tiles = (int64_t)B->tiles.size();
    B->label_mean = B->nnz ? label_sum / (double)B->nnz : 0.0;

    // ---- upload as one allocation
    BlobPlan blob;
    const size_t o_g = blob.add(B->graphs);
    const size_t o_t = blob.add(B->tiles);
    const size_t o_w = blob.add(B->w);
    const size_t o_e = blob.add(B->e);
    const size_t o_vl = blob.add(vlabel);
    const size_t o_rs = blob.add(rowsum);
    const size_t o_st = blob.add(start);
    const size_t o_rp = blob.add(rowptr);
    const size_t o_lp = blob.add(lanepos);
    const size_t o_tr = blob.add(trow_ptr);
    const size_t o_tg = blob.add(tile_graph);
    const size_t o_ip = blob.add(iperm);
    const size_t o_lo = blob.add(list_outer);
    const size_t o_li = blob.add(list_inner);
    const size_t o_sp = blob.add(regs_split), o_rd = blob.add(red_split), o_ls = blob.add(list_sched), o_ro = blob.add(red_order);
    std::vector<float> attr_outer, attr_inner;
    if (D == 1) {   // the labels of the lists
        attr_outer.resize(list_outer.size());
        attr_inner.resize(list_inner.size());
        for (size_t k = 0; k < list_outer.size(); ++k) memcpy(&attr_outer[k], &list_outer[k].z, 4);
        for (size_t k = 0; k < list_inner.size(); ++k) memcpy(&attr_inner[k], &list_inner[k].z, 4);
    } else {
        attr_outer.assign((size_t)D * B->w.size(), 0.f);
        attr_inner.assign((size_t)D * (size_t)lanes_total, 0.f);
        for (const auto& pe : attr_pos_outer)
            for (int a = 0; a < D; ++a)
                attr_outer[(size_t)a * B->w.size() + (size_t)pe.first] = edge_label ? edge_label[pe.second * D + a] : 0.f;
        for (const auto& pe : attr_pos_inner)
            for (int a = 0; a < D; ++a)
                attr_inner[(size_t)a * (size_t)lanes_total + (size_t)pe.first] = edge_label ? edge_label[pe.second * D + a] : 0.f;
    }
    const size_t o_ao = blob.add(attr_outer);
    const size_t o_ai = blob.add(attr_inner);
    const size_t o_pk[2] = {blob.add(gptr[0]), blob.add(gptr[1])};
    const size_t o_do = blob.add(deg_order), o_qo = blob.add(qoff), o_wh = blob.add(whole);
    const size_t o_sd = blob.add(B->sell_desc);
    const size_t o_sv = blob.add(sell_vtx);
    const size_t o_sn = blob.add(sell_nbr);
    B->dev.label_dim = D;
    B->dev.uniform_start = start_prob ? 0 : 1;
    B->dev.n_graphs = n_graphs;
    B->dev.n_tiles_total = (int32_t)B->tiles.size();
    B->dev.nnz_total = (int32_t)B->w.size();
    B->dev.lanes_total = (int32_t)lanes_total;
    if (ctx->device < 0) {  // host-only context: packed form is kept for inspection only
        guard.b = nullptr;
        *out = B;
        return MGK_OK;
    }
    MGK_HIP(ctx, hipSetDevice(ctx->device));
    if (mgk_status st = take_blob(ctx, blob.total, &B->blob, &B->blob_cap)) return st;
    if (ctx->calls == 0 || blob.total > kMaxStagedBytes) {
        std::vector<char> flat(blob.total);
        blob.copy_to(flat.data());
        MGK_HIP(ctx, hipMemcpy(B->blob, flat.data(), blob.total, hipMemcpyHostToDevice));
    } else {   // on a stream of the context: waits for its own copy, not for the calls under way
        Staging::Slot* slot;
        if (!ctx->upload) MGK_HIP(ctx, hipStreamCreateWithFlags(&ctx->upload, hipStreamNonBlocking));
        if (mgk_status st = staging_slot(ctx, blob.total, true, ctx->upload, &slot)) return st;
        blob.copy_to(static_cast<char*>(slot->p));
        MGK_HIP(ctx, hipMemcpyAsync(B->blob, slot->p, blob.total, hipMemcpyHostToDevice, ctx->upload));
        MGK_HIP(ctx, hipStreamSynchronize(ctx->upload));
    }
    char* base = static_cast<char*>(B->blob);
    B->dev.graphs = reinterpret_cast<const MgkGraphDesc*>(base + o_g);
    B->dev.tiles = reinterpret_cast<const MgkTile*>(base + o_t);
    B->dev.w = reinterpret_cast<const float*>(base + o_w);
    B->dev.e = reinterpret_cast<const float*>(base + o_e);
    B->dev.vlabel = reinterpret_cast<const int32_t*>(base + o_vl);
    B->dev.rowsum = reinterpret_cast<const float*>(base + o_rs);
    B->dev.start = reinterpret_cast<const float*>(base + o_st);
    B->dev.rowptr = reinterpret_cast<const int32_t*>(base + o_rp);
    B->dev.lanepos = reinterpret_cast<const int32_t*>(base + o_lp);
    B->dev.trow_ptr = reinterpret_cast<const int32_t*>(base + o_tr);
    B->dev.tile_graph = reinterpret_cast<const int32_t*>(base + o_tg);
    B->dev.iperm = reinterpret_cast<const int32_t*>(base + o_ip);
    B->dev.list_outer = reinterpret_cast<const MgkEntry*>(base + o_lo);
    B->dev.list_inner = reinterpret_cast<const MgkEntry*>(base + o_li);
    B->dev.regs_split = reinterpret_cast<const int32_t*>(base + o_sp);
    B->dev.red_split = reinterpret_cast<const uint16_t*>(base + o_rd);
    B->dev.list_sched = reinterpret_cast<const uint32_t*>(base + o_ls);
    B->dev.red_order = reinterpret_cast<const uint16_t*>(base + o_ro);
    B->dev.attr_outer = reinterpret_cast<const float*>(base + o_ao);
    B->dev.attr_inner = reinterpret_cast<const float*>(base + o_ai);
    for (int q = 0; q < 2; ++q) {
        B->sep[q].qoff = reinterpret_cast<const int32_t*>(base + o_qo);
        B->sep[q].gptr = reinterpret_cast<const int32_t*>(base + o_pk[q]);
        B->sep[q].whole = reinterpret_cast<const MgkSepGraph*>(base + o_wh);
        B->sep[q].deg_order = reinterpret_cast<const int32_t*>(base + o_do);
    }
    B->dev.sell_desc = reinterpret_cast<const MgkSellDesc*>(base + o_sd);
    B->dev.sell_vtx = reinterpret_cast<const MgkSellVertex*>(base + o_sv);
    B->dev.sell_nbr = reinterpret_cast<const MgkSellNbr*>(base + o_sn);
    reserve_packets(ctx, B);

    guard.b = nullptr;
    *out = B;
    return MGK_OK;
}

void mgk_free_batch(mgk_ctx*, mgk_batch* batch) {   // the context may be gone
    if (!batch) return;
    bool kept = false;
    if (batch->blob) {
        try { kept = keep_blob(batch); } catch (...) {}
    }
    if ((batch->blob && !kept) || batch->gram_jobs[0].list.dev || batch->gram_jobs[1].list.dev) (void)hipDeviceSynchronize();
    for (auto& g : batch->gram_jobs)
        if (g.list.dev) (void)hipFree(g.list.dev);
    for (void* p : batch->old_jobs) (void)hipFree(p);
    if (batch->blob && !kept) (void)hipFree(batch->blob);
    delete batch;
}

mgk_status mgk_batch_stats(const mgk_batch* b, int64_t* n_graphs, int64_t* n_vertices, int64_t* nnz,
                           int64_t* n_tiles, int64_t* n_offdiag_tiles) {
    if (!b) return MGK_EINVAL;
    if (n_graphs) *n_graphs = b->n_graphs;
    if (n_vertices) *n_vertices = b->n_vertices;
    if (nnz) *nnz = b->nnz;
    if (n_tiles) *n_tiles = b->n_tiles;
    if (n_offdiag_tiles) *n_offdiag_tiles = b->n_offdiag;
    return MGK_OK;
}

mgk_status mgk_batch_permutation(const mgk_batch* b, int32_t* perm_host) {
    if (!b || !perm_host) return MGK_EINVAL;
    std::copy(b->perm.begin(), b->perm.end(), perm_host);
    return MGK_OK;
}

mgk_status mgk_batch_get_tiles(const mgk_batch* b, int32_t g, int32_t* n_tiles, int32_t* nnz,
                               int32_t* tile_row, int32_t* tile_col, uint64_t* bitmap, float* w,
                               float* e) {
    if (!b || g < 0 || g >= b->n_graphs) return MGK_EINVAL;
    const MgkGraphDesc& gd = b->graphs[g];
    if (n_tiles) *n_tiles = gd.n_tiles;
    if (nnz) *nnz = gd.nnz;
    for (int t = 0; t < gd.n_tiles; ++t) {
        const MgkTile& tl = b->tiles[gd.toff + t];
        if (tile_row) tile_row[t] = tl.tr;
        if (tile_col) tile_col[t] = tl.tc;
        if (bitmap) bitmap[t] = tl.bitmap;
    }
    if (w) std::copy(b->w.begin() + gd.zoff, b->w.begin() + gd.zoff + gd.nnz, w);
    if (e) std::copy(b->e.begin() + gd.zoff, b->e.begin() + gd.zoff + gd.nnz, e);
    return MGK_OK;
}

// ----------------------------------------------------------------------------
static mgk_status gram_body(mgk_ctx* ctx, mgk_batch* batch, float* K_dev, int32_t* iters_dev,
                            int32_t* flag_dev, void* stream_);

mgk_status mgk_gram(mgk_ctx* ctx, mgk_batch* batch, float* K_dev, int32_t* iters_dev,
                    int32_t* flag_dev, void* stream_) {
    return guarded(ctx, [&] { return gram_body(ctx, batch, K_dev, iters_dev, flag_dev, stream_); });
}

static mgk_status gram_body(mgk_ctx* ctx, mgk_batch* batch, float* K_dev, int32_t* iters_dev,
                            int32_t* flag_dev, void* stream_) {
    if (!ctx || !batch || !K_dev) return fail(ctx, MGK_EINVAL, "null argument");
    if (batch->owner != ctx) return fail(ctx, MGK_ESTATE, "batch belongs to another context");
    if (ctx->device < 0) return fail(ctx, MGK_ESTATE, "host-only context cannot solve");
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (mgk_status st = check_label_dim(ctx, batch, batch)) return st;
    MGK_HIP(ctx, hipSetDevice(ctx->device));
    const int64_t G = batch->n_graphs;
    if (G * G >= (int64_t)1 << 31) return fail(ctx, MGK_ELIMIT, "Gram matrix too large for 32-bit output indices");
    auto built = [&](const mgk_batch::GramJobs& g) {
        return g.list.dev != nullptr && g.waves == ctx->waves && g.max_iter == ctx->max_iter && g.limit == ctx->onchip_limit &&
               g.cache == ctx->product_cache && g.sorted == ctx->cost_sorted && g.attr_dim == attr_dim_of(ctx) && !(g.joined && ctx->reduced_system == 2) &&
               // other launches, but the same pairs: good enough while a graph is recorded
               (!g.any_big || g.separable == separable_on_chip(ctx) || capturing(stream));
    };
    bool reduced = solve_reduced(ctx, iters_dev);
    const int waves = reduced_waves(G * (G + 1) / 2);
    // While a graph is recorded the list has to be there.  The one of the other system will do if the call shows no iterates and the
    // system was not asked for; otherwise it says that a list of the batch was made with these settings, and the one wanted is made now,
    // on a stream that takes no part in the recording.
    bool beside = false;
    if (!built(batch->gram_jobs[reduced]) && built(batch->gram_jobs[!reduced]) && capturing(stream)) {
        if (reduced && ctx->reduced_system == 1) reduced = false;
        else beside = true;
    }
    mgk_batch::GramJobs& jobs = batch->gram_jobs[reduced];
    std::optional<RelaxedCapture> relaxed;
    if (beside) {
        relaxed.emplace();
        if (!ctx->upload) MGK_HIP(ctx, hipStreamCreateWithFlags(&ctx->upload, hipStreamNonBlocking));
        if (jobs.list.dev) {
            batch->old_jobs.push_back(jobs.list.dev);
            jobs.list.dev = nullptr;
        }
    }
    if (jobs.list.dev != nullptr && !built(jobs)) {
        if (mgk_status st = refuse_capture(ctx, stream)) return st;
        MGK_HIP(ctx, hipStreamSynchronize(stream));  // launch shape changed: rebuild the job list
        MGK_HIP(ctx, hipFree(jobs.list.dev));
        jobs.list.dev = nullptr;
        for (void* p : batch->old_jobs) (void)hipFree(p);
        batch->old_jobs.clear();
    }
    if (jobs.list.dev == nullptr && G > 0) {
        if (!beside)   // the list is copied and waited for
            if (mgk_status st = refuse_capture(ctx, stream)) return st;
        // a4: job list, one job per unordered pair, kept with the batch
        JobPlan plan(separable_on_chip(ctx));
        plan.jobs.reserve((size_t)(G * (G + 1) / 2));
        for (auto& v : jobs.list.large) v.clear();
        // the plans of the G (G + 1) / 2 pairs are independent: rows of the triangle in turn on
        // several threads, row i starting at pair i G - i (i - 1) / 2
        std::vector<PairPlan> plans((size_t)(G * (G + 1) / 2));
        PlanKinds kinds;
        {
            const int cache = ctx->product_cache;
            const int attr_dim = attr_dim_of(ctx);
            const int forced = ctx->waves, limit = ctx->onchip_limit;
            const int T = (int)std::max<int64_t>(1, std::min<int64_t>(64, G / 64));
            ctx->workers.run(T, [&](int t) {   // allocates nothing, cannot throw
                PlanKinds::Part kinds_here;
                for (int64_t i = t; i < G; i += T) {
                    PairPlan* row = plans.data() + (i * G - i * (i - 1) / 2);
                    for (int64_t j = i; j < G; ++j) {
                        row[j - i] = plan_pair(batch->graphs[i], batch->graphs[j], &batch->sell_desc[(size_t)i],
                                               &batch->sell_desc[(size_t)j], true, forced, limit, cache, attr_dim, reduced ? waves : 0);
                        kinds_here.add(row[j - i], false);
                    }
                }
                kinds.add(kinds_here);
            });
        }
        jobs.joined = false;
        if (reduced) {
            std::vector<int64_t> row((size_t)G);   // first pair of each row of the triangle
            for (int64_t i = 0; i < G; ++i) row[(size_t)i] = i * G - i * (i - 1) / 2;
            auto graphs_of = [&](size_t k) {
                const int64_t i = std::upper_bound(row.begin(), row.end(), (int64_t)k) - row.begin() - 1;
                return std::make_pair(&batch->graphs[(size_t)i], &batch->graphs[(size_t)(i + (int64_t)k - row[(size_t)i])]);
            };
            if (ctx->reduced_system == 1) jobs.joined = join_few(plans, graphs_of, ctx->onchip_limit, attr_dim_of(ctx));
            join_full(plans, kinds, false, graphs_of, ctx->onchip_limit, attr_dim_of(ctx));
        }
        size_t next_plan = 0;
        for (int64_t i = 0; i < G; ++i)
            for (int64_t j = i; j < G; ++j) {
                const PairPlan pl = plans[next_plan++];
                HostJob hj;
                hj.job.g1 = (int32_t)(pl.swap ? j : i);
                hj.job.g2 = (int32_t)(pl.swap ? i : j);
                hj.job.out0 = (int32_t)(i * G + j);
                hj.job.out1 = i == j ? -1 : (int32_t)(j * G + i);
                if (pl.waves == 0) {  // vectors do not fit on chip
                    if ((int64_t)batch->graphs[i].n * batch->graphs[j].n >= ((int64_t)1 << 31) - 64)
                        return fail(ctx, MGK_ELIMIT, "pair (%lld, %lld) is too large", (long long)i, (long long)j);
                    bool sw;
                    MgkLargePair P = plan_large(batch->graphs[i], batch->graphs[j], (int32_t)i, (int32_t)j, &sw, ctx->max_iter);
                    P.out0 = hj.job.out0;
                    P.out1 = hj.job.out1;
                    jobs.list.large[0].push_back(P);
                    continue;
                }
                hj.cost = pl.cost;
                hj.shape = plan.shape_of(pl, false, batch->graphs[i], batch->graphs[j]);   // one batch: swapping is done through the indices
                plan.jobs.push_back(hj);
            }
        mgk_status st = build_job_list(ctx, plan, jobs.list, beside ? ctx->upload : stream, nullptr);
        jobs.waves = ctx->waves;
        jobs.max_iter = ctx->max_iter;
        jobs.limit = ctx->onchip_limit;
        jobs.cache = ctx->product_cache;
        jobs.sorted = ctx->cost_sorted;
        jobs.attr_dim = attr_dim_of(ctx);
        jobs.any_big = plan.any_big;
        jobs.separable = plan.separable;
        if (st != MGK_OK) return st;
    }
    relaxed.reset();
    batch->untracked = true;   // its job list has freeing wait as well
    const MgkOutputs out{K_dev, iters_dev, flag_dev, nullptr, nullptr};
    return launch_jobs(ctx, batch, batch, jobs.list, out, stream);
}

// no_alloc: the job list goes to the fixed device array of mgk_noalloc.hip, pairs that need
// the global-memory solver (whose vectors the library would allocate) are refused, and no
// HIP allocation call is made on any path.
static mgk_status pairs_impl(mgk_ctx* ctx, mgk_batch* X, mgk_batch* Y, int64_t n_pairs,
                             const int32_t* i_host, const int32_t* j_host, float* K_dev,
                             float* x_dev, const int64_t* x_off_host, int32_t* iters_dev,
                             int32_t* flag_dev, void* stream_, bool no_alloc = false) {
    if (!ctx || !X || !Y) return fail(ctx, MGK_EINVAL, "null argument");
    if (X->owner != ctx || Y->owner != ctx) return fail(ctx, MGK_ESTATE, "batch belongs to another context");
    if (ctx->device < 0) return fail(ctx, MGK_ESTATE, "host-only context cannot solve");
    if (n_pairs < 0 || n_pairs >= (int64_t)1 << 31) return fail(ctx, MGK_EINVAL, "bad pair count");
    if (n_pairs == 0) return MGK_OK;
    if (!i_host || !j_host || !K_dev) return fail(ctx, MGK_EINVAL, "null argument");
    if (mgk_status st = check_label_dim(ctx, X, Y)) return st;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    MGK_HIP(ctx, hipSetDevice(ctx->device));
    if (mgk_status st = refuse_capture(ctx, stream)) return st;
    // Either graph of a pair may be the outer operand; jobs whose outer graph
    // comes from Y are launched with the batch arguments exchanged.
    for (int64_t k = 0; k < n_pairs; ++k)
        if (i_host[k] < 0 || i_host[k] >= X->n_graphs || j_host[k] < 0 || j_host[k] >= Y->n_graphs)
            return fail(ctx, MGK_EINVAL, "pair %lld: graph index out of range", (long long)k);
    std::vector<PairPlan> plans((size_t)n_pairs);
    PlanKinds kinds;
    {
        constexpr int64_t kPart = 1024;   // about 20 us of planning
        const int attr_dim = attr_dim_of(ctx);
        const int reduced = solve_reduced(ctx, iters_dev) ? reduced_waves(n_pairs) : 0;
        ctx->workers.run((int)((n_pairs + kPart - 1) / kPart), [&](int t) {   // allocates nothing, cannot throw
            const int64_t end = std::min(n_pairs, (t + 1) * kPart);
            PlanKinds::Part kinds_here;
            for (int64_t k = t * kPart; k < end; ++k) {
                const int32_t i = i_host[k], j = j_host[k];
                plans[(size_t)k] = plan_pair(X->graphs[i], Y->graphs[j], &X->sell_desc[(size_t)i], &Y->sell_desc[(size_t)j], true,
                                             ctx->waves, ctx->onchip_limit, ctx->product_cache, attr_dim, reduced);
                kinds_here.add(plans[(size_t)k], X != Y);
            }
            kinds.add(kinds_here);
        });
    }
    if (solve_reduced(ctx, iters_dev)) {
        auto graphs_of = [&](size_t k) { return std::make_pair(&X->graphs[(size_t)i_host[k]], &Y->graphs[(size_t)j_host[k]]); };
        if (ctx->reduced_system == 1) join_few(plans, graphs_of, ctx->onchip_limit, attr_dim_of(ctx));
        join_full(plans, kinds, X != Y, graphs_of, ctx->onchip_limit, attr_dim_of(ctx));
    }
    JobPlan plan(separable_on_chip(ctx));
    plan.jobs.reserve((size_t)n_pairs);
    std::vector<MgkLargePair> large[2];
    for (int64_t k = 0; k < n_pairs; ++k) {
        const int32_t i = i_host[k], j = j_host[k];
        const PairPlan& pl = plans[(size_t)k];
        if (pl.waves == 0) {
            if (no_alloc)
                return fail(ctx, MGK_ELIMIT, "pair %lld (%d x %d vertices) needs the global-memory solver, "
                            "which allocates its vectors", (long long)k, X->graphs[i].n, Y->graphs[j].n);
            if ((int64_t)X->graphs[i].n * Y->graphs[j].n >= ((int64_t)1 << 31) - 64)
                return fail(ctx, MGK_ELIMIT, "pair %lld is too large", (long long)k);
            bool sw;
            MgkLargePair P = plan_large(X->graphs[i], Y->graphs[j], i, j, &sw, ctx->max_iter);
            P.out0 = (int32_t)k;
            P.out1 = sw ? MGK_OUT1_SWAPPED : MGK_OUT1_NONE;
            large[(sw && X != Y) ? 1 : 0].push_back(P);
            continue;
        }
        HostJob hj;
        hj.job.g1 = pl.swap ? j : i;
        hj.job.g2 = pl.swap ? i : j;
        hj.job.out0 = (int32_t)k;
        hj.job.out1 = pl.swap ? MGK_OUT1_SWAPPED : MGK_OUT1_NONE;
        hj.cost = pl.cost;
        hj.shape = plan.shape_of(pl, pl.swap && X != Y && !pl.reduced, X->graphs[(size_t)i], Y->graphs[(size_t)j]);
        plan.jobs.push_back(hj);
    }
    // The previous call's kernels may still read the job buffer: on the same stream the copy below
    // is ordered behind them.
    if (!no_alloc && ctx->pair_jobs_busy && ctx->pair_jobs_stream != stream) {
        MGK_HIP(ctx, hipStreamSynchronize(ctx->pair_jobs_stream));
        ctx->pair_jobs_busy = false;
    }
    BatchReads reads(X, Y);
    MgkOutputs out{K_dev, iters_dev, flag_dev, nullptr, nullptr};
    if (no_alloc) {
        // Job list in the fixed array of this GPU.  All calls on the GPU share it: a call
        // that overlaps another one's kernels would overwrite the jobs they still read,
        // so within this context a previous such call on another stream is waited for first.
        if (ctx->fixed_jobs_busy && ctx->fixed_jobs_stream != stream) {
            MGK_HIP(ctx, hipStreamSynchronize(ctx->fixed_jobs_stream));
            ctx->fixed_jobs_busy = false;
        }
        JobList fixed;
        int64_t cap = 0;
        hipError_t e = mgk_noalloc_job_storage(ctx->device, &fixed.dev, &cap);
        if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "fixed job storage: %s", hipGetErrorString(e));
        mgk_status st = build_job_list(ctx, plan, fixed, stream, &cap, true);
        if (st != MGK_OK) return st;
        ctx->fixed_jobs_stream = stream;
        ctx->fixed_jobs_busy = true;
        if ((st = launch_jobs(ctx, X, Y, fixed, out, stream, false)) == MGK_OK) reads.done(ctx->staging, stream, false, ctx->idle);
        return st;
    }
    mgk_status st = build_job_list(ctx, plan, ctx->pair_jobs, stream, &ctx->pair_jobs_cap);
    if (st != MGK_OK) return st;
    for (int a = 0; a < 2; ++a) ctx->pair_jobs.large[a] = std::move(large[a]);
    ctx->pair_jobs_stream = stream;
    ctx->pair_jobs_busy = true;
    if (x_dev) {
        if ((st = ensure(ctx, ctx->nodal_off, (size_t)n_pairs * sizeof(int64_t))) != MGK_OK) return st;
        const size_t bytes = (size_t)n_pairs * sizeof(int64_t);
        Staging::Slot* slot;
        if ((st = staging_slot(ctx, bytes, true, stream, &slot)) != MGK_OK) return st;
        memcpy(slot->p, x_off_host, bytes);
        MGK_HIP(ctx, hipMemcpyAsync(ctx->nodal_off.p, slot->p, bytes, hipMemcpyHostToDevice, stream));
        staging_copied(slot, stream);
        out.nodal = x_dev;
        out.nodal_off = (const int64_t*)ctx->nodal_off.p;
    }
    if ((st = launch_jobs(ctx, X, Y, ctx->pair_jobs, out, stream)) == MGK_OK) reads.done(ctx->staging, stream, true, ctx->idle);
    return st;
}

mgk_status mgk_pairs(mgk_ctx* ctx, mgk_batch* X, mgk_batch* Y, int64_t n_pairs,
                     const int32_t* i_host, const int32_t* j_host, float* K_dev, int32_t* iters_dev,
                     int32_t* flag_dev, void* stream_) {
    return guarded(ctx, [&] {
        return pairs_impl(ctx, X, Y, n_pairs, i_host, j_host, K_dev, nullptr, nullptr, iters_dev, flag_dev, stream_);
    });
}

mgk_status mgk_pairs_dev(mgk_ctx* ctx, mgk_batch* X, mgk_batch* Y, int64_t n_pairs,
                         const int32_t* i_dev, const int32_t* j_dev, float* K_dev, int32_t* iters_dev,
                         int32_t* flag_dev, void* stream_) {
    return guarded(ctx, [&]() -> mgk_status {
        if (!ctx || !X || !Y) return fail(ctx, MGK_EINVAL, "null argument");
        if (ctx->device < 0) return fail(ctx, MGK_ESTATE, "host-only context cannot solve");
        if (n_pairs < 0 || n_pairs >= (int64_t)1 << 31) return fail(ctx, MGK_EINVAL, "bad pair count");
        if (n_pairs == 0) return MGK_OK;
        if (!i_dev || !j_dev) return fail(ctx, MGK_EINVAL, "null argument");
        // the launch shape of a pair is chosen on the host from the sizes of its graphs
        hipStream_t stream = static_cast<hipStream_t>(stream_);
        MGK_HIP(ctx, hipSetDevice(ctx->device));
        if (mgk_status st = refuse_capture(ctx, stream)) return st;   // before the copies are recorded
        std::vector<int32_t> ij((size_t)(2 * n_pairs));
        MGK_HIP(ctx, hipMemcpyAsync(ij.data(), i_dev, (size_t)n_pairs * sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        MGK_HIP(ctx, hipMemcpyAsync(ij.data() + n_pairs, j_dev, (size_t)n_pairs * sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        MGK_HIP(ctx, hipStreamSynchronize(stream));
        return pairs_impl(ctx, X, Y, n_pairs, ij.data(), ij.data() + n_pairs, K_dev, nullptr, nullptr, iters_dev,
                          flag_dev, stream_);
    });
}

mgk_status mgk_pairs_noalloc(mgk_ctx* ctx, mgk_batch* X, mgk_batch* Y, int64_t n_pairs,
                             const int32_t* i_host, const int32_t* j_host, float* K_dev, int32_t* iters_dev,
                             int32_t* flag_dev, void* stream_) {
    return guarded(ctx, [&]() -> mgk_status {
        if (n_pairs > MGK_NOALLOC_MAX_PAIRS)
            return fail(ctx, MGK_ELIMIT, "mgk_pairs_noalloc takes at most %d pairs per call, got %lld",
                        MGK_NOALLOC_MAX_PAIRS, (long long)n_pairs);
        return pairs_impl(ctx, X, Y, n_pairs, i_host, j_host, K_dev, nullptr, nullptr, iters_dev, flag_dev, stream_,
                          true);
    });
}

mgk_status mgk_pairs_nodal(mgk_ctx* ctx, mgk_batch* X, mgk_batch* Y, int64_t n_pairs,
                           const int32_t* i_host, const int32_t* j_host, float* K_dev, float* x_dev,
                           const int64_t* x_off_host, int32_t* iters_dev, int32_t* flag_dev,
                           void* stream_) {
    if (n_pairs > 0 && (!x_dev || !x_off_host)) return fail(ctx, MGK_EINVAL, "null nodal output");
    return guarded(ctx, [&] {
        return pairs_impl(ctx, X, Y, n_pairs, i_host, j_host, K_dev, x_dev, x_off_host, iters_dev, flag_dev, stream_);
    });
}

int64_t mgk_launch_log(const mgk_ctx* ctx, char* buf, int64_t capacity) {
    if (!ctx) return -1;
    const int64_t need = (int64_t)ctx->launch_log.size() + 1;
    if (buf && capacity > 0) {
        const int64_t n = std::min<int64_t>(capacity - 1, (int64_t)ctx->launch_log.size());
        memcpy(buf, ctx->launch_log.data(), (size_t)n);
        buf[n] = 0;
    }
    return need;
}

mgk_status mgk_normalize_gram(mgk_ctx* ctx, int32_t n, float* K_dev, void* stream_) {
    if (!ctx || n < 0 || (n > 0 && !K_dev)) return fail(ctx, MGK_EINVAL, "bad argument");
    if (ctx->device < 0) return fail(ctx, MGK_ESTATE, "host-only context cannot solve");
    if (n == 0) return MGK_OK;
    MGK_HIP(ctx, hipSetDevice(ctx->device));
    mgk_status st = ensure(ctx, ctx->diag, (size_t)n * sizeof(float));
    if (st != MGK_OK) return st;
    hipError_t e = mgk_launch_normalize(K_dev, (float*)ctx->diag.p, n, static_cast<hipStream_t>(stream_));
    if (e != hipSuccess) return fail(ctx, MGK_EDEVICE, "normalize launch failed: %s", hipGetErrorString(e));
    return MGK_OK;
}

}  // extern "C"
