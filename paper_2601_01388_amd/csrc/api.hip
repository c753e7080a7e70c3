// C-ABI entry points of the AGIS library (declared in include/agis.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "agis.h"
#include "agis_internal.h"

using agis::DevPlan;
using agis::Partial;

// Fixed device workspace of agis_estimate_noalloc (for callers that cannot
// allocate): every buffer of such a call is carved from it.  Each GPU the
// library runs on holds its own copy until the process ends.  In host code
// the name is not a device address: its address on a device comes from
// hipGetSymbolAddress (kept per device in noalloc_scratch_ptr below).
constexpr uint64_t kNoAllocBytes = 256ull << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace agis {

hipError_t DevPool::alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> lk(mu_);
    *p = nullptr;
    if (bytes >= kPoolMin) {
        // the smallest kept buffer that holds it with at most a quarter to spare
        size_t best = idle_.size();
        for (size_t i = 0; i < idle_.size(); ++i)
            if (idle_[i].bytes >= bytes && idle_[i].bytes - bytes <= bytes / 4 &&
                (best == idle_.size() || idle_[i].bytes < idle_[best].bytes))
                best = i;
        if (best < idle_.size()) {
            const Buf b = idle_[best];
            idle_.erase(idle_.begin() + (std::ptrdiff_t)best);
            idle_bytes_ -= b.bytes;
            track_locked(b.p, b.bytes);
            *p = b.p;
            return hipSuccess;
        }
    }
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && !idle_.empty()) {
        (void)hipGetLastError();
        trim_locked();
        e = hipMalloc(p, bytes);
    }
    if (e == hipSuccess && bytes >= kPoolMin) track_locked(*p, bytes);
    return e;
}

// Notes a buffer handed out (one that cannot be noted is not kept later).
void DevPool::track_locked(void* p, size_t bytes) noexcept {
    try {
        live_[p] = bytes;
    } catch (...) {
    }
}

// Whether kept buffers leave the device enough free memory (on the pool's
// device, whichever the calling thread has current).
bool DevPool::room_locked() {
    int cur = device_;
    (void)hipGetDevice(&cur);
    if (cur != device_) (void)hipSetDevice(device_);
    size_t free_b = 0, total_b = 0;
    const bool room = hipMemGetInfo(&free_b, &total_b) == hipSuccess && free_b >= kPoolFreeFloor;
    if (cur != device_) (void)hipSetDevice(cur);
    unasked_ = 0;
    asked_ = std::chrono::steady_clock::now();
    return room;
}

void DevPool::free(void* p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(mu_);
    const auto it = live_.find(p);
    const size_t bytes = it == live_.end() ? 0 : it->second;
    if (it != live_.end()) live_.erase(it);
    bool keep = open_ && bytes >= kPoolMin && bytes <= kPoolBudget;
    if (keep && unasked_ + bytes > kPoolUnasked && !room_locked()) {
        trim_locked();
        keep = false;
    }
    if (!keep) {
        (void)hipFree(p);
        return;
    }
    while (idle_bytes_ + bytes > kPoolBudget) {
        (void)hipFree(idle_.front().p);
        idle_bytes_ -= idle_.front().bytes;
        idle_.erase(idle_.begin());
    }
    try {
        idle_.push_back(Buf{p, bytes});
    } catch (...) {  // (called from destructors)
        (void)hipFree(p);
        return;
    }
    idle_bytes_ += bytes;
    unasked_ += bytes;
}

void DevPool::check() {
    std::lock_guard<std::mutex> lk(mu_);
    if (idle_bytes_ <= kPoolUnasked) return;
    if (std::chrono::steady_clock::now() - asked_ < std::chrono::milliseconds(1)) return;
    if (!room_locked()) trim_locked();
}

void DevPool::trim_locked() {
    for (const Buf& b : idle_) (void)hipFree(b.p);
    idle_.clear();
    idle_bytes_ = 0;
    unasked_ = 0;
}

void DevPool::trim() {
    std::lock_guard<std::mutex> lk(mu_);
    trim_locked();
}

void DevPool::close() {
    std::lock_guard<std::mutex> lk(mu_);
    open_ = false;
    trim_locked();
}

size_t DevPool::kept() {
    std::lock_guard<std::mutex> lk(mu_);
    return idle_bytes_;
}

int host_oom(agis_ctx* ctx) noexcept {
    if (ctx) ctx->err.assign("host allocation");  // (fits a string's own storage)
    return AGIS_E_OOM;
}

hipError_t ctx_malloc(agis_ctx* ctx, void** p, size_t bytes) {
    *p = nullptr;
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && ctx->pool->kept()) {
        (void)hipGetLastError();
        ctx->pool->trim();
        e = hipMalloc(p, bytes);
    }
    return e;
}

}  // namespace agis

namespace {

// Ends all work on a device before buffers that it may still read (through
// pointers a caller exported, on any stream) go back to a pool.
void sync_device(int device) {
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess || hipSetDevice(device) != hipSuccess) return;
    (void)hipDeviceSynchronize();
    if (cur != device) (void)hipSetDevice(cur);
}

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mutex;
void* g_noalloc_ptr[kMaxDevices] = {};

// The device address of this device's fixed workspace, looked up once per
// device with that device current.
hipError_t noalloc_scratch_ptr(int device, void** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    if (!g_noalloc_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_noalloc_ptr[device] = p;
    }
    *out = g_noalloc_ptr[device];
    return hipSuccess;
}

int fail(agis_ctx* ctx, int code, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return code;
}

int hip_fail(agis_ctx* ctx, hipError_t e, const char* what) {
    const int code = (e == hipErrorOutOfMemory) ? AGIS_E_OOM : AGIS_E_HIP;
    return fail(ctx, code, std::string(what) + ": " + hipGetErrorString(e));
}

#define AGIS_HIP(ctx, expr, what)                     \
    do {                                              \
        hipError_t e_ = (expr);                       \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, what); \
    } while (0)

// Standard normal quantile: Abramowitz-Stegun 26.2.23 start, refined by
// Newton steps on Phi(z) = erfc(-z / sqrt 2) / 2.
double normal_quantile(double p) {
    if (p <= 0.0) return -INFINITY;
    if (p >= 1.0) return INFINITY;
    const double q = p < 0.5 ? p : 1.0 - p;
    const double t = std::sqrt(-2.0 * std::log(q));
    double z = t - (2.515517 + 0.802853 * t + 0.010328 * t * t) / (1.0 + 1.432788 * t + 0.189269 * t * t +
                                                                     0.001308 * t * t * t);
    if (p < 0.5) z = -z;
    for (int it = 0; it < 6; ++it) {
        const double cdf = 0.5 * std::erfc(-z / std::sqrt(2.0));
        const double pdf = std::exp(-0.5 * z * z) / std::sqrt(2.0 * M_PI);
        z -= (cdf - p) / pdf;
    }
    return z;
}

struct Acc {
    double n = 0, mean = 0, m2 = 0, nonzero = 0;
    void merge(const Partial& b) {
        if (b.n == 0.0) return;
        if (n == 0.0) {
            n = b.n;
            mean = b.mean;
            m2 = b.m2;
            nonzero = b.nonzero;
            return;
        }
        const double tot = n + b.n;
        const double delta = b.mean - mean;
        mean = mean + delta * (b.n / tot);
        m2 = m2 + b.m2 + delta * delta * (n * b.n / tot);
        n = tot;
        nonzero += b.nonzero;
    }
};

double eps_hat_of(const Acc& a, double z) {
    if (a.n == 0.0 || a.mean == 0.0) return INFINITY;
    const double sigma = std::sqrt(a.m2 > 0 ? a.m2 / a.n : 0.0);
    return z * sigma / (std::sqrt(a.n) * std::fabs(a.mean));
}

agis_run_params default_params() {
    agis_run_params p;
    std::memset(&p, 0, sizeof(p));
    p.mode = AGIS_MODE_SWITCH;
    p.beta_num = 4;
    p.beta_den = 5;
    p.delta = 0.05;
    return p;
}

// Everything an estimate or dump needs, prepared on the device.
struct Prepared {
    agis_plan plan;
    DevPlan hp;
    double scale = 1.0;  // embeddings per unit of the sample mean (k! on an oriented graph)
    uint32_t* q1 = nullptr;
    uint64_t* pre = nullptr;
    uint32_t* guide = nullptr;
    double tables_seconds = 0;
    bool owns = true;  // false: the buffers are carved from a fixed workspace
    agis_ctx* ctx = nullptr;
    ~Prepared() {
        if (!owns || !ctx || (!q1 && !pre && !guide)) return;
        (void)hipStreamSynchronize(ctx->stream);
        ctx->pool->free(q1);
        ctx->pool->free(pre);
        ctx->pool->free(guide);
    }
};

// Proposal tables of f_approx kept with the graph's tables across calls:
// the per-vertex step weights, the per-row pick tables and the first-step
// table depend only on the vertex records and the step's signature (b, f1,
// ie, f2), so the next estimate of the same signature reuses them.  (Tables
// built from a caller's learned weights are not kept: the caller may change
// them between calls.)  Entries in use by a running call are never evicted;
// others go least recently used first when a new one would pass the budget
// or an allocation fails.  One lock serialises the calls that prepare
// tables of one graph.
}  // namespace

enum CacheKind : uint32_t { kCacheStepWeights = 0, kCacheRowPick = 1, kCacheFirstStep = 2, kCacheCorePick = 3 };
struct CacheEntry {
    uint32_t kind = 0, b = 0, f1 = 0, ie = 0, f2 = 0, blocked = 0;
    void* buf[3] = {nullptr, nullptr, nullptr};
    uint64_t bytes = 0;
    // first step: total weight, guide shift, largest log weight (blocked)
    uint64_t total = 0;
    uint32_t shift = 0;
    int32_t lmax = 0;
    uint64_t stamp = 0;  // last use
    uint32_t users = 0;  // calls holding the entry
};
constexpr uint64_t kTableCacheBudget = 16ull << 30;
// below this much free device memory a call first frees the unused tables
constexpr uint64_t kTableCacheFreeFloor = 128ull << 30;

struct TableCache {
    std::mutex mu;
    std::vector<CacheEntry*> v;
    uint64_t bytes = 0, clock = 0;
    uint32_t* long_rows = nullptr;  // scratch of the row-table builds (2n + 2 entries)
    std::shared_ptr<agis::DevPool> pool;
    ~TableCache() {
        for (CacheEntry* e : v) {
            for (void* b : e->buf) pool->free(b);
            delete e;
        }
        pool->free(long_rows);
    }
    CacheEntry* find(uint32_t kind, uint32_t b, uint32_t f1, uint32_t ie, uint32_t f2, uint32_t blocked) {
        for (CacheEntry* e : v)
            if (e->kind == kind && e->b == b && e->f1 == f1 && e->ie == ie && e->f2 == f2 && e->blocked == blocked) {
                e->stamp = ++clock;
                ++e->users;
                return e;
            }
        return nullptr;
    }
    // frees unused entries, least recently used first, until `need` more
    // bytes fit in the budget (all unused entries when need is ~0)
    void evict(uint64_t need) {
        for (;;) {
            if (need != ~0ull && bytes + need <= kTableCacheBudget) return;
            CacheEntry* victim = nullptr;
            for (CacheEntry* e : v)
                if (e->users == 0 && (!victim || e->stamp < victim->stamp)) victim = e;
            if (!victim) return;
            for (void* b : victim->buf) pool->free(b);
            bytes -= victim->bytes;
            v.erase(std::find(v.begin(), v.end(), victim));
            delete victim;
        }
    }
    // device memory for a new entry (evicting for room first, and once more
    // after a failed allocation); nullptr when it does not fit
    void* alloc(uint64_t nbytes) {
        evict(nbytes);
        void* p = nullptr;
        if (pool->alloc(&p, nbytes) == hipSuccess) return p;
        (void)hipGetLastError();
        evict(~0ull);
        pool->trim();
        if (pool->alloc(&p, nbytes) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    // takes ownership of the buffers of a built entry, held by the caller
    CacheEntry* add(const CacheEntry& proto) {
        CacheEntry* e = new CacheEntry(proto);
        e->stamp = ++clock;
        e->users = 1;
        v.push_back(e);
        bytes += e->bytes;
        return e;
    }
};

namespace {

// Tables shared by the patterns of one call, one per (b, f1, ie, f2,
// learned table):
//  - per-vertex log weights of the weighted steps that build candidate
//    sets: a candidate's weight is then one 4-byte read instead of a 16-byte
//    record and the arithmetic (steps beyond the budget use the records);
//  - per-row pick tables of the weighted steps with one backward vertex.
struct StepTables {
    struct Entry {
        uint32_t b, f1, ie, f2;
        const int32_t* lt;
        int32_t* buf;
        bool cached;  // owned by the graph's table cache
    };
    struct RowEntry {
        uint32_t b, f1, ie, f2;
        const int32_t* lt;
        uint64_t* buf;
        bool cached;
    };
    std::vector<Entry> e;
    std::vector<RowEntry> rows;
    uint32_t* long_rows = nullptr;  // scratch of the row-table build (lists of longer rows)
    agis::Arena* arena = nullptr;   // non-null: buffers are carved from it, never allocated or freed
    TableCache* cache = nullptr;    // the graph's cache (set by prepare; none with an arena)
    std::vector<CacheEntry*> held;  // cache entries this call uses
    agis_ctx* ctx = nullptr;        // set by prepare
    StepTables() = default;
    StepTables(const StepTables&) = delete;
    StepTables& operator=(const StepTables&) = delete;
    ~StepTables() {
        if (cache) {
            std::lock_guard<std::mutex> lk(cache->mu);
            for (CacheEntry* c : held) --c->users;
        }
        if (arena || !ctx) return;
        bool waited = false;
        auto give_back = [&](void* b) {  // a table of this call alone
            if (!waited) (void)hipStreamSynchronize(ctx->stream);
            waited = true;
            ctx->pool->free(b);
        };
        for (Entry& x : e)
            if (!x.cached) give_back(x.buf);
        for (RowEntry& x : rows)
            if (!x.cached) give_back(x.buf);
        if (long_rows && !cache) give_back(long_rows);
    }
};
constexpr uint64_t kStepTableBudgetBytes = 16ull << 30;

// Per-row pick tables are built for runs of at least this many samples
// (AUTO): their build streams every CSR slot once, which a short run does
// not amortise.
constexpr uint64_t kRowtabMinSamples = 65536;
// First-step tables above this size (12 bytes per vertex) are built blocked
// unless the run asks for the full table.
constexpr uint64_t kStep1FullBudget = 2ull << 30;
constexpr uint64_t kRowtabBudgetBytes = 48ull << 30;

// Neighbourhood bitmaps of the highest-degree vertices (degree >= 64, as
// many as fit in kHubBitmapBudget, the degree threshold a power of two):
// the sampler tests membership in such a list with one probe.
constexpr uint64_t kHubBitmapBudget = 1ull << 30;
// Common-neighbour counts of every pair among the highest-degree hubs: a
// uniform last step whose candidates are the common neighbours of two such
// hubs only counts them, so the count is one table read.  The pair hubs are
// those of degree >= 2^p for the smallest p with at most kPairHubs of them
// (counts and running counts at eighths, H^2 x kPairParts x 4 B: at most
// 2 GiB) and at most kPairWork elements over the shorter lists of all pairs
// (R-MAT-20: 6,196 hubs; counting takes 2 ms there, 148 ms when each pair's
// shorter list was walked.  The bound stands as it was set for the walks:
// which hubs have a table decides which paths the samples of larger graphs
// take, and the table's size).
constexpr uint64_t kPairHubs = 8192;
constexpr double kPairWork = 6.0e10;

// Core-pair lists: the common neighbours of every pair among the
// highest-degree pair hubs, so that a candidate set over two such hubs is
// read as one list instead of walking one hub's list against the other's
// bitmap.  The core is the top C pair hubs by (degree, id) for the largest C
// (at most kCoreMax) whose lists, sized from the pair-count table, fit in
// kCorePairBudget and in an eighth of the free memory.  A graph without
// room for them samples without them (the samples are the same).
constexpr uint64_t kCorePairBudget = 4ull << 30;
constexpr uint64_t kCoreMax = 4096;

hipError_t build_core_pairs(agis_ctx* ctx, const agis_graph* g, agis_tables* t, const uint32_t* pair_hub,
                            uint64_t H) {
    const uint64_t n = g->g.n;
    const uint64_t most = std::min<uint64_t>(H, kCoreMax);
    std::vector<uint64_t> rows(most), start;
    start.reserve(most);
    uint64_t* d_rows = nullptr;
    hipError_t e = ctx->pool->alloc(&d_rows, most * sizeof(uint64_t));
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        return hipSuccess;
    }
    if (e == hipSuccess) e = agis::launch_core_rows(ctx, t->pair_count, H, most, d_rows);
    if (e == hipSuccess)
        e = hipMemcpyAsync(rows.data(), d_rows, most * sizeof(uint64_t), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        ctx->pool->free(d_rows);
        return e;
    }
    uint64_t budget = kCorePairBudget;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) == hipSuccess) budget = std::min<uint64_t>(budget, (uint64_t)free_b / 8);
    // every pair's list starts on a block of agis::kCoreBlock entries (the
    // pick tables over the lists keep one prefix per block)
    uint64_t total = 0;
    for (uint64_t c = 0; c < most; ++c) {
        const uint64_t index_bytes = (c + 1) * (c + 1) * (sizeof(uint64_t) + sizeof(uint32_t));
        if ((total + rows[c]) * sizeof(uint32_t) + index_bytes > budget) break;
        start.push_back(total);
        total += rows[c];
    }
    const uint64_t C = start.size();
    if (C < 2) {
        ctx->pool->free(d_rows);
        return hipSuccess;
    }
    t->core_entries = total;
    e = ctx->pool->alloc(&t->core_slot, n * sizeof(int32_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->core_start, C * C * sizeof(uint64_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->core_len, C * C * sizeof(uint32_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->core_nbr, std::max<uint64_t>(total, 1) * sizeof(uint32_t));
    if (e == hipSuccess) e = agis::launch_fill_u32((uint32_t*)t->core_slot, n, 0xFFFFFFFFu, ctx->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(d_rows, start.data(), C * sizeof(uint64_t), hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess)
        e = agis::launch_core_pairs(ctx, g->g, g->max_deg, pair_hub, H, t->pair_count, t->pair_quart, C, d_rows,
                                    t->core_slot, t->core_start, t->core_len, t->core_nbr);
    (void)hipStreamSynchronize(ctx->stream);
    ctx->pool->free(d_rows);
    if (e == hipSuccess) {
        t->cores = C;
        return hipSuccess;
    }
    // no room (or a failed build): sample without the core lists
    for (void* q : {(void*)t->core_slot, (void*)t->core_start, (void*)t->core_len, (void*)t->core_nbr})
        ctx->pool->free(q);
    t->core_slot = nullptr;
    t->core_start = nullptr;
    t->core_len = nullptr;
    t->core_nbr = nullptr;
    t->cores = 0;
    t->core_entries = 0;
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        return hipSuccess;
    }
    return e;
}

hipError_t build_hub_bitmaps(agis_ctx* ctx, const agis_graph* g, agis_tables* t) {
    const uint64_t n = g->g.n;
    const uint64_t words = (n + 31) / 32;
    const uint64_t max_hubs = kHubBitmapBudget / (words * sizeof(uint32_t));
    if (n == 0 || max_hubs == 0) return hipSuccess;
    uint32_t* d_hist = (uint32_t*)ctx->d_small;
    uint32_t hist[64];
    hipError_t e = agis::launch_degree_histogram(g->g, d_hist, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(hist, d_hist, sizeof(hist), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return e;
    int b = 6;
    for (;; ++b) {
        uint64_t c = 0;
        for (int j = b; j < 64; ++j) c += hist[j];
        if (c <= max_hubs || b == 63) break;
    }
    uint64_t above = 0;
    for (int j = b; j < 64; ++j) above += hist[j];
    if (above == 0) return hipSuccess;
    // Both aids are optional: where device memory runs short they are left
    // out (the sampler then merges lists) instead of failing the tables.
    uint32_t* flags = nullptr;
    uint64_t* prefix = nullptr;
    auto drop_out_of_memory = [&]() {
        (void)hipGetLastError();
        for (void* q : {(void*)flags, (void*)prefix, (void*)t->hub_slot, (void*)t->hub_bits, (void*)t->pair_slot,
                        (void*)t->pair_count, (void*)t->pair_quart})
            ctx->pool->free(q);
        t->hub_slot = nullptr;
        t->hub_bits = nullptr;
        t->pair_slot = nullptr;
        t->pair_count = nullptr;
        t->pair_quart = nullptr;
        t->hub_words = t->hubs = t->pairs = 0;
        return hipSuccess;
    };
    e = ctx->pool->alloc(&flags, n * sizeof(uint32_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&prefix, (n + 1) * sizeof(uint64_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->hub_slot, n * sizeof(int32_t));
    if (e == hipSuccess) e = agis::launch_hub_slots(ctx, g->g, 1u << b, flags, t->hub_slot, prefix);
    const uint64_t hubs = above;
    if (e == hipSuccess) e = ctx->pool->alloc(&t->hub_bits, hubs * words * sizeof(uint32_t));
    if (e == hipErrorOutOfMemory) return drop_out_of_memory();
    if (e == hipSuccess) e = hipMemsetAsync(t->hub_bits, 0, hubs * words * sizeof(uint32_t), ctx->stream);
    // (flags is free again: it takes the hubs by slot)
    if (e == hipSuccess) e = agis::launch_hub_bits(ctx, g->g, g->max_deg, t->hub_slot, hubs, flags, words, t->hub_bits);
    if (e == hipSuccess) {
        t->hub_words = words;
        t->hubs = hubs;
        t->hub_min_degree = 1u << b;
    }
    // pair hubs: the hubs of degree >= 2^p, p >= b the smallest within both
    // limits; the work bound takes every degree of bucket j as 2^(j+1) and
    // the hubs in decreasing degree (a pair costs the later one's degree)
    int pb = b;
    for (;; ++pb) {
        uint64_t c = 0;
        double work = 0.0;
        for (int j = 63; j >= pb; --j) {
            work += (double)hist[j] * ((double)c + 0.5 * (double)hist[j]) * std::ldexp(1.0, j + 1);
            c += hist[j];
        }
        if ((c <= kPairHubs && work <= kPairWork) || pb == 63) break;
    }
    uint64_t H = 0;
    uint32_t* pair_hub = nullptr;
    if (e == hipSuccess) {
        e = ctx->pool->alloc(&t->pair_slot, n * sizeof(int32_t));
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            t->pair_slot = nullptr;
            e = hipSuccess;
            ctx->pool->free(flags);
            ctx->pool->free(prefix);
            return e;  // bitmaps without the pair-hub table
        }
    }
    if (e == hipSuccess) e = agis::launch_hub_slots(ctx, g->g, 1u << pb, flags, t->pair_slot, prefix);
    for (int j = pb; j < 64; ++j) H += hist[j];
    if (e == hipSuccess && H >= 2) {
        e = ctx->pool->alloc(&pair_hub, H * sizeof(uint32_t));
        if (e == hipSuccess) e = ctx->pool->alloc(&t->pair_count, H * H * sizeof(uint32_t));
        if (e == hipSuccess) e = ctx->pool->alloc(&t->pair_quart, H * H * (agis::kPairParts - 1) * sizeof(uint32_t));
        if (e == hipSuccess)
            e = agis::launch_pair_counts(ctx, g->g, g->max_deg, t->pair_slot, H, pair_hub, t->pair_count,
                                         t->pair_quart);
        if (e == hipErrorOutOfMemory) {
            // no room for the pair-hub table: keep the bitmaps without it
            (void)hipGetLastError();
            ctx->pool->free(t->pair_count);
            ctx->pool->free(t->pair_quart);
            t->pair_count = nullptr;
            t->pair_quart = nullptr;
            H = 0;
            e = hipSuccess;
        }
        if (e == hipSuccess) {
            t->pairs = H;
            t->pair_min_degree = 1u << pb;
        }
        if (e == hipSuccess && t->pair_count) e = build_core_pairs(ctx, g, t, pair_hub, H);
    }
    ctx->pool->free(pair_hub);
    ctx->pool->free(flags);
    ctx->pool->free(prefix);
    return e;
}

agis::DevTables dev_tables(const agis_tables* t) {
    return agis::DevTables{agis::gmem((const uint4*)t->rec),        agis::gmem((const uint32_t*)t->hub_bits),
                           agis::gmem((const int32_t*)t->hub_slot),    t->hub_words,
                           agis::gmem((const int32_t*)t->pair_slot),   agis::gmem((const uint32_t*)t->pair_count),
                           t->pair_count ? t->pairs : 0,               agis::gmem((const uint32_t*)t->pair_quart),
                           agis::gmem((const int32_t*)t->core_slot),   agis::gmem((const uint64_t*)t->core_start),
                           agis::gmem((const uint32_t*)t->core_len),   agis::gmem((const uint32_t*)t->core_nbr),
                           t->cores};
}

// Device memory for a proposal table: from the cache (keep) or the call.
// The sampler's scratch that the context keeps between calls is idle while
// tables are prepared (the sampler sizes it again from the memory then
// free), so a failed allocation releases it and tries once more.
void* table_alloc(agis_ctx* ctx, TableCache* cache, bool keep, uint64_t nbytes) {
    for (int attempt = 0; attempt < 2; ++attempt) {
        void* p = nullptr;
        if (keep) {
            p = cache->alloc(nbytes);
            if (p) return p;
        } else {
            if (ctx->pool->alloc(&p, nbytes) == hipSuccess) return p;
            (void)hipGetLastError();
        }
        if (attempt > 0 || !ctx->d_scratch) break;
        (void)hipFree(ctx->d_scratch);
        ctx->d_scratch = nullptr;
        ctx->scratch_bytes = 0;
    }
    return nullptr;
}

int prepare(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p, const uint8_t* order,
            const agis_run_params* params, uint64_t n_samples, StepTables* st, Prepared* out) {
    int rc = agis::compile_plan(p, order, params->mode, params->beta_num, params->beta_den, &out->plan, &ctx->err);
    if (rc != AGIS_OK) return rc;
    // On a degree-oriented graph (agis_orient) a k-clique is found exactly
    // once, as the increasing sequence of its vertices: only cliques are
    // sampled there, the weights count the later vertices among the out-
    // neighbours (no backward vertex is an out-neighbour: |B| enters as 0),
    // and the mean counts cliques, k! embeddings each.
    const bool oriented = g->parent != nullptr;
    out->scale = 1.0;
    if (oriented) {
        for (uint32_t u = 0; u < p->k; ++u)
            if (p->adj[u] != (uint8_t)(((1u << p->k) - 1u) & ~(1u << u)))
                return fail(ctx, AGIS_E_UNSUPPORTED, "an oriented graph samples clique patterns only");
        for (uint32_t j = 2; j <= p->k; ++j) out->scale *= (double)j;
    }
    const uint32_t rowtab = params->flags & 3u;
    const uint32_t step1 = params->flags & (AGIS_RUN_STEP1_BLOCKS | AGIS_RUN_STEP1_FULL);
    if (rowtab > AGIS_RUN_ROWTAB_OFF ||
        (params->flags & ~(3u | AGIS_RUN_STEP1_BLOCKS | AGIS_RUN_STEP1_FULL | AGIS_RUN_HOST_ROUNDS | AGIS_RUN_WAVE_SAMPLES)) ||
        step1 == (AGIS_RUN_STEP1_BLOCKS | AGIS_RUN_STEP1_FULL))
        return fail(ctx, AGIS_E_INVALID_ARG, "unknown run flag");
    if (params->terms > AGIS_TERMS_F1_I1) return fail(ctx, AGIS_E_INVALID_ARG, "unknown term set");
    st->ctx = out->ctx = ctx;
    DevPlan& hp = out->hp;
    std::memset(&hp, 0, sizeof(hp));
    hp.k = out->plan.k;
    hp.pattern_id = params->pattern_id;
    for (uint32_t i = 0; i < hp.k; ++i) {
        hp.bmask[i] = out->plan.bmask[i];
        hp.b[i] = oriented ? 0 : out->plan.b[i];
        hp.f1[i] = out->plan.f1[i];
        // the term ablation drops T[I1] (exponent ie) and T[F2] (exponent f2)
        hp.ie[i] = params->terms == AGIS_TERMS_F1 ? 0 : out->plan.ie[i];
        hp.f2[i] = params->terms == AGIS_TERMS_ALL ? out->plan.f2[i] : 0;
        // |F1| = 0 makes every weight C(d - b, 0) = 1: a uniform draw.
        hp.weighted[i] = (out->plan.decision[i] && out->plan.f1[i] > 0) ? 1 : 0;
        if (params->mode == AGIS_MODE_LEARNED && hp.weighted[i]) {
            if (!params->learned[i]) return fail(ctx, AGIS_E_INVALID_ARG, "learned mode needs a table for every weighted step");
            hp.lt[i] = agis::gmem(params->learned[i]);
        }
    }
    const auto t0 = std::chrono::steady_clock::now();
    // the graph's table cache (not with a fixed workspace), locked until the
    // tables of this pattern are built
    TableCache* cache = (!st->arena && t->cache) ? t->cache : nullptr;
    std::unique_lock<std::mutex> cache_lock;
    if (cache) {
        cache_lock = std::unique_lock<std::mutex>(cache->mu);
        st->cache = cache;
        // when device memory is scarce (a graph of a large part of the GPU),
        // the memory of kept tables goes back to this call's tables and the
        // sampler's scratch, whose size sets the number of waves
        size_t free_b = 0, total_b = 0;
        if ((cache->bytes || ctx->pool->kept()) && hipMemGetInfo(&free_b, &total_b) == hipSuccess &&
            free_b < kTableCacheFreeFloor) {
            cache->evict(~0ull);
            ctx->pool->trim();
        }
    }
    // per-vertex log weights of step i (shared by the call), nullptr beyond
    // the budget
    int step_rc = AGIS_OK;
    auto step_table = [&](uint32_t i) -> const int32_t* {
        for (const StepTables::Entry& e : st->e)
            if (e.b == hp.b[i] && e.f1 == hp.f1[i] && e.ie == hp.ie[i] && e.f2 == hp.f2[i] && e.lt == hp.lt[i])
                return e.buf;
        const bool keep = cache && hp.lt[i] == nullptr;
        if (keep) {
            if (CacheEntry* c = cache->find(kCacheStepWeights, hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], 0)) {
                st->held.push_back(c);
                st->e.push_back(StepTables::Entry{hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], nullptr, (int32_t*)c->buf[0], true});
                return (const int32_t*)c->buf[0];
            }
        }
        if ((st->e.size() + 1) * g->g.n * sizeof(int32_t) > kStepTableBudgetBytes) return nullptr;
        const uint64_t nbytes = g->g.n * sizeof(int32_t);
        int32_t* buf = nullptr;
        hipError_t e = hipSuccess;
        if (st->arena) {
            // no room left in the fixed workspace: the weights come from the records
            buf = (int32_t*)st->arena->take(nbytes);
            if (!buf) return nullptr;
        } else {
            buf = (int32_t*)table_alloc(ctx, cache, keep, nbytes);
            if (!buf) e = hipErrorOutOfMemory;
        }
        if (e == hipSuccess)
            e = agis::launch_step_log_weights(*t, g->g.n, hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], hp.lt[i], buf,
                                              ctx->stream);
        if (e != hipSuccess) {
            if (buf && !st->arena) ctx->pool->free(buf);
            step_rc = fail(ctx, e == hipErrorOutOfMemory ? AGIS_E_OOM : AGIS_E_HIP,
                           std::string("step weight table: ") + hipGetErrorString(e));
            return nullptr;
        }
        st->e.push_back(StepTables::Entry{hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], hp.lt[i], buf, keep});
        if (keep) {
            CacheEntry proto;
            proto.kind = kCacheStepWeights;
            proto.b = hp.b[i];
            proto.f1 = hp.f1[i];
            proto.ie = hp.ie[i];
            proto.f2 = hp.f2[i];
            proto.buf[0] = buf;
            proto.bytes = nbytes;
            st->held.push_back(cache->add(proto));
        }
        return buf;
    };
    // per-row pick tables for weighted steps with one backward vertex
    // (never with a fixed workspace: a row table takes 8 bytes per CSR slot)
    bool want_rows = !st->arena && (rowtab == AGIS_RUN_ROWTAB_ON ||
                                    (rowtab == AGIS_RUN_ROWTAB_AUTO && n_samples >= kRowtabMinSamples));
    if (want_rows && g->g.nnz > 0) {
        for (uint32_t i = 1; i < hp.k; ++i) {
            if (!hp.weighted[i] || __builtin_popcount(hp.bmask[i]) != 1) continue;
            const int32_t* lt = (const int32_t*)hp.lt[i];
            const bool keep = cache && lt == nullptr;
            uint64_t* buf = nullptr;
            for (const StepTables::RowEntry& r : st->rows)
                if (r.b == hp.b[i] && r.f1 == hp.f1[i] && r.ie == hp.ie[i] && r.f2 == hp.f2[i] && r.lt == lt)
                    buf = r.buf;
            if (!buf && keep) {
                if (CacheEntry* c = cache->find(kCacheRowPick, hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], 0)) {
                    st->held.push_back(c);
                    buf = (uint64_t*)c->buf[0];
                    st->rows.push_back(StepTables::RowEntry{hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], nullptr, buf, true});
                }
            }
            if (!buf) {
                if ((st->rows.size() + 1) * g->g.nnz * sizeof(uint64_t) > kRowtabBudgetBytes) continue;
                const int32_t* sw = step_table(i);
                if (step_rc != AGIS_OK) return step_rc;
                if (!sw) continue;
                const uint64_t lbytes = (2 * g->g.n + 2) * sizeof(uint32_t);
                if (cache) {
                    if (!cache->long_rows)
                        AGIS_HIP(ctx, ctx->pool->alloc(&cache->long_rows, lbytes), "allocate row lists");
                    st->long_rows = cache->long_rows;
                } else if (!st->long_rows) {
                    AGIS_HIP(ctx, ctx->pool->alloc(&st->long_rows, lbytes), "allocate row lists");
                }
                const uint64_t nbytes = g->g.nnz * sizeof(uint64_t);
                buf = (uint64_t*)table_alloc(ctx, cache, keep, nbytes);
                if (!buf) return fail(ctx, AGIS_E_OOM, "allocate row pick table: out of device memory");
                const hipError_t e = agis::launch_rowtab(ctx, g->g, sw, buf, st->long_rows);
                if (e != hipSuccess) {
                    ctx->pool->free(buf);
                    return hip_fail(ctx, e, "row pick table");
                }
                st->rows.push_back(StepTables::RowEntry{hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], lt, buf, keep});
                if (keep) {
                    CacheEntry proto;
                    proto.kind = kCacheRowPick;
                    proto.b = hp.b[i];
                    proto.f1 = hp.f1[i];
                    proto.ie = hp.ie[i];
                    proto.f2 = hp.f2[i];
                    proto.buf[0] = buf;
                    proto.bytes = nbytes;
                    st->held.push_back(cache->add(proto));
                }
            }
            hp.rowpre[i] = agis::gmem((const uint64_t*)buf);
        }
    }
    // A step builds its candidate set in the wave's scratch unless it draws
    // uniformly from one backward list or through a row table.  When step
    // i-1 did and its backward set is contained in step i's, step i starts
    // from that set.
    auto general = [&](uint32_t i) {
        return (hp.weighted[i] && hp.rowpre[i] == nullptr) || __builtin_popcount(hp.bmask[i]) > 1;
    };
    for (uint32_t i = 2; i < hp.k; ++i)
        hp.reuse[i] = (general(i) && general(i - 1) && (hp.bmask[i - 1] & ~hp.bmask[i]) == 0) ? 1 : 0;
    for (uint32_t i = 1; i < hp.k && g->g.n > 0; ++i) {
        if (!hp.weighted[i] || hp.rowpre[i] != nullptr) continue;
        const int32_t* buf = step_table(i);
        if (step_rc != AGIS_OK) return step_rc;
        if (buf) hp.sw[i] = agis::gmem(buf);
    }
    // the pick tables over the core-pair lists of the weighted steps with
    // two backward vertices, one per step signature (built where row tables
    // are and kept in the cache like them; not for learned weights): per
    // list its largest log weight, per block of kCoreBlock entries a prefix
    const uint64_t core_lb = t->cores * t->cores * sizeof(int32_t);
    const uint64_t core_pb = (t->core_entries / agis::kCoreBlock + 1) * sizeof(uint64_t);
    for (uint32_t i = 2; i < hp.k && want_rows && t->cores && cache && core_lb + core_pb <= kRowtabBudgetBytes; ++i) {
        if (!hp.weighted[i] || __builtin_popcount(hp.bmask[i]) != 2 || hp.lt[i] != nullptr || hp.sw[i] == nullptr)
            continue;
        CacheEntry* c = cache->find(kCacheCorePick, hp.b[i], hp.f1[i], hp.ie[i], hp.f2[i], 0);
        if (!c) {
            void* clm = table_alloc(ctx, cache, true, core_lb);
            void* cbp = clm ? table_alloc(ctx, cache, true, core_pb) : nullptr;
            hipError_t e = (clm && cbp) ? agis::launch_core_pick(ctx, *t, (const int32_t*)hp.sw[i], (int32_t*)clm,
                                                                 (uint64_t*)cbp)
                                        : hipErrorOutOfMemory;
            if (e != hipSuccess) {
                ctx->pool->free(clm);
                ctx->pool->free(cbp);
                if (e != hipErrorOutOfMemory) return hip_fail(ctx, e, "core-pair pick table");
                (void)hipGetLastError();  // no room: the step walks the lists
                continue;
            }
            CacheEntry proto;
            proto.kind = kCacheCorePick;
            proto.b = hp.b[i];
            proto.f1 = hp.f1[i];
            proto.ie = hp.ie[i];
            proto.f2 = hp.f2[i];
            proto.buf[0] = clm;
            proto.buf[1] = cbp;
            proto.bytes = core_lb + core_pb;
            c = cache->add(proto);
        }
        st->held.push_back(c);
        hp.clm[i] = agis::gmem((const int32_t*)c->buf[0]);
        hp.cbp[i] = agis::gmem((const uint64_t*)c->buf[1]);
    }
    // the blocked first-step table (8 bytes per kStep1Block vertices instead
    // of 12 per vertex) when asked for, or by default when the full table
    // would exceed kStep1FullBudget
    const bool blocked = step1 == AGIS_RUN_STEP1_BLOCKS ||
                         (step1 == 0 && 12ull * g->g.n > kStep1FullBudget);
    const bool keep1 = cache && hp.weighted[0] && hp.lt[0] == nullptr && g->g.n > 0;
    CacheEntry* c1 = keep1 ? cache->find(kCacheFirstStep, 0, hp.f1[0], hp.ie[0], hp.f2[0], blocked ? 1u : 0u) : nullptr;
    if (c1) {
        st->held.push_back(c1);
        if (blocked) {
            hp.s1_blk = agis::gmem((const uint64_t*)c1->buf[0] + 1);
            hp.s1_lmax = c1->lmax;
        } else {
            hp.s1_q = agis::gmem((const uint32_t*)c1->buf[0]);
            hp.s1_pre = agis::gmem((const uint64_t*)c1->buf[1]);
        }
        hp.s1_total = c1->total;
        if (c1->total > 0) {
            hp.s1_guide = agis::gmem((const uint32_t*)c1->buf[2]);
            hp.s1_shift = c1->shift;
        }
    }
    // a new first-step buffer: from the fixed workspace, the cache or the call
    auto alloc1 = [&](void** p, uint64_t nbytes, const char* what) -> int {
        *p = table_alloc(ctx, cache, keep1, nbytes);
        return *p ? AGIS_OK : fail(ctx, AGIS_E_OOM, std::string(what) + ": out of device memory");
    };
    if (!c1 && hp.weighted[0] && g->g.n > 0 && blocked) {
        const uint64_t nblk = (g->g.n + agis::kStep1Block - 1) / agis::kStep1Block;
        uint64_t* blk = nullptr;
        uint32_t* guide = nullptr;
        if (st->arena) {
            out->owns = false;
            blk = (uint64_t*)st->arena->take((nblk + 1) * sizeof(uint64_t));
            guide = (uint32_t*)st->arena->take(((1ull << agis::kGuideBits) + 1) * sizeof(uint32_t));
            if (!blk || !guide)
                return fail(ctx, AGIS_E_UNSUPPORTED, "the first-step table does not fit in the fixed workspace");
        } else {
            rc = alloc1((void**)&blk, (nblk + 1) * sizeof(uint64_t), "allocate first-step block prefix");
            if (rc != AGIS_OK) return rc;
        }
        if (!keep1) out->pre = blk;  // owned as the prefix buffer
        uint64_t total = 0;
        int32_t lmax = 0;
        uint64_t gbytes = 0;
        hipError_t e = agis::build_step1_blocks(ctx, *g, *t, hp, blk, &lmax, &total);
        hp.s1_blk = agis::gmem((const uint64_t*)(blk + 1));
        hp.s1_lmax = lmax;
        hp.s1_total = total;
        if (e == hipSuccess && total > 0) {
            const uint32_t shift = agis::guide_shift(total);
            const uint64_t buckets = ((total - 1) >> shift) + 1;
            gbytes = (buckets + 1) * sizeof(uint32_t);
            if (!st->arena) {
                rc = alloc1((void**)&guide, gbytes, "allocate first-step guide");
                if (rc != AGIS_OK) {
                    if (keep1) ctx->pool->free(blk);
                    return rc;
                }
            }
            if (!keep1) out->guide = guide;
            e = agis::launch_prefix_guide(blk + 1, nblk, total, shift, guide, ctx->stream);
            hp.s1_guide = agis::gmem((const uint32_t*)guide);
            hp.s1_shift = shift;
        }
        if (e != hipSuccess) {
            if (keep1) {
                ctx->pool->free(blk);
                ctx->pool->free(guide);
            }
            return hip_fail(ctx, e, "first-step block table");
        }
        if (keep1) {
            CacheEntry proto;
            proto.kind = kCacheFirstStep;
            proto.f1 = hp.f1[0];
            proto.ie = hp.ie[0];
            proto.f2 = hp.f2[0];
            proto.blocked = 1;
            proto.buf[0] = blk;
            proto.buf[2] = guide;
            proto.bytes = (nblk + 1) * sizeof(uint64_t) + gbytes;
            proto.total = total;
            proto.shift = hp.s1_shift;
            proto.lmax = lmax;
            st->held.push_back(cache->add(proto));
        }
    }
    if (!c1 && hp.weighted[0] && g->g.n > 0 && !blocked) {
        uint64_t* blocksums = nullptr;
        uint32_t* q1 = nullptr;
        uint64_t* pre = nullptr;
        uint32_t* guide = nullptr;
        if (st->arena) {
            out->owns = false;
            q1 = (uint32_t*)st->arena->take(g->g.n * sizeof(uint32_t));
            pre = (uint64_t*)st->arena->take(g->g.n * sizeof(uint64_t));
            guide = (uint32_t*)st->arena->take(((1ull << agis::kGuideBits) + 1) * sizeof(uint32_t));
            blocksums = (uint64_t*)st->arena->take(agis::step1_scan_tiles(g->g.n) * sizeof(uint64_t));
            if (!q1 || !pre || !guide || !blocksums)
                return fail(ctx, AGIS_E_UNSUPPORTED, "the first-step table does not fit in the fixed workspace");
        } else {
            rc = alloc1((void**)&q1, g->g.n * sizeof(uint32_t), "allocate first-step weights");
            if (rc == AGIS_OK) rc = alloc1((void**)&pre, g->g.n * sizeof(uint64_t), "allocate first-step prefix");
            if (rc != AGIS_OK) {
                ctx->pool->free(q1);
                return rc;
            }
        }
        if (!keep1) {
            out->q1 = q1;
            out->pre = pre;
        }
        uint64_t total = 0;
        uint64_t gbytes = 0;
        hipError_t e = agis::build_step1(ctx, *g, *t, hp, q1, pre, &total, blocksums);
        hp.s1_q = agis::gmem((const uint32_t*)q1);
        hp.s1_pre = agis::gmem((const uint64_t*)pre);
        hp.s1_total = total;
        if (e == hipSuccess && total > 0) {
            const uint32_t shift = agis::guide_shift(total);
            const uint64_t buckets = ((total - 1) >> shift) + 1;
            gbytes = (buckets + 1) * sizeof(uint32_t);
            if (!st->arena) {
                rc = alloc1((void**)&guide, gbytes, "allocate first-step guide");
                if (rc != AGIS_OK) {
                    if (keep1) {
                        ctx->pool->free(q1);
                        ctx->pool->free(pre);
                    }
                    return rc;
                }
            }
            if (!keep1) out->guide = guide;
            e = agis::launch_prefix_guide(pre, g->g.n, total, shift, guide, ctx->stream);
            hp.s1_guide = agis::gmem((const uint32_t*)guide);
            hp.s1_shift = shift;
        }
        if (e != hipSuccess) {
            if (keep1) {
                ctx->pool->free(q1);
                ctx->pool->free(pre);
                ctx->pool->free(guide);
            }
            return hip_fail(ctx, e, "first-step table");
        }
        if (keep1) {
            CacheEntry proto;
            proto.kind = kCacheFirstStep;
            proto.f1 = hp.f1[0];
            proto.ie = hp.ie[0];
            proto.f2 = hp.f2[0];
            proto.buf[0] = q1;
            proto.buf[1] = pre;
            proto.buf[2] = guide;
            proto.bytes = g->g.n * 12ull + gbytes;
            proto.total = total;
            proto.shift = hp.s1_shift;
            st->held.push_back(cache->add(proto));
        }
    }
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "proposal tables");
    out->tables_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return AGIS_OK;
}

// State of one pattern inside a run of rounds.
struct PatternRun {
    Prepared prep;
    uint64_t budget = 0;
    uint64_t done = 0;
    Acc acc;
    bool active = true;
    bool converged = false;
    double seconds = 0;  // from the start of the run until this pattern stopped
    double kernel_seconds = 0;
    uint64_t launches = 0;
};

// Whether a plan has a step the pair-hub paths serve (an unweighted step
// over exactly two backward lists) and the tables have the pair-hub table.
// Whether a launch over these plans runs on the lane sampler.
bool use_lanes(const std::vector<PatternRun>& runs, const agis_run_params* pp) {
    if (pp->flags & AGIS_RUN_WAVE_SAMPLES) return false;
    for (const PatternRun& r : runs)
        if (!agis::lane_plan(r.prep.hp)) return false;
    return !runs.empty();
}

bool uses_pair_hubs(const DevPlan& hp, const agis_tables* t) {
    if (!t->pair_count || t->pairs == 0) return false;
    for (uint32_t i = 2; i < hp.k; ++i)
        if (!hp.weighted[i] && __builtin_popcount(hp.bmask[i]) == 2) return true;
    return false;
}

// Rounds of at most this many samples bound the weight buffer (8 B each).
constexpr uint64_t kMaxRoundSlots = 1ull << 24;
constexpr uint64_t kFixedRoundSlots = 1ull << 20;
static_assert(kFixedRoundSlots % agis::kReduceTileSamples == 0, "round size");

int replay_or_launch(agis_ctx* ctx, const agis::SampleLaunch& L, const agis_graph* g, const agis_tables* t,
                     float* ms, bool direct) {
    if (!ctx->use_graphs || direct) {
        AGIS_HIP(ctx, agis::launch_round(ctx, ctx->stream, L, ctx->ev_start, ctx->ev_stop), "launch round");
        AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "round");
        AGIS_HIP(ctx, hipEventElapsedTime(ms, ctx->ev_start, ctx->ev_stop), "event time");
        return AGIS_OK;
    }
    // kernel arguments and grids of the captured sequence: the descriptor's
    // contents may change between replays, its address and the grids not
    const uint64_t key[8] = {(uint64_t)(uintptr_t)ctx->d_launch, (uint64_t)L.blocks, (uint64_t)L.threads,
                             L.max_tiles, (uint64_t)(uintptr_t)L.partials, (uint64_t)(uintptr_t)ctx->d_small,
                             (uint64_t)L.variant, (uint64_t)L.pairs | ((uint64_t)L.lanes << 1)};
    if (!ctx->graph_exec || std::memcmp(key, ctx->graph_key, sizeof(key)) != 0) {
        if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
        if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
        ctx->graph_exec = nullptr;
        ctx->graph = nullptr;
        AGIS_HIP(ctx, hipStreamBeginCapture(ctx->graph_stream, hipStreamCaptureModeThreadLocal), "begin capture");
        hipError_t e = agis::launch_round(ctx, ctx->graph_stream, L, nullptr, nullptr);
        hipGraph_t gr = nullptr;
        hipError_t e2 = hipStreamEndCapture(ctx->graph_stream, &gr);
        if (e != hipSuccess) return hip_fail(ctx, e, "capture round");
        if (e2 != hipSuccess) return hip_fail(ctx, e2, "end capture");
        ctx->graph = gr;
        AGIS_HIP(ctx, hipGraphInstantiate(&ctx->graph_exec, gr, nullptr, nullptr, 0), "instantiate round graph");
        std::memcpy(ctx->graph_key, key, sizeof(key));
    }
    // order the replay after the caller's stream, and the caller's stream after it
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_in, ctx->stream), "record event");
    AGIS_HIP(ctx, hipStreamWaitEvent(ctx->graph_stream, ctx->ev_in, 0), "wait event");
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_start, ctx->graph_stream), "record event");
    AGIS_HIP(ctx, hipGraphLaunch(ctx->graph_exec, ctx->graph_stream), "replay round graph");
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_stop, ctx->graph_stream), "record event");
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_out, ctx->graph_stream), "record event");
    AGIS_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->ev_out, 0), "wait event");
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "round");
    AGIS_HIP(ctx, hipEventElapsedTime(ms, ctx->ev_start, ctx->ev_stop), "event time");
    return AGIS_OK;
}

// Runs the patterns' samples in rounds.  to_eps: every active pattern gets
// check_every samples per round and stops once Algorithm 1's eps_hat <= eps
// (with at least min_samples) or at its budget; otherwise each pattern runs
// exactly its budget, rounds filled in pattern order.  Samples of a pattern
// use indices 0, 1, 2, ... in order, so the stopping point of each pattern
// depends only on its own samples.
int run_rounds(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, std::vector<PatternRun>& runs,
               const agis_run_params* pp, uint64_t seed, bool* cancelled, agis::Arena* arena = nullptr) {
    *cancelled = false;
    const bool to_eps = pp->eps > 0;
    const uint64_t check = pp->check_every ? pp->check_every : 65536;
    const double z = normal_quantile(1.0 - (to_eps ? pp->delta : 0.05) / 2.0);
    const uint32_t npat = (uint32_t)runs.size();
    std::vector<DevPlan> plans(npat);
    for (uint32_t p = 0; p < npat; ++p) plans[p] = runs[p].prep.hp;
    AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_plans, plans.data(), npat * sizeof(DevPlan), hipMemcpyHostToDevice, ctx->stream),
             "upload plans");
    uint64_t max_slots = 0, total_budget = 0;
    for (const PatternRun& r : runs) {
        total_budget += r.budget;
        max_slots += to_eps ? std::min(check, r.budget) : r.budget;
    }
    // rounds within a fixed workspace hold at most kFixedRoundSlots slots (a
    // multiple of the reduction tile, so the tiles and hence the estimate are
    // the same as with larger rounds)
    max_slots = std::min(max_slots, arena ? kFixedRoundSlots : kMaxRoundSlots);
    if (max_slots == 0) return AGIS_OK;
    agis::SampleLaunch L;
    L.lanes = use_lanes(runs, pp);
    for (const PatternRun& r : runs) L.pairs = L.pairs || (!L.lanes && uses_pair_hubs(r.prep.hp, t));
    int rc = agis::plan_sample_launch(ctx, *g, max_slots, npat, &L, &ctx->err, arena);
    if (rc != AGIS_OK) return rc;
    agis::LaunchDesc ld;
    std::memset(&ld, 0, sizeof(ld));
    agis::fill_launch(ctx, L, g->g, dev_tables(t), nullptr, nullptr, &ld);
    agis::RoundDesc& rd = ld.round;
    std::vector<Partial> parts;
    std::vector<uint32_t> members;
    const auto t0 = std::chrono::steady_clock::now();
    for (;;) {
        if (pp->cancel && *pp->cancel) {
            // stop between rounds: every pattern keeps the whole rounds it
            // finished, a prefix of its sample sequence
            *cancelled = true;
            const double now = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
            for (PatternRun& r : runs)
                if (r.active) {
                    r.active = false;
                    r.seconds = now;
                }
            break;
        }
        std::memset(&rd, 0, sizeof(rd));
        rd.k0 = (uint32_t)seed;
        rd.k1 = (uint32_t)(seed >> 32);
        members.clear();
        uint64_t used = 0, tiles = 0;
        for (uint32_t p = 0; p < npat && used < max_slots; ++p) {
            PatternRun& r = runs[p];
            if (!r.active) continue;
            uint64_t cnt = r.budget - r.done;
            if (to_eps) cnt = std::min(cnt, check);
            cnt = std::min(cnt, max_slots - used);
            if (cnt == 0) continue;
            agis::Segment& S = rd.seg[rd.nseg++];
            S.plan = p;
            S.start = pp->first_sample + r.done;
            S.base = used;
            S.count = cnt;
            S.ntiles = (uint32_t)((cnt + agis::kReduceTileSamples - 1) / agis::kReduceTileSamples);
            S.tile_base = tiles;
            used += cnt;
            tiles += S.ntiles;
            members.push_back(p);
        }
        if (rd.nseg == 0) break;
        rd.total = used;
        AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_launch, &ld, sizeof(ld), hipMemcpyHostToDevice, ctx->stream),
                 "upload round");
        float ms = 0.0f;
        rc = replay_or_launch(ctx, L, g, t, &ms, arena != nullptr);
        if (rc != AGIS_OK) return rc;
        parts.resize((size_t)tiles);
        AGIS_HIP(ctx,
                 hipMemcpyAsync(parts.data(), L.partials, tiles * sizeof(Partial), hipMemcpyDeviceToHost,
                                ctx->stream),
                 "read partials");
        AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "read partials");
        const double now = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        for (uint32_t q = 0; q < rd.nseg; ++q) {
            PatternRun& r = runs[rd.seg[q].plan];
            for (uint32_t k = 0; k < rd.seg[q].ntiles; ++k) r.acc.merge(parts[rd.seg[q].tile_base + k]);
            r.done += rd.seg[q].count;
            r.kernel_seconds += 1e-3 * (double)ms * (double)rd.seg[q].count / (double)used;
            r.launches += 1;
            if (to_eps && r.done >= pp->min_samples && eps_hat_of(r.acc, z) <= pp->eps) {
                r.converged = true;
                r.active = false;
            }
            if (r.done >= r.budget) r.active = false;
            if (!r.active) r.seconds = now;
        }
    }
    (void)total_budget;
    return AGIS_OK;
}

// Offsets in the context's small device buffer of the launch's start clock
// and of the fault flag of a run to epsilon in one launch.
constexpr uint32_t kClockOffset = 520;
// A run to epsilon's later workgroups: time between two looks, the mean time
// of a sample from which they join, and the same in a run that has merged
// kEpsLateMerged samples (see eps_joins).
constexpr int kEpsLookMicroseconds = 40;
constexpr int kEpsJoinMicroseconds = 16;
constexpr int kEpsLateMicroseconds = 4;
constexpr uint64_t kEpsLateMerged = 1ull << 18;
constexpr uint32_t kFaultOffset = 528;

// Runs every pattern to epsilon (or its budget) in one persistent launch
// (k_sample_eps): the checks, merges and stops happen on the device at the
// same check points, over the same reduction tiles, as run_rounds'.  The
// caller's cancel flag is polled while the launch runs and forwarded to a
// pinned host flag that the kernel reads (a copy to device memory could not
// start while the persistent kernel holds the compute units).
int run_device_eps(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, std::vector<PatternRun>& runs,
                   const agis_run_params* pp, uint64_t seed, bool* cancelled) {
    *cancelled = false;
    const uint64_t check = pp->check_every ? pp->check_every : 65536;
    const double z = normal_quantile(1.0 - pp->delta / 2.0);
    const uint32_t npat = (uint32_t)runs.size();
    std::vector<DevPlan> plans(npat);
    uint64_t total = 0;
    for (uint32_t p = 0; p < npat; ++p) {
        plans[p] = runs[p].prep.hp;
        total += runs[p].budget;
    }
    AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_plans, plans.data(), npat * sizeof(DevPlan), hipMemcpyHostToDevice, ctx->stream),
             "upload plans");
    if (total == 0) return AGIS_OK;
    agis::SampleLaunch L;
    L.eps = true;
    for (const PatternRun& r : runs) L.pairs = L.pairs || uses_pair_hubs(r.prep.hp, t);
    int rc = agis::plan_sample_launch(ctx, *g, std::min<uint64_t>(total, kMaxRoundSlots), npat, &L, &ctx->err);
    if (rc != AGIS_OK) return rc;
    // ring: the window of slots ahead of the merged prefix, plus two tiles.
    // A wide window keeps the waves busy while one slow sample holds the
    // oldest tile open (sample costs are heavy-tailed); handing out stays
    // demand-driven, so the samples drawn past a stopping point are about
    // the waves in flight, whatever the window.
    const uint64_t window = std::max<uint64_t>(2 * check, (1ull << 20) - 2 * agis::kEpsTile);
    uint64_t ring = agis::kEpsTile;
    while (ring < window + 2 * agis::kEpsTile) ring <<= 1;
    const uint64_t rtiles = ring / agis::kEpsTile;
    const size_t pat_bytes = npat * sizeof(agis::EpsPattern);
    const size_t ring_bytes = (size_t)npat * ring * sizeof(double);
    const size_t part_bytes = (size_t)npat * rtiles * sizeof(Partial);
    const size_t ready_bytes = (size_t)npat * rtiles * sizeof(unsigned long long);
    const size_t done_bytes = (size_t)npat * rtiles * sizeof(uint32_t);
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    const uint32_t rank_blocks = (uint32_t)std::max(1, ctx->num_cus);
    const size_t rank_bytes = (1 + (size_t)rank_blocks) * sizeof(uint32_t);
    const size_t need = up(rank_bytes) + up(pat_bytes) + up(ring_bytes) + up(part_bytes) + up(ready_bytes) + up(done_bytes);
    if (ctx->eps_bytes < need) {
        if (ctx->d_eps) (void)hipFree(ctx->d_eps);
        ctx->d_eps = nullptr;
        ctx->eps_bytes = 0;
        AGIS_HIP(ctx, agis::ctx_malloc(ctx, &ctx->d_eps, need), "allocate run-to-eps buffers");
        ctx->eps_bytes = need;
    }
    char* base = (char*)ctx->d_eps;
    agis::EpsPattern* d_pat = (agis::EpsPattern*)base;
    double* d_ring = (double*)(base + up(pat_bytes));
    Partial* d_part = (Partial*)((char*)d_ring + up(ring_bytes));
    unsigned long long* d_ready = (unsigned long long*)((char*)d_part + up(part_bytes));
    uint32_t* d_done = (uint32_t*)((char*)d_ready + up(ready_bytes));
    uint32_t* d_ranks = (uint32_t*)((char*)d_done + up(done_bytes));
    std::vector<agis::EpsPattern> hp(npat);
    std::memset(hp.data(), 0, pat_bytes);
    for (uint32_t p = 0; p < npat; ++p) {
        hp[p].budget = runs[p].budget;
        hp[p].start = pp->first_sample;
        hp[p].check = check;
        hp[p].min_samples = pp->min_samples;
        hp[p].plan = p;
        hp[p].stop = runs[p].budget == 0 ? 1u : 0u;
    }
    AGIS_HIP(ctx, hipMemcpyAsync(d_pat, hp.data(), pat_bytes, hipMemcpyHostToDevice, ctx->stream), "upload states");
    // ready marks, tile counters, ranks and sample times start at zero (a fill
    // kernel, not a memset: the sequence could be captured)
    const size_t clear_bytes = up(ready_bytes) + up(done_bytes) + up(rank_bytes);
    AGIS_HIP(ctx, agis::launch_fill_u32((uint32_t*)d_ready, clear_bytes / 4, 0u, ctx->stream), "clear run-to-eps state");
    *ctx->h_cancel = 0;
    unsigned long long* d_clock = (unsigned long long*)((char*)ctx->d_small + kClockOffset);
    uint32_t* d_fault = (uint32_t*)((char*)ctx->d_small + kFaultOffset);
    AGIS_HIP(ctx, agis::launch_fill_u32(d_fault, 1, 0u, ctx->stream), "clear fault flag");
    agis::LaunchDesc ld;
    std::memset(&ld, 0, sizeof(ld));
    agis::fill_launch(ctx, L, g->g, dev_tables(t), nullptr, nullptr, &ld);
    ld.round.k0 = (uint32_t)seed;
    ld.round.k1 = (uint32_t)(seed >> 32);
    agis::EpsDesc& E = ld.eps;
    E.pat = agis::gmem(d_pat);
    E.ring = agis::gmem(d_ring);
    E.tile_done = agis::gmem(d_done);
    E.tile_part = agis::gmem(d_part);
    E.tile_ready = agis::gmem(d_ready);
    E.cancel = (const volatile uint32_t*)ctx->d_cancel;
    E.fault = agis::gmem(d_fault);
    E.clock0 = agis::gmem(d_clock);
    E.ring_samples = ring;
    E.window = window;
    E.npat = npat;
    // the largest grab of a wave (grabs grow with the merged count, see
    // k_sample_eps): 16 slots per atomic on the pattern's counter
    E.grab = std::max<uint32_t>(L.grab, 16u);
    E.ranks = agis::gmem(d_ranks);
    E.costs = agis::gmem(d_ranks + 1);
    E.rank_blocks = rank_blocks;
    E.look_ticks = (uint32_t)((int64_t)kEpsLookMicroseconds * ctx->wall_clock_khz / 1000);
    E.join_ticks = (uint32_t)((int64_t)kEpsJoinMicroseconds * ctx->wall_clock_khz / 1000);
    E.late_ticks = (uint32_t)((int64_t)kEpsLateMicroseconds * ctx->wall_clock_khz / 1000);
    E.late_merged = kEpsLateMerged;
    E.z = z;
    E.eps = pp->eps;
    AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_launch, &ld, sizeof(ld), hipMemcpyHostToDevice, ctx->stream), "upload launch");
    const auto t0 = std::chrono::steady_clock::now();
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_start, ctx->stream), "record event");
    const agis::LaunchDesc* desc = ctx->d_launch;
    void* args[] = {(void*)&desc};
    AGIS_HIP(ctx, hipLaunchKernel(agis::sample_eps_kernel(L.variant, L.pairs), dim3((unsigned)L.blocks),
                                  dim3((unsigned)L.threads), args, 0, ctx->stream),
             "launch run-to-eps sampler");
    AGIS_HIP(ctx, hipEventRecord(ctx->ev_stop, ctx->stream), "record event");
    if (pp->cancel) {
        // the caller's flag is forwarded to the pinned flag the kernel reads
        for (;;) {
            const hipError_t q = hipEventQuery(ctx->ev_stop);
            if (q == hipSuccess) break;
            if (q != hipErrorNotReady) return hip_fail(ctx, q, "run-to-eps sampler");
            if (!*cancelled && *pp->cancel) {
                *ctx->h_cancel = 1;
                *cancelled = true;
            }
            std::this_thread::sleep_for(std::chrono::microseconds(100));
        }
    }
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "run-to-eps sampler");
    const double wall = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    float ms = 0.0f;
    AGIS_HIP(ctx, hipEventElapsedTime(&ms, ctx->ev_start, ctx->ev_stop), "event time");
    unsigned long long clock0 = 0;
    uint32_t fault = 0;
    AGIS_HIP(ctx, hipMemcpy(hp.data(), d_pat, pat_bytes, hipMemcpyDeviceToHost), "read states");
    AGIS_HIP(ctx, hipMemcpy(&clock0, d_clock, sizeof(clock0), hipMemcpyDeviceToHost), "read clock");
    AGIS_HIP(ctx, hipMemcpy(&fault, d_fault, sizeof(fault), hipMemcpyDeviceToHost), "read fault flag");
    if (fault) return fail(ctx, AGIS_E_HIP, "run to eps: a wave waited too long for the merge (window wait bound)");
    *ctx->h_cancel = 0;
    double handed = 0.0;
    for (uint32_t p = 0; p < npat; ++p) handed += (double)std::min<uint64_t>(hp[p].next, hp[p].budget);
    const double tick = 1.0 / (1000.0 * (double)ctx->wall_clock_khz);
    for (uint32_t p = 0; p < npat; ++p) {
        PatternRun& r = runs[p];
        const agis::EpsPattern& s = hp[p];
        r.acc = Acc();
        r.acc.merge(s.acc);
        r.done = s.merged;
        r.converged = s.converged != 0;
        r.active = false;
        r.seconds = (s.stop && s.stop_clock >= clock0) ? (double)(s.stop_clock - clock0) * tick : wall;
        r.kernel_seconds = handed > 0 ? 1e-3 * (double)ms * (double)std::min<uint64_t>(s.next, s.budget) / handed : 0.0;
        r.launches = 1;
    }
    return AGIS_OK;
}

// Whether a run goes to epsilon in one persistent launch: runs to epsilon
// whose checks fall on reduction tiles, unless the caller asks for rounds.
bool device_eps(const agis_run_params* pp) {
    const uint64_t check = pp->check_every ? pp->check_every : 65536;
    return pp->eps > 0 && check % agis::kEpsTile == 0 && !(pp->flags & AGIS_RUN_HOST_ROUNDS);
}

void fill_result(const PatternRun& r, double z, double extra_seconds, agis_result* out) {
    std::memset(out, 0, sizeof(*out));
    const Acc& acc = r.acc;
    const double sc = r.prep.scale;
    out->estimate = acc.mean * sc;
    out->copies = r.prep.plan.aut ? acc.mean * sc / (double)r.prep.plan.aut : 0.0;
    out->variance = acc.n > 0 ? acc.m2 / acc.n * sc * sc : 0.0;
    out->eps_hat = eps_hat_of(acc, z);
    out->n = (uint64_t)acc.n;
    out->n_nonzero = (uint64_t)acc.nonzero;
    out->aut = r.prep.plan.aut;
    out->converged = r.converged ? 1 : 0;
    out->seconds = r.seconds + extra_seconds;
    out->tables_seconds = r.prep.tables_seconds;
    out->sample_kernel_seconds = r.kernel_seconds;
    out->sample_launches = r.launches;
    out->plan = r.prep.plan;
}

int check_handles(const agis_ctx* ctx, const agis_graph* g, const agis_tables* t) {
    if (!ctx || !g || !t) return AGIS_E_INVALID_ARG;
    if (g->ctx != ctx || t->ctx != ctx || t->graph != g) return AGIS_E_INVALID_ARG;
    return AGIS_OK;
}

}  // namespace

extern "C" {

int agis_create(agis_ctx** out, int device, void* hip_stream) try {
    if (!out) return AGIS_E_INVALID_ARG;
    *out = nullptr;
    agis_ctx* ctx = new (std::nothrow) agis_ctx();
    if (!ctx) return AGIS_E_OOM;
    ctx->device = device;
    ctx->pool->set_device(device);
    ctx->stream = (hipStream_t)hip_stream;
    hipError_t e = hipSetDevice(device);
    if (e == hipSuccess) {
        hipDeviceProp_t prop;
        e = hipGetDeviceProperties(&prop, device);
        if (e == hipSuccess) ctx->num_cus = prop.multiProcessorCount;
    }
    if (e == hipSuccess) e = hipMalloc(&ctx->d_plans, agis::kMaxSegs * sizeof(DevPlan));
    if (e == hipSuccess) e = hipMalloc(&ctx->d_launch, sizeof(agis::LaunchDesc));
    if (e == hipSuccess) e = hipMalloc(&ctx->d_small, agis::kSmallBytes);
    if (e == hipSuccess) {
        // the fixed workspace of agis_estimate_noalloc; a failed lookup only
        // disables that entry point (it reports the failure)
        void* p = nullptr;
        if (noalloc_scratch_ptr(device, &p) == hipSuccess)
            ctx->noalloc_scratch = p;
        else
            (void)hipGetLastError();
    }
    if (e == hipSuccess) {
        void* h = nullptr;
        void* d = nullptr;
        e = hipHostMalloc(&h, 64, hipHostMallocMapped | hipHostMallocCoherent);
        if (e == hipSuccess) {
            ctx->h_cancel = (volatile uint32_t*)h;
            *ctx->h_cancel = 0;
            e = hipHostGetDevicePointer(&d, h, 0);
            ctx->d_cancel = (const volatile uint32_t*)d;
        }
    }
    if (e == hipSuccess) {
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) == hipSuccess && khz > 0)
            ctx->wall_clock_khz = khz;
    }
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&ctx->graph_stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_in, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_out, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreate(&ctx->ev_start);
    if (e == hipSuccess) e = hipEventCreate(&ctx->ev_stop);
    if (e == hipSuccess) e = agis::upload_fixed_point_tables(ctx->stream);
    if (e != hipSuccess) {
        agis_destroy(ctx);
        return e == hipErrorOutOfMemory ? AGIS_E_OOM : AGIS_E_HIP;
    }
    *out = ctx;
    return AGIS_OK;
} AGIS_CATCH(nullptr)

void agis_destroy(agis_ctx* ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
    if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
    if (ctx->graph_stream) (void)hipStreamDestroy(ctx->graph_stream);
    if (ctx->ev_in) (void)hipEventDestroy(ctx->ev_in);
    if (ctx->ev_out) (void)hipEventDestroy(ctx->ev_out);
    if (ctx->d_plans) (void)hipFree(ctx->d_plans);
    if (ctx->d_launch) (void)hipFree(ctx->d_launch);
    if (ctx->d_small) (void)hipFree(ctx->d_small);
    if (ctx->d_partials) (void)hipFree(ctx->d_partials);
    if (ctx->d_scratch) (void)hipFree(ctx->d_scratch);
    if (ctx->d_xout) (void)hipFree(ctx->d_xout);
    if (ctx->d_blocksums) (void)hipFree(ctx->d_blocksums);
    if (ctx->d_eps) (void)hipFree(ctx->d_eps);
    if (ctx->h_cancel) (void)hipHostFree((void*)ctx->h_cancel);
    ctx->pool->close();
    if (ctx->ev_start) (void)hipEventDestroy(ctx->ev_start);
    if (ctx->ev_stop) (void)hipEventDestroy(ctx->ev_stop);
    delete ctx;
}

int agis_release_scratch(agis_ctx* ctx) try {
    if (!ctx) return AGIS_E_INVALID_ARG;
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "wait for the context's stream");
    // the captured round refers to these buffers
    if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
    if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
    ctx->graph_exec = nullptr;
    ctx->graph = nullptr;
    std::memset(ctx->graph_key, 0, sizeof(ctx->graph_key));
    for (void** q : {&ctx->d_scratch, (void**)&ctx->d_xout, (void**)&ctx->d_partials, &ctx->d_eps}) {
        if (*q) AGIS_HIP(ctx, hipFree(*q), "free sampler buffers");
        *q = nullptr;
    }
    ctx->scratch_bytes = 0;
    ctx->xout_cap = 0;
    ctx->partials_cap = 0;
    ctx->eps_bytes = 0;
    ctx->pool->trim();
    return AGIS_OK;
} AGIS_CATCH(ctx)

const char* agis_last_error(const agis_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int agis_load_csr(agis_ctx* ctx, const uint64_t* off, const uint32_t* nbr, uint64_t n, uint64_t nnz, uint32_t flags,
                  agis_graph** out) try {
    if (!ctx || !out) return AGIS_E_INVALID_ARG;
    *out = nullptr;
    if (n == 0 || n >= (1ull << 32)) return fail(ctx, AGIS_E_INVALID_ARG, "n must be in [1, 2^32)");
    if (!off || (nnz > 0 && !nbr)) return fail(ctx, AGIS_E_INVALID_ARG, "null CSR pointer");
    if (flags & ~AGIS_CSR_VALIDATE) return fail(ctx, AGIS_E_INVALID_ARG, "unknown flag");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    uint64_t ends[2] = {1, 1};
    AGIS_HIP(ctx, hipMemcpyAsync(&ends[0], off, sizeof(uint64_t), hipMemcpyDeviceToHost, ctx->stream), "read off[0]");
    AGIS_HIP(ctx, hipMemcpyAsync(&ends[1], off + n, sizeof(uint64_t), hipMemcpyDeviceToHost, ctx->stream),
             "read off[n]");
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "read offsets");
    if (ends[0] != 0 || ends[1] != nnz) return fail(ctx, AGIS_E_INVALID_CSR, "off[0] must be 0 and off[n] must be nnz");
    if (nnz & 1ull) return fail(ctx, AGIS_E_INVALID_CSR, "nnz of a symmetric graph must be even");
    agis::DevGraph dg{agis::gmem(off), agis::gmem(nbr), n, nnz};
    uint32_t* d_cells = (uint32_t*)ctx->d_small;
    // fault flags, largest degree, and where a round's slot counters are the
    // counts of the slots that point down
    uint32_t cells[agis::kSmallBytes / 4] = {0};
    AGIS_HIP(ctx, hipMemsetAsync(d_cells, 0, sizeof(cells), ctx->stream), "clear flags");
    if (flags & AGIS_CSR_VALIDATE) {
        AGIS_HIP(ctx, agis::launch_validate_rows(dg, d_cells, ctx->stream), "validate CSR rows");
        AGIS_HIP(ctx, hipMemcpyAsync(cells, d_cells, sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->stream),
                 "read flags");
        AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "validate CSR rows");
        if (cells[0] == 0)
            AGIS_HIP(ctx, agis::launch_validate_edges(ctx, dg, d_cells, (uint64_t*)(d_cells + agis::kQueueOffset / 4)), "validate CSR edges");
    }
    if (cells[0] == 0) AGIS_HIP(ctx, agis::launch_max_degree(dg, d_cells + 1, ctx->stream), "max degree");
    AGIS_HIP(ctx, hipMemcpyAsync(cells, d_cells, sizeof(cells), hipMemcpyDeviceToHost, ctx->stream), "read flags");
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "validate CSR");
    if ((flags & AGIS_CSR_VALIDATE) && cells[0] == 0) {
        uint64_t lower = 0;
        for (uint32_t q = 0; q < agis::kQueues; ++q) {
            uint64_t c = 0;
            std::memcpy(&c, (const char*)cells + agis::kQueueOffset + (size_t)q * agis::kQueueStride * 8, sizeof(c));
            lower += c;
        }
        if (2 * lower != nnz) cells[0] |= 16u;
    }
    if (cells[0]) {
        std::string m = "invalid CSR:";
        if (cells[0] & 1u) m += " offsets not non-decreasing or beyond nnz;";
        if (cells[0] & 2u) m += " neighbour id >= n;";
        if (cells[0] & 4u) m += " self-loop;";
        if (cells[0] & 8u) m += " row not strictly ascending (unsorted or duplicate);";
        if (cells[0] & 16u) m += " not symmetric;";
        return fail(ctx, AGIS_E_INVALID_CSR, m);
    }
    agis_graph* g = new (std::nothrow) agis_graph();
    if (!g) return fail(ctx, AGIS_E_OOM, "host allocation");
    g->ctx = ctx;
    g->g = dg;
    g->max_deg = cells[1];
    *out = g;
    return AGIS_OK;
} AGIS_CATCH(ctx)

void agis_graph_destroy(agis_graph* g) {
    if (!g) return;
    if (g->own_off || g->own_nbr) {
        sync_device(g->device);
        g->pool->free(g->own_off);
        g->pool->free(g->own_nbr);
    }
    delete g;
}

int agis_orient(agis_ctx* ctx, const agis_graph* g, agis_graph** out) try {
    if (!ctx || !g || !out || g->ctx != ctx) return AGIS_E_INVALID_ARG;
    *out = nullptr;
    if (g->parent) return fail(ctx, AGIS_E_INVALID_ARG, "the graph is already oriented");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    const uint64_t n = g->g.n;
    agis_graph* o = new (std::nothrow) agis_graph();
    if (!o) return fail(ctx, AGIS_E_OOM, "host allocation");
    o->ctx = ctx;
    o->parent = g;
    o->pool = ctx->pool;
    o->device = ctx->device;
    uint64_t *mask = nullptr, *run_kept = nullptr;
    uint32_t* deg = nullptr;
    hipError_t e = ctx->pool->alloc(&o->own_off, (n + 1) * sizeof(uint64_t));
    if (e == hipSuccess)
        e = ctx->pool->alloc(&mask, std::max<uint64_t>(agis::orient_words(g->g.nnz), 1) * sizeof(uint64_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&run_kept, (agis::orient_runs(g->g.nnz) + 1) * sizeof(uint64_t));
    if (e == hipSuccess && ctx->pool->alloc(&deg, n * sizeof(uint32_t)) != hipSuccess) {
        (void)hipGetLastError();  // no room: the degrees come from the offsets
        deg = nullptr;
    }
    if (e == hipSuccess) e = agis::launch_orient_offsets(ctx, g->g, deg, mask, run_kept, o->own_off);
    uint64_t nnz = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&nnz, o->own_off + n, sizeof(uint64_t), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    ctx->pool->free(deg);
    if (e == hipSuccess) e = ctx->pool->alloc(&o->own_nbr, (nnz ? nnz : 1) * sizeof(uint32_t));
    if (e == hipSuccess) e = agis::launch_orient_fill(ctx, g->g, mask, run_kept, o->own_nbr);
    uint32_t* d_max = (uint32_t*)ctx->d_small;
    uint32_t maxd = 0;
    o->g = agis::DevGraph{agis::gmem((const uint64_t*)o->own_off), agis::gmem((const uint32_t*)o->own_nbr), n, nnz};
    if (e == hipSuccess) e = hipMemsetAsync(d_max, 0, sizeof(uint32_t), ctx->stream);
    if (e == hipSuccess) e = agis::launch_max_degree(o->g, d_max, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(&maxd, d_max, sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) (void)hipStreamSynchronize(ctx->stream);
    ctx->pool->free(mask);
    ctx->pool->free(run_kept);
    if (e != hipSuccess) {
        agis_graph_destroy(o);
        return hip_fail(ctx, e, "orient graph");
    }
    o->max_deg = maxd;
    *out = o;
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_graph_export(agis_ctx* ctx, const agis_graph* g, uint64_t* n, uint64_t* nnz, const uint64_t** off,
                      const uint32_t** nbr) {
    if (!ctx || !g || g->ctx != ctx) return AGIS_E_INVALID_ARG;
    if (n) *n = g->g.n;
    if (nnz) *nnz = g->g.nnz;
    if (off) *off = (const uint64_t*)g->g.off;
    if (nbr) *nbr = (const uint32_t*)g->g.nbr;
    return AGIS_OK;
}

int agis_build_proposal_tables(agis_ctx* ctx, const agis_graph* g, uint64_t cv_seed, int32_t lc_min_q16,
                               int32_t exact_cv, agis_tables** out) try {
    if (!ctx || !g || !out || g->ctx != ctx) return AGIS_E_INVALID_ARG;
    *out = nullptr;
    if (lc_min_q16 > 0) return fail(ctx, AGIS_E_INVALID_ARG, "log2 of the clustering floor must be <= 0");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    ctx->pool->check();
    agis_tables* t = new (std::nothrow) agis_tables();
    if (t) t->cache = new (std::nothrow) TableCache();
    if (!t || !t->cache) {
        delete t;
        return fail(ctx, AGIS_E_OOM, "host allocation");
    }
    std::unique_ptr<agis_tables, void (*)(agis_tables*)> hold(t, agis_tables_destroy);
    t->ctx = ctx;
    t->pool = t->cache->pool = ctx->pool;
    t->device = ctx->device;
    t->graph = g;
    const uint64_t n = g->g.n;
    hipError_t e = ctx->pool->alloc(&t->rec, n * sizeof(uint4));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->s2, n * sizeof(uint64_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->hits, n * sizeof(uint64_t));
    if (e == hipSuccess) e = ctx->pool->alloc(&t->trials, n * sizeof(uint64_t));
    // the bitmaps first: they decide most of the clustering trials
    if (e == hipSuccess) e = build_hub_bitmaps(ctx, g, t);
    if (e == hipSuccess)
        e = agis::launch_build_tables(ctx, g->g, g->parent ? g->parent->g : g->g, *t, (uint32_t)cv_seed,
                                      (uint32_t)(cv_seed >> 32), lc_min_q16, exact_cv ? 1 : 0);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(ctx, e, "build proposal tables");
    *out = hold.release();
    return AGIS_OK;
} AGIS_CATCH(ctx)

void agis_tables_destroy(agis_tables* t) {
    if (!t) return;
    sync_device(t->device);
    delete t->cache;
    for (void* q : {(void*)t->rec, (void*)t->s2, (void*)t->hits, (void*)t->trials, (void*)t->hub_bits,
                    (void*)t->hub_slot, (void*)t->pair_slot, (void*)t->pair_count, (void*)t->pair_quart,
                    (void*)t->core_slot, (void*)t->core_start, (void*)t->core_len, (void*)t->core_nbr})
        t->pool->free(q);
    delete t;
}

int agis_tables_export(agis_ctx* ctx, const agis_tables* t, uint32_t* deg, uint64_t* s2, uint64_t* hits,
                       uint64_t* trials, int32_t* la, int32_t* lc) try {
    if (!ctx || !t || t->ctx != ctx) return AGIS_E_INVALID_ARG;
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    const uint64_t n = t->graph->g.n;
    hipStream_t st = ctx->stream;
    if (s2) AGIS_HIP(ctx, hipMemcpyAsync(s2, t->s2, n * 8, hipMemcpyDeviceToDevice, st), "export s2");
    if (hits) AGIS_HIP(ctx, hipMemcpyAsync(hits, t->hits, n * 8, hipMemcpyDeviceToDevice, st), "export hits");
    if (trials) AGIS_HIP(ctx, hipMemcpyAsync(trials, t->trials, n * 8, hipMemcpyDeviceToDevice, st), "export trials");
    AGIS_HIP(ctx, agis::launch_export_tables(*t, n, deg, la, lc, st), "export tables");
    AGIS_HIP(ctx, hipStreamSynchronize(st), "export tables");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_compile_pattern(const agis_pattern* p, const uint8_t* order, const agis_run_params* params, agis_plan* out) try {
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    std::string err;
    return agis::compile_plan(p, order, pp->mode, pp->beta_num, pp->beta_den, out, &err);
} AGIS_CATCH(nullptr)

int agis_step1_weights(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                       const uint8_t* order, const agis_run_params* params, uint32_t* q1, uint64_t* total) try {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (!p || !q1 || !total) return fail(ctx, AGIS_E_INVALID_ARG, "null pattern, weights or total");
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    // the weights of every vertex are exported: the full first-step table
    agis_run_params full = *pp;
    full.flags = (full.flags & ~AGIS_RUN_STEP1_BLOCKS) | AGIS_RUN_STEP1_FULL;
    StepTables st;
    Prepared prep;
    rc = prepare(ctx, g, t, p, order, &full, 0, &st, &prep);
    if (rc != AGIS_OK) return rc;
    const uint64_t n = g->g.n;
    if (prep.hp.weighted[0]) {
        if (n)
            AGIS_HIP(ctx,
                     hipMemcpyAsync(q1, (const uint32_t*)prep.hp.s1_q, n * sizeof(uint32_t), hipMemcpyDeviceToDevice,
                                    ctx->stream),
                     "copy first-step weights");
        *total = prep.hp.s1_total;
    } else {
        // edge-uniform first step: P(v) = d(v) / nnz
        AGIS_HIP(ctx, agis::launch_export_tables(*t, n, q1, nullptr, nullptr, ctx->stream), "degrees");
        *total = g->g.nnz;
    }
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "first-step weights");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_connected_patterns(uint32_t k, agis_pattern* out, uint32_t cap, uint32_t* count) try {
    if (!count) return AGIS_E_INVALID_ARG;
    std::string err;
    return agis::connected_patterns(k, out, cap, count, &err);
} AGIS_CATCH(nullptr)

int agis_concentrations(uint32_t n_patterns, const agis_pattern* patterns, const double* copies, double* conc_edge,
                        double* induced, double* conc_induced) try {
    std::string err;
    return agis::concentrations(n_patterns, patterns, copies, conc_edge, induced, conc_induced, &err);
} AGIS_CATCH(nullptr)

int agis_estimate(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                  const uint8_t* order, uint64_t n_samples, uint64_t seed, const agis_run_params* params,
                  agis_result* out) try {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (!p || !out) return fail(ctx, AGIS_E_INVALID_ARG, "null pattern or result");
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    if (pp->eps > 0 && !(pp->delta > 0 && pp->delta < 1)) return fail(ctx, AGIS_E_INVALID_ARG, "delta must be in (0, 1)");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    const auto t0 = std::chrono::steady_clock::now();
    StepTables st;
    std::vector<PatternRun> runs(1);
    rc = prepare(ctx, g, t, p, order, pp, n_samples, &st, &runs[0].prep);
    if (rc != AGIS_OK) return rc;
    runs[0].budget = n_samples;
    const double setup = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    bool cancelled = false;
    rc = device_eps(pp) ? run_device_eps(ctx, g, t, runs, pp, seed, &cancelled)
                        : run_rounds(ctx, g, t, runs, pp, seed, &cancelled);
    if (rc != AGIS_OK) return rc;
    const double z = normal_quantile(1.0 - (pp->eps > 0 ? pp->delta : 0.05) / 2.0);
    fill_result(runs[0], z, setup, out);
    if (cancelled) return fail(ctx, AGIS_E_CANCELLED, "cancelled by the caller");
    if (pp->eps > 0 && !runs[0].converged) return fail(ctx, AGIS_E_NOT_CONVERGED, "sample budget reached before eps");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_estimate_noalloc(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                          const uint8_t* order, uint64_t n_samples, uint64_t seed, const agis_run_params* params,
                          agis_result* out) try {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (!p || !out) return fail(ctx, AGIS_E_INVALID_ARG, "null pattern or result");
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    if (pp->eps > 0 && !(pp->delta > 0 && pp->delta < 1)) return fail(ctx, AGIS_E_INVALID_ARG, "delta must be in (0, 1)");
    if (!ctx->noalloc_scratch) return fail(ctx, AGIS_E_HIP, "the fixed workspace has no device address");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    const auto t0 = std::chrono::steady_clock::now();
    // every buffer of this call comes from this device's fixed workspace;
    // calls on one device share it (overlapping calls race)
    agis::Arena arena;
    arena.base = (char*)ctx->noalloc_scratch;
    arena.cap = kNoAllocBytes;
    StepTables st;
    st.arena = &arena;
    std::vector<PatternRun> runs(1);
    rc = prepare(ctx, g, t, p, order, pp, n_samples, &st, &runs[0].prep);
    if (rc != AGIS_OK) return rc;
    runs[0].budget = n_samples;
    const double setup = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    bool cancelled = false;
    rc = run_rounds(ctx, g, t, runs, pp, seed, &cancelled, &arena);
    if (rc != AGIS_OK) return rc;
    const double z = normal_quantile(1.0 - (pp->eps > 0 ? pp->delta : 0.05) / 2.0);
    fill_result(runs[0], z, setup, out);
    if (cancelled) return fail(ctx, AGIS_E_CANCELLED, "cancelled by the caller");
    if (pp->eps > 0 && !runs[0].converged) return fail(ctx, AGIS_E_NOT_CONVERGED, "sample budget reached before eps");
    return AGIS_OK;
} AGIS_CATCH(ctx)

int agis_estimate_batch(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, uint32_t n_patterns,
                        const agis_pattern* patterns, const uint64_t* budgets, uint64_t seed,
                        const agis_run_params* params, agis_result* out) try {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (n_patterns == 0 || n_patterns > agis::kMaxSegs) return fail(ctx, AGIS_E_INVALID_ARG, "1..64 patterns per batch");
    if (!patterns || !budgets || !out) return fail(ctx, AGIS_E_INVALID_ARG, "null pattern, budget or result array");
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    if (pp->eps > 0 && !(pp->delta > 0 && pp->delta < 1)) return fail(ctx, AGIS_E_INVALID_ARG, "delta must be in (0, 1)");
    if (pp->mode == AGIS_MODE_LEARNED && !pp->batch_learned)
        return fail(ctx, AGIS_E_INVALID_ARG, "learned mode in a batch needs batch_learned (tables per pattern)");
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    const auto t0 = std::chrono::steady_clock::now();
    StepTables st;
    std::vector<PatternRun> runs(n_patterns);
    for (uint32_t i = 0; i < n_patterns; ++i) {
        agis_run_params pi = *pp;
        pi.pattern_id = pp->pattern_id + i;
        if (pp->mode == AGIS_MODE_LEARNED)
            for (int j = 0; j < AGIS_MAX_K; ++j) pi.learned[j] = pp->batch_learned[(size_t)i * AGIS_MAX_K + j];
        rc = prepare(ctx, g, t, &patterns[i], nullptr, &pi, budgets[i], &st, &runs[i].prep);
        if (rc != AGIS_OK) return rc;
        runs[i].budget = budgets[i];
        runs[i].active = budgets[i] > 0;
    }
    const double setup = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    bool cancelled = false;
    rc = device_eps(pp) ? run_device_eps(ctx, g, t, runs, pp, seed, &cancelled)
                        : run_rounds(ctx, g, t, runs, pp, seed, &cancelled);
    if (rc != AGIS_OK) return rc;
    const double z = normal_quantile(1.0 - (pp->eps > 0 ? pp->delta : 0.05) / 2.0);
    bool all = true;
    for (uint32_t i = 0; i < n_patterns; ++i) {
        fill_result(runs[i], z, setup, &out[i]);
        all = all && runs[i].converged;
    }
    if (cancelled) return fail(ctx, AGIS_E_CANCELLED, "cancelled by the caller");
    if (pp->eps > 0 && !all) return fail(ctx, AGIS_E_NOT_CONVERGED, "a pattern reached its budget before eps");
    return AGIS_OK;
} AGIS_CATCH(ctx)

// Runs the samples listed in idx (device uint64[m]) once: with `out` the
// record-writing kernel writes one record each; with `meter` the metering
// kernel (production paths) writes four request counters each.
static int run_indexed(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                       const uint8_t* order, uint64_t seed, const agis_run_params* params, const uint64_t* idx,
                       uint64_t m, agis_record* out, uint64_t* meter) {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (!p || (m > 0 && (!idx || (!out && !meter)))) return fail(ctx, AGIS_E_INVALID_ARG, "null pattern, index list or output");
    static_assert(sizeof(agis_record) == sizeof(agis::Record), "record layout");
    const agis_run_params dp = default_params();
    const agis_run_params* pp = params ? params : &dp;
    AGIS_HIP(ctx, hipSetDevice(ctx->device), "set device");
    StepTables st;
    Prepared prep;
    rc = prepare(ctx, g, t, p, order, pp, m, &st, &prep);
    if (rc != AGIS_OK) return rc;
    if (m == 0) return AGIS_OK;
    if (m > kMaxRoundSlots) return fail(ctx, AGIS_E_INVALID_ARG, "at most 2^24 samples per call");
    agis::SampleLaunch L;
    L.lanes = !(pp->flags & AGIS_RUN_WAVE_SAMPLES) && agis::lane_plan(prep.hp);
    L.pairs = !L.lanes && uses_pair_hubs(prep.hp, t);
    rc = agis::plan_sample_launch(ctx, *g, m, 1, &L, &ctx->err);
    if (rc != AGIS_OK) return rc;
    L.dump = out != nullptr;
    L.meter = out == nullptr;
    agis::LaunchDesc ld;
    std::memset(&ld, 0, sizeof(ld));
    agis::fill_launch(ctx, L, g->g, dev_tables(t), idx, (agis::Record*)out, &ld, meter);
    agis::RoundDesc& rd = ld.round;
    rd.total = m;
    rd.nseg = 1;
    rd.k0 = (uint32_t)seed;
    rd.k1 = (uint32_t)(seed >> 32);
    rd.seg[0].count = m;
    rd.seg[0].ntiles = (uint32_t)((m + agis::kReduceTileSamples - 1) / agis::kReduceTileSamples);
    AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_plans, &prep.hp, sizeof(DevPlan), hipMemcpyHostToDevice, ctx->stream),
             "upload plan");
    AGIS_HIP(ctx, hipMemcpyAsync(ctx->d_launch, &ld, sizeof(ld), hipMemcpyHostToDevice, ctx->stream), "upload round");
    AGIS_HIP(ctx, agis::launch_round(ctx, ctx->stream, L, nullptr, nullptr), "launch sampler");
    AGIS_HIP(ctx, hipStreamSynchronize(ctx->stream), "sampler");
    return AGIS_OK;
}

int agis_dump_samples(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                      const uint8_t* order, uint64_t seed, const agis_run_params* params, const uint64_t* idx,
                      uint64_t m, agis_record* out) try {
    if (ctx && m > 0 && !out) return fail(ctx, AGIS_E_INVALID_ARG, "null output");
    return run_indexed(ctx, g, t, p, order, seed, params, idx, m, out, nullptr);
} AGIS_CATCH(ctx)

int agis_meter_samples(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, const agis_pattern* p,
                       const uint8_t* order, uint64_t seed, const agis_run_params* params, const uint64_t* idx,
                       uint64_t m, uint64_t* out) try {
    if (ctx && m > 0 && !out) return fail(ctx, AGIS_E_INVALID_ARG, "null output");
    return run_indexed(ctx, g, t, p, order, seed, params, idx, m, nullptr, out);
} AGIS_CATCH(ctx)

int agis_set_launch(agis_ctx* ctx, int32_t use_graphs, int32_t blocks_per_cu, uint32_t grab, int32_t variant,
                    uint32_t hub_window) {
    if (!ctx || blocks_per_cu < 0 || grab > 1024 || variant < -1 || variant > 2) return AGIS_E_INVALID_ARG;
    ctx->use_graphs = use_graphs ? 1 : 0;
    ctx->tune_blocks_per_cu = blocks_per_cu;
    ctx->tune_grab = grab;
    ctx->tune_variant = variant;
    ctx->tune_hub_window = hub_window;
    return AGIS_OK;
}

// For tests (not declared in the header): rows of at most `words` words (a
// power of two up to 64), as where memory is short.
__attribute__((visibility("default"))) int agis_internal_row_words(agis_ctx* ctx, uint32_t words) {
    if (!ctx || words == 0 || words > agis::kPairRowWords || (words & (words - 1))) return AGIS_E_INVALID_ARG;
    ctx->max_row_words = words;
    return AGIS_OK;
}

int agis_autotune(agis_ctx* ctx, const agis_graph* g, const agis_tables* t, uint32_t n_patterns,
                  const agis_pattern* patterns, uint64_t pilot_samples, const agis_run_params* params,
                  agis_tuning* out) try {
    int rc = check_handles(ctx, g, t);
    if (rc != AGIS_OK) return ctx ? fail(ctx, rc, "bad handle") : rc;
    if (!patterns || !out || n_patterns == 0 || n_patterns > agis::kMaxSegs || pilot_samples == 0)
        return fail(ctx, AGIS_E_INVALID_ARG, "1..64 patterns and a nonzero pilot size");
    agis_run_params pp = params ? *params : default_params();
    pp.eps = 0.0;  // pilots run fixed budgets
    if (pp.mode == AGIS_MODE_LEARNED) pp.mode = AGIS_MODE_SWITCH;
    std::vector<uint64_t> budgets(n_patterns, pilot_samples);
    std::vector<agis_result> res(n_patterns);
    const int saved_graphs = ctx->use_graphs, saved_blocks = ctx->tune_blocks_per_cu, saved_variant = ctx->tune_variant;
    const uint32_t saved_grab = ctx->tune_grab, saved_window = ctx->tune_hub_window;
    struct Cand {
        int variant;
        uint32_t grab;
        uint32_t window;
    };
    // first the register budget x queue grab, then the hub-bitmap window
    // with the best of those
    // explicit grabs (the automatic one depends on the round size, which
    // differs between the pilots and the runs the tuning is for); the
    // launch's own register budget (-1) first, as the default, then the others
    const int own = agis::fixed_variant(g->g);
    const int budgets_tried[3] = {-1, own == 0 ? 1 : 0, own == 2 ? 1 : 2};
    Cand cands[9 + 3];
    for (uint32_t i = 0; i < 9; ++i) cands[i] = Cand{budgets_tried[i % 3], 1u << (i / 3), 0};
    double best = INFINITY, first = 0.0;
    Cand best_c = cands[0];
    auto time_config = [&](const Cand& c, double* secs) -> int {
        ctx->use_graphs = 1;
        ctx->tune_blocks_per_cu = 0;
        ctx->tune_variant = c.variant;
        ctx->tune_grab = c.grab;
        ctx->tune_hub_window = c.window;
        *secs = 0.0;
        for (int rep = 0; rep < 2; ++rep) {  // first repetition warms caches and captures the graph
            const int r = agis_estimate_batch(ctx, g, t, n_patterns, patterns, budgets.data(), 0x5eed, &pp, res.data());
            if (r != AGIS_OK) return r;
            if (rep == 1)
                for (const agis_result& x : res) *secs += x.sample_kernel_seconds;
        }
        return AGIS_OK;
    };
    for (int ci = 0; ci < 12 && rc == AGIS_OK; ++ci) {
        if (ci == 9) {
            const uint32_t windows[3] = {256, 1024, 4096};
            for (int w = 0; w < 3; ++w) cands[9 + w] = Cand{best_c.variant, best_c.grab, windows[w]};
        }
        double secs = 0.0;
        rc = time_config(cands[ci], &secs);
        if (rc != AGIS_OK) break;
        if (ci == 0) first = secs;
        // a candidate must beat the best so far by 2%: pilot times carry
        // noise of about that size (the first candidate is the launch's own
        // register budget, grab 1, no hub window)
        if (secs < best * 0.98) {
            best = secs;
            best_c = cands[ci];
        }
    }
    ctx->use_graphs = saved_graphs;
    ctx->tune_blocks_per_cu = saved_blocks;
    ctx->tune_variant = saved_variant;
    ctx->tune_grab = saved_grab;
    ctx->tune_hub_window = saved_window;
    if (rc != AGIS_OK) return rc;
    out->use_graphs = 1;
    out->blocks_per_cu = 0;
    out->grab = best_c.grab;
    out->variant = best_c.variant < 0 ? own : best_c.variant;
    out->hub_window = best_c.window;
    out->seconds = best;
    out->default_seconds = first;
    return agis_set_launch(ctx, 1, 0, best_c.grab, best_c.variant, best_c.window);
} AGIS_CATCH(ctx)

int agis_fixed_point_tables(int32_t* logtab, uint32_t* exp2tab) {
    if (!logtab || !exp2tab) return AGIS_E_INVALID_ARG;
    std::memcpy(logtab, agis::host_logtab(), 4096 * sizeof(int32_t));
    std::memcpy(exp2tab, agis::host_exp2tab(), 4096 * sizeof(uint32_t));
    return AGIS_OK;
}

int agis_philox4x32_10(const uint32_t ctr[4], const uint32_t key[2], uint32_t out[4]) {
    if (!ctr || !key || !out) return AGIS_E_INVALID_ARG;
    agis::U32x4 o = agis::philox4x32_10(agis::U32x4{ctr[0], ctr[1], ctr[2], ctr[3]}, key[0], key[1]);
    out[0] = o.x;
    out[1] = o.y;
    out[2] = o.z;
    out[3] = o.w;
    return AGIS_OK;
}

}  // extern "C"
