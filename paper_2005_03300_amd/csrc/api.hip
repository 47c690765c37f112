// Error reporting, settings, event timing, allocation helpers and gcn_csr accessors.
#include <stdarg.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "common.h"
#include "copy_rule.h"
#include "scratch_pool.h"

namespace gcn {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

// ---- device memory ---------------------------------------------------------------------------
namespace {
struct Block { void* p; size_t bytes; int device; };
std::mutex g_pool_mu;
std::vector<Block> g_pool;                          // given back and kept, oldest first
std::unordered_map<void*, Block> g_live;            // handed out

int current_device() {
    int dev = 0;
    (void)hipGetDevice(&dev);
    return dev;
}

// takes the smallest block of `list` that holds `bytes` and is not larger than `most`
bool take_block(std::vector<Block>& list, int dev, size_t bytes, size_t most, Block* out) {
    int best = -1;
    for (int i = 0; i < (int)list.size(); ++i)
        if (list[i].device == dev && list[i].bytes >= bytes && list[i].bytes <= most &&
            (best < 0 || list[i].bytes < list[best].bytes))
            best = i;
    if (best < 0) return false;
    *out = list[best];
    list.erase(list.begin() + best);
    return true;
}

size_t pool_limit(int dev) {
    static std::mutex mu;
    static size_t limit[64] = {};
    if (dev < 0 || dev >= 64) dev = 0;
    std::lock_guard<std::mutex> lk(mu);
    if (!limit[dev]) {
        size_t total = 0;
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess) total = prop.totalGlobalMem;
        limit[dev] = total / 64 + 1;
    }
    return limit[dev];
}
}  // namespace

void device_pool_release() {
    std::vector<Block> all;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        all.swap(g_pool);
    }
    for (auto& b : all) (void)hipFree(b.p);
}

int device_alloc(void** p, size_t bytes) {
    *p = nullptr;
    const size_t unit = bytes >= (1u << 20) ? (size_t)1 << 16 : 512;
    bytes = bytes == 0 ? unit : (bytes + unit - 1) / unit * unit;
    const int dev = current_device();
    Block b;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        if (take_block(g_pool, dev, bytes, bytes + bytes / 8 + 4096, &b)) {
            g_live[b.p] = b;
            *p = b.p;
            return GCN_OK;
        }
    }
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        device_pool_release();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return fail(e == hipErrorOutOfMemory ? GCN_ERR_OOM : GCN_ERR_HIP, "hipMalloc(%zu) failed: %s", bytes,
                    hipGetErrorString(e));
    }
    std::lock_guard<std::mutex> lk(g_pool_mu);
    g_live[*p] = Block{*p, bytes, dev};
    return GCN_OK;
}

void device_free(void* p) {
    if (!p) return;
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        auto it = g_live.find(p);
        if (it == g_live.end()) {
            out.push_back({p, 0, 0});
        } else {
            const Block b = it->second;
            g_live.erase(it);
            const size_t limit = pool_limit(b.device);
            if (b.bytes > limit) {
                out.push_back(b);
            } else {
                size_t held = b.bytes;
                for (auto& x : g_pool)
                    if (x.device == b.device) held += x.bytes;
                for (size_t i = 0; i < g_pool.size() && held > limit;) {
                    if (g_pool[i].device != b.device) { ++i; continue; }
                    held -= g_pool[i].bytes;
                    out.push_back(g_pool[i]);
                    g_pool.erase(g_pool.begin() + (long)i);
                }
                g_pool.push_back(b);
            }
        }
    }
    for (auto& x : out) (void)hipFree(x.p);
}

// ---- temporaries of graph construction ---------------------------------------------------------
namespace {
struct Build {
    hipStream_t stream;
    std::vector<Block> spare;                       // dropped by this build, reusable on its stream
};
thread_local Build* g_build = nullptr;
constexpr size_t BUILD_SPARE_MAX = (size_t)1 << 30; // larger temporaries leave at once: they decide the peak
}  // namespace

BuildScope::BuildScope(hipStream_t s) : owner(g_build == nullptr) {
    if (owner) g_build = new Build{s, {}};
}
BuildScope::~BuildScope() {
    if (!owner) return;
    Build* b = g_build;
    g_build = nullptr;
    (void)hipStreamSynchronize(b->stream);
    for (auto& x : b->spare) device_free(x.p);
    delete b;
}

int temp_alloc(void** p, size_t bytes) {
    Block b;
    if (g_build && take_block(g_build->spare, current_device(), bytes, 2 * bytes + 65536, &b)) {
        *p = b.p;
        return GCN_OK;
    }
    return device_alloc(p, bytes);
}

void temp_free(void* p) {
    if (!p) return;
    if (g_build) {
        Block b{p, 0, 0};
        {
            std::lock_guard<std::mutex> lk(g_pool_mu);
            auto it = g_live.find(p);
            if (it != g_live.end()) b = it->second;
        }
        if (b.bytes > 0 && b.bytes <= BUILD_SPARE_MAX) {
            g_build->spare.push_back(b);
            return;
        }
        (void)hipStreamSynchronize(g_build->stream);
    } else {
        (void)hipDeviceSynchronize();
    }
    device_free(p);
}

// ---- per-stream scratch ------------------------------------------------------------------------
static ScratchPool g_scratch;

static thread_local void* g_scope_p = nullptr;
static thread_local size_t g_scope_bytes = 0;

ScratchScope::ScratchScope(void* p, size_t bytes) : prev_p(g_scope_p), prev_bytes(g_scope_bytes) {
    g_scope_p = p;
    g_scope_bytes = bytes;
}
ScratchScope::~ScratchScope() {
    g_scope_p = prev_p;
    g_scope_bytes = prev_bytes;
}

static thread_local EpochEnd* g_epoch_end = nullptr;
EpochEnd::EpochEnd(const Room& r) : room(r) {
    if (room.any) g_epoch_end = this;
}
EpochEnd::~EpochEnd() {
    if (g_epoch_end == this) g_epoch_end = nullptr;
}
EpochEnd* epoch_end() { return g_epoch_end; }

int ScratchLease::get(void** p, size_t bytes, hipStream_t s) {
    if (g_scope_p) {
        if (bytes > g_scope_bytes)
            return fail(GCN_ERR_WORKSPACE, "workspace scratch region has %zu bytes, %zu needed", g_scope_bytes, bytes);
        *p = g_scope_p;
        return GCN_OK;
    }
    int dev = 0;
    GCN_HIP_TRY(hipGetDevice(&dev));
    GCN_TRY(g_scratch.take(dev, s, bytes, &p_, [](void** q, size_t size) { return device_alloc(q, size); }));
    *p = p_;
    return GCN_OK;
}
ScratchLease::~ScratchLease() {
    if (p_) g_scratch.give(p_);
}

int grow_retire(gcn_csr* a, float** buf, size_t* have, size_t need) {
    if (need <= *have) return GCN_OK;
    void* fresh = nullptr;
    GCN_TRY(device_alloc(&fresh, need));
    if (*buf) a->retired.push_back(*buf);
    *buf = (float*)fresh;
    *have = need;
    return GCN_OK;
}

const DeviceInfo& device_info() {
    static std::mutex mu;
    static DeviceInfo info[64];
    static bool known[64] = {};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64) dev = 0;
    std::lock_guard<std::mutex> lk(mu);
    if (!known[dev]) {
        int cus = 0, l2 = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
        if (hipDeviceGetAttribute(&l2, hipDeviceAttributeL2CacheSize, dev) != hipSuccess || l2 <= 0) l2 = 4 << 20;
        info[dev] = {cus, (int64_t)l2};
        known[dev] = true;
    }
    return info[dev];
}

Config& config() {
    static Config c;
    return c;
}

int g_last_schedule = 0;

static std::atomic<int64_t> g_builds{0};
void count_build() { g_builds.fetch_add(1); }

// ---- event timing ---------------------------------------------------------------------------
struct TimedSpan { hipEvent_t a, b; int phase; };
static std::mutex g_time_mu;
static std::vector<TimedSpan> g_events;
static thread_local hipEvent_t g_open[GCN_PHASE_COUNT] = {};

void timing_begin(hipStream_t s, int phase) {
    if (!config().timing || g_open[phase]) return;
    hipEvent_t a;
    if (hipEventCreate(&a) != hipSuccess) return;
    (void)hipEventRecord(a, s);
    g_open[phase] = a;
}

void timing_end(hipStream_t s, int phase) {
    if (!g_open[phase]) return;
    hipEvent_t b;
    if (hipEventCreate(&b) != hipSuccess) {
        (void)hipEventDestroy(g_open[phase]);
        g_open[phase] = nullptr;
        return;
    }
    (void)hipEventRecord(b, s);
    std::lock_guard<std::mutex> lk(g_time_mu);
    g_events.push_back({g_open[phase], b, phase});
    g_open[phase] = nullptr;
}

void free_blocked(Blocked& b) {
    device_free(b.colidx);
    device_free(b.val);
    device_free(b.flags);
    device_free(b.sub_row);
    device_free(b.rp);
    device_free(b.fix_list);
    device_free(b.rq_ptr);
    device_free(b.rq_idx);
    b = Blocked();
}

void free_matrix(Matrix& m);

void free_sweep(Sweep& w) {
    device_free(w.colidx);
    device_free(w.val);
    device_free(w.lrow);
    device_free(w.task_base);
    device_free(w.task_len);
    device_free(w.task_order);
    if (w.heavy) {
        free_matrix(*w.heavy);
        delete w.heavy;
    }
    w = Sweep();
}

void free_hub(Hub& h) {
    device_free(h.hot_col);
    device_free(h.heavy_rows);
    device_free(h.defer);
    device_free(h.xhot);
    if (h.hot) { free_matrix(*h.hot); delete h.hot; }
    if (h.rest) { free_matrix(*h.rest); delete h.rest; }
    h = Hub();
}

void free_matrix(Matrix& m) {
    device_free(m.rowptr);
    device_free(m.colidx);
    device_free(m.val);
    device_free(m.flags);
    device_free(m.sub_row);
    device_free(m.ne_rows);
    device_free(m.ne_rowptr);
    device_free(m.empty_rows);
    device_free(m.short_col);
    device_free(m.fix_list);
    free_blocked(m.blk);
    free_sweep(m.swp);
    free_hub(m.hub);
    for (auto& b : m.blk_parked) free_blocked(b);
    for (auto& w : m.swp_parked) free_sweep(w);
    for (auto& h : m.hub_parked) free_hub(h);
    m = Matrix();
}

}  // namespace gcn

using namespace gcn;

// Up to four arrays copied by one launch, a workgroup per tile of 16-byte pieces, four loads of a thread in flight (eight: 4.2 TB/s); neither side is
// read again soon, hence the non-temporal forms.  Bound by memory.  A copy of the runtime's for each of the four, against this: two arrays of 2 M
// words, 8 and 4 MB 12.7 -> 7.4 us; of 34.6 M 114 -> 94 (6.2 TB/s); of 300 M 942 -> 781.
struct CopyArgs {
    static constexpr int THREADS = 256, PER = 4;
    struct Array {
        const uint4* src;
        uint4* dst;
        int64_t pieces;
        uint32_t words, first;                    // words behind the last whole piece; first of its workgroups
    } array[4];
    int count = 0;
    uint32_t blocks = 0;
    void add(void* dst, const void* src, size_t bytes) {
        array[count++] = Array{(const uint4*)src, (uint4*)dst, (int64_t)(bytes / 16), (uint32_t)(bytes % 16 / 4), blocks};
        blocks += (uint32_t)(bytes / 16 / (THREADS * PER)) + 1;
    }
};
__global__ __launch_bounds__(CopyArgs::THREADS) void k_copy_arrays(CopyArgs a) {
    constexpr int THREADS = CopyArgs::THREADS, PER = CopyArgs::PER;
    typedef uint32_t Piece __attribute__((ext_vector_type(4)));
    int k = 0;
    while (k + 1 < a.count && blockIdx.x >= a.array[k + 1].first) ++k;
    const CopyArgs::Array g = a.array[k];
    const Piece* const src = (const Piece*)g.src;
    Piece* const dst = (Piece*)g.dst;
    const int64_t at = (int64_t)(blockIdx.x - g.first) * (THREADS * PER) + threadIdx.x;
    Piece x[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (at + e * THREADS < g.pieces) x[e] = __builtin_nontemporal_load(src + at + e * THREADS);
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (at + e * THREADS < g.pieces) __builtin_nontemporal_store(x[e], dst + at + e * THREADS);
    if (at < g.words) ((uint32_t*)(dst + g.pieces))[at] = ((const uint32_t*)(src + g.pieces))[at];
}

// What kernel_copies asks of the runtime.
static MemoryOf memory_of(const void* p) {
    MemoryOf of;
    hipPointerAttribute_t what;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&what, p) != hipSuccess || what.type != hipMemoryTypeDevice ||
        hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
        (void)hipGetLastError();
        return of;
    }
    of.device = true;
    of.gpu = what.device;
    of.base = (uintptr_t)base;
    of.size = size;
    return of;
}
static int device_of(hipStream_t s) {
    if (!s) return current_device();
    hipDevice_t dev = -1;
    if (hipStreamGetDevice(s, &dev) != hipSuccess) (void)hipGetLastError();
    return (int)dev;
}

extern "C" {

const char* gcn_last_error(void) { return g_err; }
const char* gcn_version(void) { return "gcn-hip 0.1 (gfx950)"; }

int gcn_last_spmm_schedule(void) { return gcn::g_last_schedule; }

static int set_config(Config& c, int key, int value) {
    switch (key) {
        case GCN_CFG_SPMM_ALGO:
            if (value < 0 || value > 4) return fail(GCN_ERR_BADARG, "GCN_CFG_SPMM_ALGO must be 0, 1, 2, 3 or 4");
            c.spmm_algo = value;
            return GCN_OK;
        case GCN_CFG_SPMM_BLOCKS:
            if (value < 0 || value > (1 << 24)) return fail(GCN_ERR_BADARG, "GCN_CFG_SPMM_BLOCKS must be in [0, 2^24]");
            c.spmm_blocks = value;
            return GCN_OK;
        case GCN_CFG_SPLIT_LDS_KB:
            if (value != 0 && (value < 18 || value > 64)) return fail(GCN_ERR_BADARG, "GCN_CFG_SPLIT_LDS_KB must be 0 or in [18, 64]");
            c.split_lds_kb = value;
            return GCN_OK;
        case GCN_CFG_SWEEP_WAVES:
            if (value < 1 || value > 18) return fail(GCN_ERR_BADARG, "GCN_CFG_SWEEP_WAVES must be in [1, 18]");
            c.sweep_waves = value;
            return GCN_OK;
        case GCN_CFG_SWEEP_HEAVY:
            if (value < 1) return fail(GCN_ERR_BADARG, "GCN_CFG_SWEEP_HEAVY must be at least 1");
            c.sweep_heavy = value;
            return GCN_OK;
        case GCN_CFG_HUB_MB:
            if (value < 1 || value > 4096) return fail(GCN_ERR_BADARG, "GCN_CFG_HUB_MB must be in [1, 4096]");
            c.hub_mb = value;
            return GCN_OK;
        case GCN_CFG_HUB_BLOCK_COLS:
            if (value < 0 || (value % 64) != 0) return fail(GCN_ERR_BADARG, "GCN_CFG_HUB_BLOCK_COLS must be 0 or a multiple of 64");
            c.hub_block_cols = value;
            return GCN_OK;
        case GCN_CFG_HUB_DMIN:
            if (value < 1) return fail(GCN_ERR_BADARG, "GCN_CFG_HUB_DMIN must be at least 1");
            c.hub_dmin = value;
            return GCN_OK;
        case GCN_CFG_PATTERN_SPMM:
            if (value < 0 || value > 2) return fail(GCN_ERR_BADARG, "GCN_CFG_PATTERN_SPMM must be 0, 1 or 2");
            c.pattern_spmm = value;
            return GCN_OK;
        case GCN_CFG_FUSED_LAST_LAYER:
            if (value < 0 || value > 2) return fail(GCN_ERR_BADARG, "GCN_CFG_FUSED_LAST_LAYER must be 0, 1 or 2");
            c.fused_last = value;
            return GCN_OK;
        case GCN_CFG_TIMING:
            if (value != 0 && value != 1) return fail(GCN_ERR_BADARG, "GCN_CFG_TIMING must be 0 or 1");
            c.timing = value;
            return GCN_OK;
        default:
            return fail(GCN_ERR_BADARG, "unknown config key %d", key);
    }
}

int gcn_config(int key, int value) { return set_config(config(), key, value); }

int gcn_csr_config(gcn_csr* a, int key, int value) {
    if (!a) return fail(GCN_ERR_BADARG, "gcn_csr_config: NULL matrix");
    if (key == GCN_CFG_TIMING) return fail(GCN_ERR_BADARG, "gcn_csr_config: GCN_CFG_TIMING is process-wide (gcn_config)");
    if (!a->own_cfg) {               // from now on this matrix no longer follows gcn_config
        a->cfg = config();
        a->own_cfg = true;
    }
    return set_config(a->cfg, key, value);
}

int gcn_timing_read_phases(int64_t* spans, double* total_ms) {
    if (!spans || !total_ms) return fail(GCN_ERR_BADARG, "gcn_timing_read_phases: NULL output");
    std::lock_guard<std::mutex> lk(g_time_mu);
    for (int p = 0; p < GCN_PHASE_COUNT; ++p) { spans[p] = 0; total_ms[p] = 0.0; }
    int rc = GCN_OK;
    for (auto& ev : g_events) {
        float t = 0.f;
        hipError_t e = hipEventSynchronize(ev.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&t, ev.a, ev.b);
        if (e == hipSuccess) {
            total_ms[ev.phase] += t;
            spans[ev.phase] += 1;
        } else {
            rc = fail(GCN_ERR_HIP, "event timing failed: %s", hipGetErrorString(e));
        }
        (void)hipEventDestroy(ev.a);
        (void)hipEventDestroy(ev.b);
    }
    g_events.clear();
    return rc;
}

int gcn_timing_read(int64_t* launches, double* total_ms) {
    if (!launches || !total_ms) return fail(GCN_ERR_BADARG, "gcn_timing_read: NULL output");
    int64_t spans[GCN_PHASE_COUNT];
    double ms[GCN_PHASE_COUNT];
    const int rc = gcn_timing_read_phases(spans, ms);
    *launches = spans[GCN_PHASE_SPMM_KERNEL];
    *total_ms = ms[GCN_PHASE_SPMM_KERNEL];
    return rc;
}

int gcn_csr_destroy(gcn_csr* a) {
    if (!a) return GCN_OK;
    // what the matrix owns is given back to be used again: nothing queued on its device may still need it
    const int dev = current_device();
    if (dev != a->device) (void)hipSetDevice(a->device);
    (void)hipDeviceSynchronize();
    if (dev != a->device) (void)hipSetDevice(dev);
    free_matrix(a->A);
    if (!a->symmetric) free_matrix(a->At);
    device_free(a->carry2);
    device_free(a->deg);
    device_free(a->inv_sqrt_deg);
    device_free(a->carry);
    device_free(a->partial);
    device_free(a->xs);
    for (void* p : a->retired) device_free(p);
    delete a;
    return GCN_OK;
}

int gcn_scratch_release(void) {
    GCN_HIP_TRY(hipDeviceSynchronize());
    g_scratch.clear([](void* p) { device_free(p); });
    device_pool_release();
    return GCN_OK;
}

int64_t gcn_build_count(void) { return g_builds.load(); }

int gcn_csr_last_spmm_schedule(const gcn_csr* a) { return a ? a->last_schedule : 0; }

int gcn_csr_info(const gcn_csr* a, int64_t* n, int64_t* nnz, int32_t* max_degree) {
    if (!a) return fail(GCN_ERR_BADARG, "gcn_csr_info: NULL matrix");
    if (n) *n = a->n;
    if (nnz) *nnz = a->nnz;
    if (max_degree) *max_degree = a->A.max_degree;
    return GCN_OK;
}

int gcn_csr_shape(const gcn_csr* a, int64_t* n_rows, int64_t* n_cols) {
    if (!a) return fail(GCN_ERR_BADARG, "gcn_csr_shape: NULL matrix");
    if (n_rows) *n_rows = a->n;
    if (n_cols) *n_cols = a->ncols;
    return GCN_OK;
}

int gcn_csr_arrays(const gcn_csr* a, int transposed, const int64_t** rowptr, const int32_t** colidx,
                   const float** val, const int32_t** deg) {
    if (!a) return fail(GCN_ERR_BADARG, "gcn_csr_arrays: NULL matrix");
    if (transposed && !a->has_t) return fail(GCN_ERR_NOTRANSPOSE, "matrix was built without GCN_BUILD_TRANSPOSE");
    const Matrix& m = matrix_of(a, transposed);
    if (rowptr) *rowptr = m.rowptr;
    if (colidx) *colidx = m.colidx;
    if (val) *val = m.val;
    if (deg) *deg = a->deg;
    return GCN_OK;
}

int gcn_csr_export(const gcn_csr* a, int transposed, int64_t* rowptr, int32_t* colidx, float* val, int32_t* deg,
                   void* stream) {
    if (!a) return fail(GCN_ERR_BADARG, "gcn_csr_export: NULL matrix");
    if (transposed && !a->has_t) return fail(GCN_ERR_NOTRANSPOSE, "matrix was built without GCN_BUILD_TRANSPOSE");
    const Matrix& m = matrix_of(a, transposed);
    hipStream_t s = (hipStream_t)stream;
    const int current = current_device(), runs_on = device_of(s);
    CopyArgs copy;
    auto add = [&](void* dst, const void* src, size_t bytes) -> int {
        if (!dst || !bytes) return GCN_OK;
        const uintptr_t to = (uintptr_t)dst;                    // (the runtime is asked only where it matters)
        if (to % 16 == 0 && kernel_copies(a->device, current, runs_on, memory_of(dst), to, bytes)) copy.add(dst, src, bytes);
        else GCN_HIP_TRY(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s));
        return GCN_OK;
    };
    GCN_TRY(add(rowptr, m.rowptr, ((size_t)m.nrows + 1) * sizeof(int64_t)));
    GCN_TRY(add(colidx, m.colidx, (size_t)a->nnz * sizeof(int32_t)));
    GCN_TRY(add(val, m.val, (size_t)a->nnz * sizeof(float)));
    GCN_TRY(add(deg, a->deg, (size_t)a->n * sizeof(int32_t)));
    if (copy.count) {
        hipLaunchKernelGGL(k_copy_arrays, dim3(copy.blocks), dim3(CopyArgs::THREADS), 0, s, copy);
        GCN_LAUNCH_CHECK();
    }
    return GCN_OK;
}

}  // extern "C"
