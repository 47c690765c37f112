// Internal declarations shared by the translation units of libgcn_hip.so (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include <string>
#include <vector>

#include "epoch_layout.h"
#include "gcn.h"
#include "largest_asked.h"
#include "spmm_cost.h"

namespace gcn {

// 16 bytes at any 4-byte aligned address: the same instruction as for an aligned one, so one kernel serves every width
// and leading dimension.
struct __attribute__((packed, aligned(4))) f4u { float x, y, z, w; };

// Thread-local error text returned by gcn_last_error().
void set_error(const char* fmt, ...);
int fail(int code, const char* fmt, ...);

#define GCN_HIP_TRY(expr)                                                                       \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess)                                                                   \
            return gcn::fail(e_ == hipErrorOutOfMemory ? GCN_ERR_OOM : GCN_ERR_HIP,             \
                             "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__,   \
                             __LINE__);                                                         \
    } while (0)

#define GCN_TRY(expr)          \
    do {                       \
        int rc_ = (expr);      \
        if (rc_ != GCN_OK) return rc_; \
    } while (0)

// Launch check: a bad configuration is reported by hipGetLastError right after the launch.
#define GCN_LAUNCH_CHECK()                                                                      \
    do {                                                                                        \
        hipError_t e_ = hipGetLastError();                                                      \
        if (e_ != hipSuccess)                                                                   \
            return gcn::fail(GCN_ERR_HIP, "kernel launch failed: %s (%s:%d)",                   \
                             hipGetErrorString(e_), __FILE__, __LINE__);                        \
    } while (0)

// Nonzero-split schedule constants: a wavefront owns CHUNK consecutive stored entries, cut into
// SUB-entry pieces that each carry one 32-bit word of row-start flags.
constexpr int SUB = 32;
constexpr int CHUNK = 512;
constexpr int SUBS_PER_CHUNK = CHUNK / SUB;
// Rows of up to SHORT_ROW entries, as many as k_spmm_short takes at any width (SHORT_LANES lanes at two per row; see short_rows).
constexpr int SHORT_ROW = 64;
constexpr int64_t SHORT_LANES = 256 * 8 * 64;
// Matrices of fewer entries keep the schedule of the sizes.
constexpr int64_t PLANNED_NNZ = 1 << 20;

// Column-blocked copy of a matrix: the entries re-sorted by (column block, row, column).  Each
// non-empty (block, row) pair is a row of a partial-result matrix P; the SpMM kernel runs over this
// order unchanged, so all wavefronts gather from one block of X at a time and that block stays in
// L2.  A second kernel adds each row's partials in ascending block order.
struct Blocked {
    int64_t cols_per_block = 0;
    int32_t nblocks = 0;
    int64_t nrows = 0;           // R: non-empty (block, row) pairs
    int32_t* colidx = nullptr;   // [nnz]
    float* val = nullptr;        // [nnz]
    uint32_t* flags = nullptr;   // [nsub + pad]
    int32_t* sub_row = nullptr;  // [nsub + pad]
    int64_t* rp = nullptr;       // [R+1] first entry of each partial row
    int4* fix_list = nullptr;    // [n_fix] the rows that cross chunks (see build_fix_list)
    int64_t n_fix = 0, n_fix_long = 0;   // the first n_fix_long of them cover a whole further chunk
    int64_t* rq_ptr = nullptr;   // [n+1]  row i owns partial rows rq_idx[rq_ptr[i] .. rq_ptr[i+1])
    int32_t* rq_idx = nullptr;   // [R]    ascending block order inside a row
};

struct Matrix;

// The sweep kernel: tasks (wavefronts) of a workgroup, which takes a compute unit, and the steps that a lane group works through in
// one trip.  The entries of a trip lie group by group, so that neighbouring lanes fetch a group's entries.
constexpr int SWEEP_TASKS = 5;
constexpr int SWEEP_STEPS = 8;

// Sweep copy of a matrix for operands far larger than the caches.  Rows are cut into tasks of
// `rb` consecutive rows; a wavefront owns a task, accumulates its rows in LDS and walks the task's
// entries in ascending column order, so all wavefronts of a launch (started together, equal length)
// gather from one narrow band of X at a time and that band stays in L2.  The entries of a task are
// stored in steps of `groups` entries, those of two steps all of different rows (packed that way when the copy is
// built, an entry whose row is already there moving to one of the next pairs), so the lane groups of
// two steps add to LDS without any conflict.  Padding entries name the row behind the task's last.  Rows longer than
// `heavy_threshold` are kept apart and go through the nonzero-split kernel.
struct Sweep {
    int32_t groups = 0;
    int32_t rb = 0;
    int32_t heavy_threshold = 0;
    int64_t ntasks = 0, nnz_light = 0, nnz_heavy = 0, n_heavy = 0;
    int64_t padded = 0;           // entries stored, padding included
    bool built = false;           // or counted only and found to be sparser than was asked for
    bool sparser(double most) const { return most > 0 && (double)padded > most * (double)nnz_light; }
    int32_t* colidx = nullptr;    // [padded] column
    float* val = nullptr;         // [padded]
    uint16_t* lrow = nullptr;     // [padded] row inside the task, rb for a padding entry
    int64_t* task_base = nullptr; // [ntasks] first stored entry of the task (a multiple of SWEEP_STEPS * groups)
    int32_t* task_len = nullptr;  // [ntasks] stored entries of the task (as above)
    int32_t* task_order = nullptr;// [ntasks] task ids, longest first
    Matrix* heavy = nullptr;      // the heavy rows as a row-subset matrix (ne_rows = their ids)
};

// Hub copy of a matrix with a skewed degree distribution: A = A_hot + A_rest, where A_hot holds the
// entries of long rows (at least `dmin` entries) whose column is one of the `H` columns with the most
// entries, and A_rest everything else.  The rows of X that the hot columns select are packed, in
// descending order of column length, into a buffer of their own at every product; A_hot runs over it
// in column blocks that stay in one L2 each (every XCD works on its own blocks), A_rest runs over X
// unchanged, and the partial rows of A_hot are added to the rows that A_rest wrote.
struct Hub {
    int state = 0;                // 0 not tried, 1 built, -1 tried and rejected (not skewed enough)
    int64_t H = 0, cpb = 0;       // hot columns, columns per block (H is a multiple of cpb)
    int32_t dmin = 0;
    int32_t cfg_mb = 0, cfg_block_cols = 0;   // settings at build time: a change of settings rebuilds, a change of f does not
    int64_t nnz_hot = 0, nnz_rest = 0, n_heavy = 0;
    int32_t* hot_col = nullptr;   // [H] position in the packed buffer -> column
    int32_t* heavy_rows = nullptr;// [n_heavy] the long rows, ascending
    uint8_t* defer = nullptr;     // [nrows] 1 for a long row: A_rest stores its sum raw, A_hot's pass finishes it
    Matrix* hot = nullptr;        // n_heavy x H, column = position in the packed buffer
    Matrix* rest = nullptr;       // nrows x ncols
    float* xhot = nullptr;        // [H][f] packed rows of X, grown on demand
    size_t xhot_bytes = 0;
};

// One stored matrix in compressed rows plus its nonzero-split schedule.
struct Matrix {
    int64_t nrows = 0, ncols = 0;
    int64_t* rowptr = nullptr;   // [nrows+1]
    int32_t* colidx = nullptr;   // [nnz]
    float* val = nullptr;        // [nnz]
    // schedule (built once at creation)
    uint32_t* flags = nullptr;   // [nsub]  bit b of word j: entry 32j+b is the first of its row
    int32_t* sub_row = nullptr;  // [nsub]  index (among non-empty rows) of the row holding entry 32j
    int32_t* ne_rows = nullptr;  // [n_ne]  non-empty row index -> row, or NULL when no row is empty
    int64_t* ne_rowptr = nullptr;// [n_ne+1] rowptr restricted to non-empty rows, or NULL (= rowptr)
    int32_t* empty_rows = nullptr;// [nrows - n_ne] the rows without entries, or NULL when there are none
    int64_t n_ne = 0;
    int4* fix_list = nullptr;    // [n_fix] the rows that cross chunks (see build_fix_list)
    int64_t n_fix = 0, n_fix_long = 0;   // the first n_fix_long of them cover a whole further chunk
    int64_t nsub = 0, nchunks = 0;
    int32_t max_degree = 0;
    Lengths lengths;             // of its rows (not kept for the long rows of a sweep copy)
    RowOrder order;              // how they lie (likewise)
    Terms terms = Terms::UNKNOWN;
    std::vector<SpmmPlan> plans; // schedules chosen so far, one per width and kind of terms
    // Rows of equal pitch for the kernel of few and short rows (see build_short), or NULL.
    int32_t* short_col = nullptr;   // [nrows][short_pitch] columns, 0 behind a row's last; the other two are of the same allocation
    float* short_val = nullptr;     // likewise
    int32_t* short_rows = nullptr;  // [nrows] entries of the row, and where they begin modulo CHUNK from bit 16 up
    int32_t short_pitch = 0;
    // Other stored orders of the matrix, built on first use (or by a prepare call) and kept until the
    // matrix is destroyed.  blk / swp / hub are the copies the latest product used; a product that needs
    // another key (block width; lane groups, task height and long-row threshold; hub settings) parks the
    // current copy in the list beside it and takes the matching one from there, or builds it.  Nothing is
    // freed before destroy, so kernels already queued (or captured in a HIP graph) keep valid pointers.
    Blocked blk;
    Sweep swp;
    Hub hub;
    std::vector<Blocked> blk_parked;
    std::vector<Sweep> swp_parked;
    std::vector<Hub> hub_parked;
};

struct Config {
    int spmm_algo = 0;
    int spmm_blocks = 0;
    int sweep_heavy = 1024;
    int split_lds_kb = 0;        // nonzero-split kernels with 16 lane groups: LDS per workgroup incl. padding (0: see occupancy_pad)
    int sweep_waves = 9;
    int hub_mb = 32;             // hub schedule: size of the packed buffer of hot rows of X, MB
    int hub_block_cols = 0;      // hub schedule: columns per block (0: about 2 MB of the gathered panel)
    int hub_dmin = 64;           // hub schedule: rows with at least this many entries are long rows
    int pattern_spmm = 2;        // epoch: value-free SpMM for symmetric normalisation (0 never, 1 always, 2 by row length)
    int fused_last = 1;          // epoch: fused last layer (0 off, 1 on without storing Z^L and G^L, 2 on and stored)
    int timing = 0;
};

}  // namespace gcn

struct gcn_csr {
    int64_t n = 0, ncols = 0, nnz = 0;   // A is n x ncols (square unless made by gcn_csr_create_from_csr_rect)
    int device = 0;
    bool has_t = false;
    bool symmetric = false;      // A^T is A, entry by entry and value by value: At is not used, A serves both
    gcn::Matrix A, At;
    int32_t* deg = nullptr;      // [n] entries per row of A
    float* inv_sqrt_deg = nullptr; // [n] (float)(1/sqrt(deg)); set only when this library normalised the matrix
                                 // symmetrically, i.e. val_ij == 1/sqrt(deg_i deg_j) for every stored entry
    float* carry = nullptr;      // per-chunk partial rows for the nonzero-split SpMM
    size_t carry_bytes = 0;
    float* carry2 = nullptr;     // the same for the second matrix of a paired launch
    size_t carry2_bytes = 0;
    float* partial = nullptr;    // P of the column-blocked SpMM
    size_t partial_bytes = 0;
    float* xs = nullptr;         // operand of gcn_spmm with its rows pre-scaled (value-free form)
    size_t xs_bytes = 0;
    std::vector<void*> retired;  // buffers replaced by larger ones: kept until destroy (queued or captured work may use them)
    bool own_cfg = false;        // set by gcn_csr_config: this matrix has settings of its own
    gcn::Config cfg;             // valid when own_cfg
    int last_schedule = 0;       // GCN_SCHED_* of the latest product on this matrix
};

namespace gcn {

// Device memory of the library.  Blocks that are given back are kept for the next matrix, so that building one does not
// pay for mapping and clearing memory each time (a graph of 16 M pairs: 5 of 14 ms, and up to 40 ms more when other
// memory of the process had just been released): at most 1/64 of the device's memory, the oldest leave first,
// everything leaves when an allocation fails and in gcn_scratch_release.  device_free may only be called when no
// queued work uses the block any more, on any stream.
int device_alloc(void** p, size_t bytes);
template <typename T>
int device_alloc_t(T** p, size_t count) { return device_alloc((void**)p, count * sizeof(T)); }
void device_free(void* p);
void device_pool_release();

// While one of these is alive on a thread, the temporaries of graph construction (TempBuf) that the thread allocates
// and drops are reused in stream order, without waiting; the destructor waits for the stream and gives them back.
// Every entry point that builds something opens one; an inner one joins the outer.
struct BuildScope {
    explicit BuildScope(hipStream_t s);
    ~BuildScope();
    bool owner;
};
int temp_alloc(void** p, size_t bytes);
void temp_free(void* p);
struct TempBuf {   // given back on scope exit
    void* p = nullptr;
    TempBuf() = default;
    TempBuf(const TempBuf&) = delete;
    TempBuf& operator=(const TempBuf&) = delete;
    ~TempBuf() { temp_free(p); }
    int alloc(size_t bytes) { temp_free(p); p = nullptr; return temp_alloc(&p, bytes ? bytes : 16); }
    void drop() { temp_free(p); p = nullptr; }
    template <typename T> T* as() const { return (T*)p; }
};

// Library-owned scratch for the split-K partial sums of the weight-gradient product, the column sums and the
// loss (see ScratchPool): the buffer is the call's from get() to the end of its scope, and no other call's.  It grows on demand; the
// buffers are kept until gcn_scratch_release.
class ScratchLease {
public:
    ScratchLease() = default;
    ScratchLease(const ScratchLease&) = delete;
    ScratchLease& operator=(const ScratchLease&) = delete;
    ~ScratchLease();
    int get(void** p, size_t bytes, hipStream_t s);
private:
    void* p_ = nullptr;
};
// While one of these is alive on a thread, leases of that thread are the given caller-owned
// buffer instead (GCN_ERR_WORKSPACE if it is too small): the epoch calls keep their partial sums in the
// caller's workspace.
struct ScratchScope {
    ScratchScope(void* p, size_t bytes);
    ~ScratchScope();
    void* prev_p;
    size_t prev_bytes;
};
// The additions that an epoch leaves to its end: the partial results of the weight gradients, those of the loss, and the update of the
// weights, all in one kernel.  While one of these is alive on a thread, the products and the loss that it has room for leave their
// partial results there (epoch_end); finish() adds them up in the order in which kernels of their own do.
struct EpochEnd {
    static constexpr int MOST = EpochRoom::MOST;
    struct Sum {                                  // Y (M x N) = the sum of `parts` partial results, each M x N, or N x M when transposed
        const float* part;
        float* Y;
        float* W;                                 // W -= lr Y, or NULL
        int32_t M, N, parts, transposed, first;   // first: of its workgroups
    };
    struct Fused {                                // partial results of the fused last layer (see k_fused_y)
        const float* part = nullptr;
        float* Y = nullptr;
        float* W = nullptr;
        int32_t C = 0, CP = 0, blocks = 0, first = 0;
    };
    struct Args {
        Sum sums[MOST];
        Fused fused;
        const double* lpart = nullptr;
        double inv_m = 0;
        float* loss = nullptr;
        int64_t lparts = 0;
        int32_t count = 0, loss_at = -1;
        float lr = 0;
    } args;
    struct Room {                                 // where the partial results lie: of the loss, of a bias gradient, of the layers' weight gradients
        void* loss = nullptr;
        void* bias = nullptr;
        void* grad[MOST] = {};
        bool few[MOST] = {};                      // shares of 64 rows (see few_rows)
        bool any = false;
    } room;
    float* W = nullptr;                           // of the layer whose gradient comes next
    int layer = 0;                                // and its number
    explicit EpochEnd(const Room& r);             // no room: everything as without it
    ~EpochEnd();
    void add(const float* part, float* Y, int32_t M, int32_t N, int parts, bool transposed) {
        args.sums[args.count++] = Sum{part, Y, W, M, N, (int32_t)parts, transposed ? 1 : 0, 0};
    }
    int finish(float lr, hipStream_t s);
};
EpochEnd* epoch_end();                            // the thread's, or NULL
// bytes of scratch that the column sums take
size_t colsum_scratch_bytes(int64_t rows, int32_t cols);

// Compute units and L2 size (one XCD's) of the current device, read once per device from the runtime.
struct DeviceInfo { int cus; int64_t l2_bytes; };
const DeviceInfo& device_info();
// op(A) as stored
inline Matrix& matrix_of(gcn_csr* a, int trans) { return (trans && !a->symmetric) ? a->At : a->A; }
inline const Matrix& matrix_of(const gcn_csr* a, int trans) { return (trans && !a->symmetric) ? a->At : a->A; }

Config& config();                               // the process-wide settings (gcn_config)
inline const Config& cfg_of(const gcn_csr* a) { return a->own_cfg ? a->cfg : config(); }
// schedule taken by the most recent sparse product of this process (GCN_SCHED_*), for tests and reports
extern int g_last_schedule;
void count_build();                             // one stored order has been built (gcn_build_count)

// event bracketing of the dominant kernel (GCN_CFG_TIMING)
void timing_begin(hipStream_t s, int phase = GCN_PHASE_SPMM_KERNEL);
void timing_end(hipStream_t s, int phase = GCN_PHASE_SPMM_KERNEL);
// brackets a scope of host code (all kernels it queues on `s`) under one phase
struct PhaseTimer {
    hipStream_t s;
    int phase;
    PhaseTimer(hipStream_t s_, int phase_) : s(s_), phase(phase_) { timing_begin(s, phase); }
    ~PhaseTimer() { timing_end(s, phase); }
};

// Launches a kernel with dynamic LDS.  More than 64 KB per workgroup (static part included) has to be asked for, once
// per kernel, device and larger size.  A request that fails is made again by the next launch, and reported by the
// launch check.
template <auto Kernel, typename... Args>
void launch_lds(dim3 grid, int threads, size_t lds, hipStream_t s, const Args&... args) {
    if (lds > 44 * 1024) {
        static LargestAsked asked[64];
        int dev = 0;
        (void)hipGetDevice(&dev);
        asked[dev & 63].reach(lds, [](size_t bytes) {
            return hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
        });
    }
    hipLaunchKernelGGL(Kernel, grid, dim3(threads), lds, s, args...);
}

int build_short(Matrix& m, int64_t nnz, hipStream_t s);       // once the values are there
int build_schedule(Matrix& m, int64_t n, int64_t nnz, hipStream_t s, int32_t* deg = nullptr);   // deg: also receives the row lengths
// One record per row whose entries run on into further chunks: x, y = the first and the last of them, z = the row (its
// index among the non-empty rows).  Rows that leave no row start in chunk x come first (n_long of them).
int build_fix_list(const uint32_t* flags, const int32_t* sub_row, const int64_t* rp, int64_t nnz, int4** list,
                   int64_t* count, int64_t* n_long, hipStream_t s);
int build_blocked(Matrix& m, int64_t nnz, int64_t cols_per_block, hipStream_t s);
// make m.blk / m.swp the copy with the given key: the current one, a parked one, or a newly built one
int want_blocked(Matrix& m, int64_t nnz, int64_t cols_per_block, hipStream_t s);
// most > 0: a copy that would store more than `most` places per entry (see Sweep::sparser) is not built
int want_sweep(Matrix& m, int64_t nnz, int32_t groups, int32_t rb, int32_t heavy_threshold, double most, hipStream_t s);
void free_blocked(Blocked& b);
int build_sweep(Matrix& m, int64_t nnz, int32_t groups, int32_t rb, int32_t heavy_threshold, double most, hipStream_t s);
void free_sweep(Sweep& w);
int build_hub(Matrix& m, int64_t nnz, int64_t H, int64_t cpb, int32_t dmin, hipStream_t s);
void free_hub(Hub& h);
void free_matrix(Matrix& m);

// Variants of the sparse product: `pattern` ignores the stored values (every entry counts as 1),
// `row_scale` multiplies output row i by row_scale[i] before the epilogue.
// What a layer does with its product: Z = product + bias, and ReLU in place or into H (rows as far apart as those of Z).  Some of the
// schedules do it where they store a row and set `done`; behind the others it is a pass of its own.
static constexpr int EPI_LAYER = 3;       // internal epilogue, beside GCN_EPI_*
struct LayerEnd {
    const float* bias = nullptr;
    float* H = nullptr;
    bool relu = false;                    // in place
    bool done = false;
};
// What an epoch does next with the rows of a product: T = Z op(W) in front of the next sparse product, masked where that is Equation 2's, or
// the loss.  The kernel of few and short rows does it where the rows are made and sets `done` (see next_of); behind the others it
// is a launch of its own.
struct RowsNext {
    enum Kind { NONE = 0, GEMM = 1, LOSS = 2, GRAD = 4 };
    int kind = NONE;                      // GEMM, LOSS, GRAD or GEMM | GRAD
    const float* W = nullptr;             // f x N, or N x f when transposed
    int32_t N = 0, transposed = 0;
    float* T = nullptr;                   // n x N
    const float* mask = nullptr;          // NULL, or n x N: T where it is positive
    const int32_t* labels = nullptr;      // loss: as gcn_softmax_nll_masked takes them
    float* G = nullptr;                   // n x f
    double* part = nullptr;               // a partial sum of every 16 rows
    float inv_m = 0;
    const float* H = nullptr;             // gradient: the partial results of H^T Z, H n x M, as the launch of its own leaves them: of every
    int64_t ldh = 0;                      // 64 rows one of M x f
    int32_t M = 0;
    float* ypart = nullptr;
    bool done = false;
};
// The weight gradient H^T Z (M x f, over n rows) of the EpochEnd's layer as what is next to the rows of Z: whether a kernel of them can leave its partial
// results; gradient_made says that they lie there.
bool gradient_next(RowsNext& next, int64_t n, int32_t f, const float* H, int64_t ldh, int32_t M);
void gradient_made(const RowsNext& next, int64_t n, int32_t f, float* Y);
// The loss of an epoch as what is next to a product of C columns, whose `parts` partial sums lie in the EpochEnd's room (NONE: it has to be a launch of
// its own); loss_made says that they do.
RowsNext loss_next(int32_t C, int64_t parts, const int32_t* labels, int64_t n_labelled, float* G);
void loss_made(int64_t parts, int64_t n_labelled, float* loss);
struct SpmmOpt {
    bool pattern = false;
    const float* row_scale = nullptr;
    bool any_order = false;           // no ReLU decides on the result: a faster kernel may add a row's terms in another order
    // Another schedule may add the terms in another order: also set for the stand-alone products A X, and A^T X with a mask (of
    // widths that are a multiple of four, see free_schedule).  The forward products A^T X, on whose sums a ReLU decides, keep one
    // schedule, chosen by sizes alone: where a sum is zero to rounding another order puts it on the other side, and every
    // such element moves the gradient of the weights by 1e-4 of its norm.
    bool any_schedule = false;
    LayerEnd* end = nullptr;          // only with the epilogue GCN_EPI_NONE
    RowsNext* next = nullptr;
    bool narrow = false;              // internal, see SpmmPlan::narrow
    // internal to the hub schedule:
    const uint8_t* defer = nullptr;   // rows whose sum is stored raw (no scale, no epilogue)
    bool accumulate = false;          // column-blocked reduce adds to what Z already holds
    // prepare / describe:
    bool dry = false;                 // build the stored order and size the buffers, launch nothing
    std::string* describe = nullptr;  // receives the schedule and its launch shape as text
};
int scale_rows_launch(int64_t rows, int32_t cols, const float* X, int64_t ldx, const float* scale, float* Y, int64_t ldy,
                      hipStream_t s);
// whether products with this matrix take the value-free form (GCN_CFG_PATTERN_SPMM and the matrix's own shape)
bool use_value_free(const gcn_csr* a);
int inv_sqrt_deg_launch(int64_t n, const int32_t* deg, float* out, hipStream_t s);
int spmm_launch(gcn_csr* a, Matrix& m, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s, const SpmmOpt& o = SpmmOpt());
// builds the stored order and sizes the handle's buffers that spmm_launch would need for width f (16-byte
// aligned operands with leading dimensions that are multiples of 4 assumed), without running the product
int spmm_prepare(gcn_csr* a, Matrix& m, int32_t f, hipStream_t s, bool any_schedule, bool pattern = false);
// grows one of the handle's buffers; the replaced buffer is retired, not freed
int grow_retire(gcn_csr* a, float** buf, size_t* have, size_t need);

// `row_scale` (optional): row i of C is multiplied by row_scale[i] after bias and epilogue
int gemm_back_launch(int64_t n, int32_t f_in, int32_t f_out, const float* Hin, int64_t ldh, const float* S, const float* W,
                     const float* Zprev, float* Y, float* Gprev, bool few, hipStream_t s, bool* handled);
// `few`: a product with ta = 1 is cut into shares of 64 rows (see few_rows)
int gemm_launch(int ta, int tb, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                int64_t ldb, float* C, int64_t ldc, const float* bias, int epilogue, const float* Zprev,
                int64_t ldzprev, hipStream_t s, const float* row_scale = nullptr, bool few = false);
// the fused last layer of the epoch (f_in = 16, up to 256 classes)
int fused_last_launch(int64_t n, int32_t C, const float* T, const float* W, const int32_t* labels, int64_t n_labelled,
                      float* loss, float* Y, float* S, const float* s_scale, float* Zout, float* Gout, void* scratch,
                      hipStream_t s);
int colsum_launch(int64_t rows, int32_t cols, const float* G, int64_t ldg, float* out, hipStream_t s);
int update_launch(int32_t L, const int32_t* dims, float* const* W, float* const* Y, float lr, hipStream_t s);
int relu_launch(int64_t rows, int32_t cols, const float* Z, int64_t ldz, float* H, int64_t ldh, hipStream_t s);
// Z (dense rows) += 1 bias^T, then max(Z, 0) in place (relu) or, when H is given, into H
int bias_add_launch(int64_t rows, int32_t cols, float* Z, const float* bias, int relu, float* H, hipStream_t s);

}  // namespace gcn
