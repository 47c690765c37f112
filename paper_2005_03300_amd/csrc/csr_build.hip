// Graph construction on the GPU: cleaned entry set -> compressed rows, degrees, normalised
// values, the transposed matrix, and the nonzero-split schedule used by the SpMM kernel.
//
// Section "Graph Neural Networks" of the paper defines the matrix (self-connections added,
// D^-1/2 (A+I) D^-1/2); section "Communication Schemes and their Analyses" keeps both A and A^T
// so that neither product needs a transposition (or, here, floating-point atomics) at run time.
//
// Entries are encoded as 64-bit keys row<<cbits|col with cbits the bits of a column (so that the sort takes no pass over
// unused bits); their sort and the removal of equal neighbours yield the canonical row-major order with ascending columns.  Where
// the rows fall into buckets that a compute unit sorts, that is done by row_sort.h, otherwise by the device-wide sort and selection
// of prims.h.
#include <cstring>
#include <new>

#include "common.h"
#include "prims.h"
#include "build_util.h"
#include "launch_rules.h"
#include "row_sort.h"

namespace gcn {

// ---- kernels ---------------------------------------------------------------------------------

// The keys of the radix sort: one per stored direction of each input pair, then the diagonal.  A pair with u == v is dropped: with
// self loops its key is that of the diagonal entry, which exists anyway; without, it becomes the key n<<cbits, which sorts
// behind every real one.  The first pass of the sort reads the pairs themselves: a kernel that wrote the keys and one that checked
// the ids took 104 us for 16.8 M pairs, the pass takes 65 us longer than over written keys.  *bad is set where an id
// is outside [0, n), and nothing may be indexed by the keys then.
struct PairKeys {
    typedef uint64_t Key;
    const int32_t* src;
    const int32_t* dst;
    int64_t m, n;
    bool symmetrise, self_loops;
    unsigned cbits;
    int* bad;
    __device__ uint64_t operator()(size_t i, bool& wrong) const {
        const int64_t pairs = symmetrise ? 2 * m : m;
        if ((int64_t)i >= pairs) {
            const uint64_t v = (uint64_t)((int64_t)i - pairs);
            return v << cbits | v;
        }
        const int64_t t = symmetrise ? (int64_t)(i >> 1) : (int64_t)i;
        const uint64_t u = (uint32_t)src[t], v = (uint32_t)dst[t];
        wrong |= u >= (uint64_t)n || v >= (uint64_t)n;
        if (u == v && !self_loops) return (uint64_t)n << cbits;
        return symmetrise && (i & 1) ? (v << cbits | u) : (u << cbits | v);
    }
    __device__ void report() const { *bad = 1; }
};

// The first key of every run of equal ones becomes an entry: its column, the row pointers of the rows it opens (all those after
// the row of the key before it) and, where they are wanted, the key itself.  Keys of row n (dropped pairs) open the rows
// that are left and are no entry.
struct EmitEntry {
    const uint64_t* in;
    int64_t n;                   // rows
    unsigned cbits;
    int64_t* rowptr;
    int32_t* colidx;
    uint64_t* keys;              // or NULL
    __device__ void operator()(int64_t i, int64_t pos) const {
        const uint64_t key = in[i];
        const int64_t r = (int64_t)(key >> cbits);
        for (int64_t q = i > 0 ? (int64_t)(in[i - 1] >> cbits) + 1 : 0; q <= r; ++q) rowptr[q] = pos;
        if (r >= n) return;
        colidx[pos] = (int32_t)(key & ((1ull << cbits) - 1));
        if (keys) keys[pos] = key;
    }
};

// What the host has to know after the sort, in one copy (three copies that each wait for the stream took 60 us).
struct SortResult {
    int64_t kept;
    uint64_t last;
    int32_t bad;
};
__global__ void k_sort_result(const int64_t* __restrict__ kept, const uint64_t* __restrict__ last, const int* __restrict__ bad,
                              SortResult* __restrict__ out) {
    *out = SortResult{*kept, *last, *bad};
}

// Closes the rows behind the last key's.
__global__ __launch_bounds__(256) void k_close_rows(int64_t n, int64_t nnz, const uint64_t* __restrict__ last, unsigned cbits,
                                                    int64_t* __restrict__ rowptr) {
    const int64_t from = last ? (int64_t)(*last >> cbits) + 1 : 0;
    for (int64_t q = from + (int64_t)blockIdx.x * 256 + threadIdx.x; q <= n; q += (int64_t)gridDim.x * 256) rowptr[q] = nnz;
}

// A fixed number of workgroups strides over the rows, so that there are few atomics on the two counters (one per
// wavefront of 64 rows took 385 us on a million rows, nearly all of it waiting for the counters' one address).
struct DegreeSums {
    int32_t max_deg, pad;
    unsigned long long n_nonempty;
    unsigned long long rows[Lengths::BINS], entries[Lengths::BINS];        // as in Lengths
    unsigned long long sum, squares;                                       // as in RowOrder
    unsigned ones[RowOrder::WINDOWS];
};

// The columns of a window of entries (see RowOrder), each of them one bit of a table: how many bits get set.  A workgroup per window,
// 2^18 bits for 2^15 entries, eight loads in flight.  nnz >= RowOrder::STRETCH.  (34 M entries: 9 us of 1.3 ms of construction.)
__global__ __launch_bounds__(1024) void k_sample_columns(int64_t nnz, const int32_t* __restrict__ colidx, unsigned* __restrict__ ones) {
    constexpr int WORDS = (1 << RowOrder::BITS) / 32, LOADS = RowOrder::WINDOW / 4 / 1024, AT_ONCE = 1024 * 4 / RowOrder::GROUP_ENTRIES;
    __shared__ unsigned s_bits[WORDS];
    __shared__ unsigned s_ones;
    const int64_t first = ((nnz - RowOrder::STRETCH) / (RowOrder::WINDOWS - 1) * blockIdx.x) & ~3ll;
    const int per = 1024 / AT_ONCE, group = (int)threadIdx.x / per, at = (int)threadIdx.x % per;
    int4 c[LOADS];
#pragma unroll
    for (int p = 0; p < LOADS; ++p)
        c[p] = *reinterpret_cast<const int4*>(colidx + first + (int64_t)(p * AT_ONCE + group) * (RowOrder::APART * RowOrder::GROUP_ENTRIES) + 4 * at);
    for (int w = threadIdx.x; w < WORDS; w += 1024) s_bits[w] = 0;
    if (threadIdx.x == 0) s_ones = 0;
    __syncthreads();
    auto set = [&](int32_t column) {
        const uint32_t b = RowOrder::bit_of((uint32_t)column);
        atomicOr(&s_bits[b / 32], 1u << b % 32);
    };
#pragma unroll
    for (int p = 0; p < LOADS; ++p) { set(c[p].x); set(c[p].y); set(c[p].z); set(c[p].w); }
    __syncthreads();
    unsigned n = 0;
    for (int w = threadIdx.x; w < WORDS; w += 1024) n += __popc(s_bits[w]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_ones, n);
    __syncthreads();
    if (threadIdx.x == 0) ones[blockIdx.x] = s_ones;
}

// As few workgroups as keep the loads going: each of them ends with up to 70 additions to counters that all share (1 M rows, 512 workgroups of
// 256: 27 us; 128 of 1024: 17).
constexpr int DEGREE_THREADS = 1024;
__global__ __launch_bounds__(DEGREE_THREADS) void k_degrees(int64_t n, const int64_t* __restrict__ rowptr, int32_t* __restrict__ deg,
                                                 DegreeSums* __restrict__ sums) {
    __shared__ unsigned s_rows[Lengths::BINS];
    __shared__ unsigned long long s_entries[Lengths::BINS];
    if (threadIdx.x < Lengths::BINS) { s_rows[threadIdx.x] = 0; s_entries[threadIdx.x] = 0; }
    __syncthreads();
    int32_t m = 0;
    unsigned nz = 0;
    unsigned long long sum = 0, squares = 0;
    for (int64_t first = (int64_t)blockIdx.x * DEGREE_THREADS; first < n; first += (int64_t)gridDim.x * DEGREE_THREADS) {
        const int64_t i = first + threadIdx.x;
        int32_t d = 0;
        if (i < n) {
            d = (int32_t)(rowptr[i + 1] - rowptr[i]);
            if (deg) deg[i] = d;
        }
        m = d > m ? d : m;
        nz += d > 0;
        if (d > 0) {
            const int b = 31 - __clz(d);
            atomicAdd(&s_rows[b], 1u);
            atomicAdd(&s_entries[b], (unsigned long long)d);
        }
        unsigned group = d < RowOrder::LONG ? d : RowOrder::LONG;      // 64 rows: a wavefront's
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) group += __shfl_xor(group, s, 64);
        sum += group;
        squares += (unsigned long long)group * group;
    }
    static_assert(RowOrder::GROUP == 64, "one wavefront");
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const int32_t o = __shfl_xor(m, s, 64);
        m = o > m ? o : m;
        nz += __shfl_xor(nz, s, 64);
    }
    __shared__ int32_t s_m[DEGREE_THREADS / 64];
    __shared__ unsigned s_nz[DEGREE_THREADS / 64];
    __shared__ unsigned long long s_sum[DEGREE_THREADS / 64], s_squares[DEGREE_THREADS / 64];
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        s_m[w] = m; s_nz[w] = nz; s_sum[w] = sum; s_squares[w] = squares;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < DEGREE_THREADS / 64; ++w) { m = s_m[w] > m ? s_m[w] : m; nz += s_nz[w]; sum += s_sum[w]; squares += s_squares[w]; }
        atomicMax(&sums->max_deg, m);
        if (nz) {
            atomicAdd(&sums->n_nonempty, (unsigned long long)nz);
            atomicAdd(&sums->sum, sum);
            atomicAdd(&sums->squares, squares);
        }
    }
    if (threadIdx.x < Lengths::BINS && s_rows[threadIdx.x]) {
        atomicAdd(&sums->rows[threadIdx.x], (unsigned long long)s_rows[threadIdx.x]);
        atomicAdd(&sums->entries[threadIdx.x], s_entries[threadIdx.x]);
    }
}
static unsigned degree_blocks(int64_t n) {
    const int64_t b = (n + DEGREE_THREADS - 1) / DEGREE_THREADS;
    return (unsigned)(b < 1 ? 1 : (b > 128 ? 128 : b));
}

// val(i,j) = (float)(1 / sqrt(d_i d_j)): exact integer product in double, correctly rounded
// square root and division, one rounding to float -- the same value on any IEEE machine.
// norm 2 is the row normalisation D^-1 (A+I): val(i,j) = (float)(1 / d_i).
// Four entries per thread; their rows follow from the schedule (the row of every 32nd entry and the flag of every row start), so
// that only the columns are read.  Bound by the gathers of the columns' degrees: 16 bits where the longest row allows it, so that an
// L2 holds the table.  34.3 M entries, 1 M rows: 231 us with an entry per thread and 8-byte keys, 204 this way with 32 bits, 179 with 16.
template <typename Degree>
__global__ __launch_bounds__(256) void k_values(int64_t nnz, const int32_t* __restrict__ colidx, const uint32_t* __restrict__ flags,
                                                const int32_t* __restrict__ sub_row, const int32_t* __restrict__ ne_rows,
                                                const Degree* __restrict__ deg, int norm, float* __restrict__ val) {
    const int64_t k0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (k0 >= nnz) return;
    const uint32_t word = flags[k0 / SUB] & ~1u;
    const int32_t first = sub_row[k0 / SUB];
    const int b0 = (int)(k0 % SUB), here = nnz - k0 < 4 ? (int)(nnz - k0) : 4;
    int32_t c[4], di[4], dj[4];
    if (here == 4) {
        const int4 cc = *reinterpret_cast<const int4*>(colidx + k0);
        c[0] = cc.x; c[1] = cc.y; c[2] = cc.z; c[3] = cc.w;
    } else {
        for (int e = 0; e < 4; ++e) c[e] = e < here ? colidx[k0 + e] : 0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int32_t q = first + __popc(e < here ? word & (0xffffffffu >> (31 - b0 - e)) : 0u);
        di[e] = deg[ne_rows ? ne_rows[q] : q];
        dj[e] = norm == 1 ? deg[c[e]] : 0;
    }
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (norm == 2) v[e] = (float)__ddiv_rn(1.0, (double)di[e]);
        else {
            // a vertex whose row is empty (no self loops, no outgoing edge) scales by 0: D^-1/2 as a pseudo-inverse,
            // the same convention as the per-vertex factors of the value-free product
            const double dd = __dmul_rn((double)di[e], (double)dj[e]);
            v[e] = dd > 0.0 ? (float)__ddiv_rn(1.0, __dsqrt_rn(dd)) : 0.f;
        }
    }
    if (here == 4) *reinterpret_cast<float4*>(val + k0) = make_float4(v[0], v[1], v[2], v[3]);
    else
        for (int e = 0; e < here; ++e) val[k0 + e] = v[e];
}

// keys row<<cbits|col from compressed rows: thread k finds its row by bisection on rowptr.  *bad is set unless the columns
// ascend strictly inside every row and lie in [0, ncols).
__global__ void k_keys_from_csr(int64_t nnz, int64_t n, int64_t ncols, const int64_t* __restrict__ rowptr,
                                const int32_t* __restrict__ colidx, unsigned cbits, uint64_t* __restrict__ keys,
                                int* __restrict__ bad) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    int64_t lo = 0, hi = n;   // largest r with rowptr[r] <= k
    while (hi - lo > 1) {
        int64_t mid = (lo + hi) >> 1;
        if (rowptr[mid] <= k) lo = mid; else hi = mid;
    }
    const int32_t c = colidx[k];
    if (c < 0 || c >= ncols || (k > rowptr[lo] && colidx[k - 1] >= c)) *bad = 1;
    keys[k] = ((uint64_t)lo << cbits) | (uint32_t)c;
}

__global__ __launch_bounds__(256) void k_narrow(int64_t n, const int32_t* __restrict__ in, uint16_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (uint16_t)in[i];
}

__global__ void k_validate_rowptr(int64_t n, const int64_t* __restrict__ rowptr, int* __restrict__ bad) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (i == 0 && rowptr[0] != 0) *bad = 1;
    if (rowptr[i + 1] < rowptr[i]) *bad = 1;
}

__global__ void k_fill_f32(int64_t count, float v, float* __restrict__ out) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) out[k] = v;
}

// ---- schedule kernels ---------------------------------------------------------------------------

struct NonEmpty {
    const int64_t* rowptr;
    __device__ bool operator()(const int32_t& r) const { return rowptr[r + 1] > rowptr[r]; }
};
struct IsEmpty {
    const int64_t* rowptr;
    __device__ bool operator()(const int32_t& r) const { return rowptr[r + 1] == rowptr[r]; }
};

__global__ void k_ne_rowptr(int64_t n_ne, int64_t nnz, const int32_t* __restrict__ ne_rows,
                            const int64_t* __restrict__ rowptr, int64_t* __restrict__ out) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n_ne) out[q] = rowptr[ne_rows[q]];
    if (q == n_ne) out[q] = nnz;
}

// ---- host helpers ---------------------------------------------------------------------------------

// The chunks c >= 1 whose first entry continues a row begun earlier and that are the first such chunk
// of that row: exactly the chunks for which the fix-up kernel has work.  `covered`: only those in which no row starts,
// otherwise only the others.
struct LeadsCarry {
    const uint32_t* flags;
    const int32_t* sub_row;
    const int64_t* rp;
    int64_t nnz;
    bool covered;
    __device__ bool operator()(const int64_t& c0) const {
        const int64_t c = c0 + 1;
        const int64_t j0 = c * SUBS_PER_CHUNK;
        if (flags[j0] & 1u) return false;
        const int32_t q = sub_row[j0];
        if (c != rp[q] / CHUNK + 1) return false;
        const int64_t end = (c + 1) * CHUNK < nnz ? (c + 1) * CHUNK : nnz;
        return (rp[q + 1] >= end) == covered;
    }
};

__global__ void k_two_totals(const int64_t* __restrict__ a, const int64_t* __restrict__ b, int64_t* __restrict__ out) {
    out[0] = *a;
    out[1] = *b;
}

__global__ void k_fix_records(int64_t count, const int32_t* __restrict__ sel, const int32_t* __restrict__ sub_row,
                              const int64_t* __restrict__ rp, int4* __restrict__ list) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const int32_t c = sel[t] + 1;
    const int32_t q = sub_row[(int64_t)c * SUBS_PER_CHUNK];
    list[t] = make_int4(c, (int32_t)((rp[q + 1] - 1) / CHUNK), q, 0);
}

int build_fix_list(const uint32_t* flags, const int32_t* sub_row, const int64_t* rp, int64_t nnz, int4** list,
                   int64_t* count, int64_t* n_long, hipStream_t s) {
    *count = *n_long = 0;
    const int64_t nchunks = (nnz + CHUNK - 1) / CHUNK;
    if (nchunks <= 1) return GCN_OK;
    if (nchunks >= (1ll << 31)) return fail(GCN_ERR_RANGE, "schedule: too many chunks");
    // both kinds are positioned before the host waits for their numbers, once
    const LeadsCarry longs{flags, sub_row, rp, nnz, true}, shorts{flags, sub_row, rp, nnz, false};
    TempBuf sel, off_long, off_short, totals;
    GCN_TRY(prims::select_positions<1>(nchunks - 1, longs, off_long, s));
    GCN_TRY(prims::select_positions<1>(nchunks - 1, shorts, off_short, s));
    GCN_TRY(totals.alloc(16));
    hipLaunchKernelGGL(k_two_totals, dim3(1), dim3(1), 0, s, prims::select_total<1>(nchunks - 1, off_long), prims::select_total<1>(nchunks - 1, off_short),
                       totals.as<int64_t>());
    GCN_LAUNCH_CHECK();
    int64_t h[2] = {0, 0};
    GCN_HIP_TRY(hipMemcpyAsync(h, totals.p, 16, hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipStreamSynchronize(s));
    *n_long = h[0];
    const int64_t nsel = h[0] + h[1];
    if (nsel > 0) {
        GCN_TRY(sel.alloc((size_t)nsel * 4));
        GCN_TRY(prims::select_store<1>(nchunks - 1, longs, prims::EmitIndex32{sel.as<int32_t>()}, off_long, s));
        GCN_TRY(prims::select_store<1>(nchunks - 1, shorts, prims::EmitIndex32{sel.as<int32_t>() + h[0]}, off_short, s));
        GCN_TRY(device_alloc_t(list, (size_t)nsel));
        hipLaunchKernelGGL(k_fix_records, dim3(blocks_for(nsel)), dim3(TPB), 0, s, nsel, sel.as<int32_t>(), sub_row, rp, *list);
        GCN_LAUNCH_CHECK();
    }
    *count = nsel;
    return GCN_OK;
}

// The flag words and the rows of every 32nd entry, zeroed.
static int alloc_subs(Matrix& m, int64_t nnz, hipStream_t s) {
    const size_t words = (size_t)((nnz + SUB - 1) / SUB) + SUBS_PER_CHUNK;                // padded: one chunk of zero words
    GCN_TRY(device_alloc_t(&m.flags, words));
    GCN_TRY(device_alloc_t(&m.sub_row, words));
    GCN_HIP_TRY(hipMemsetAsync(m.flags, 0, words * sizeof(uint32_t), s));
    GCN_HIP_TRY(hipMemsetAsync(m.sub_row, 0, words * sizeof(int32_t), s));
    return GCN_OK;
}

int build_schedule(Matrix& m, int64_t n, int64_t nnz, hipStream_t s, int32_t* deg) {
    m.nsub = (nnz + SUB - 1) / SUB;
    m.nchunks = (nnz + CHUNK - 1) / CHUNK;
    TempBuf counters;
    GCN_TRY(counters.alloc(sizeof(DegreeSums)));
    GCN_HIP_TRY(hipMemsetAsync(counters.p, 0, sizeof(DegreeSums), s));
    hipLaunchKernelGGL(k_degrees, dim3(degree_blocks(n)), dim3(DEGREE_THREADS), 0, s, n, m.rowptr, deg, counters.as<DegreeSums>());
    GCN_LAUNCH_CHECK();
    const bool sampled = nnz >= PLANNED_NNZ;
    static_assert(PLANNED_NNZ >= RowOrder::STRETCH, "windows lie inside the matrix");
    if (sampled) {
        hipLaunchKernelGGL(k_sample_columns, dim3(RowOrder::WINDOWS), dim3(1024), 0, s, nnz, m.colidx, counters.as<DegreeSums>()->ones);
        GCN_LAUNCH_CHECK();
    }
    DegreeSums h;
    GCN_HIP_TRY(hipMemcpyAsync(&h, counters.p, sizeof h, hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipStreamSynchronize(s));
    m.max_degree = h.max_deg;
    m.n_ne = (int64_t)h.n_nonempty;
    for (int b = 0; b < Lengths::BINS; ++b) {
        m.lengths.rows[b] = (int64_t)h.rows[b];
        m.lengths.entries[b] = (int64_t)h.entries[b];
    }
    m.order.sum = (double)h.sum;
    m.order.squares = (double)h.squares;
    m.order.distinct = sampled ? RowOrder::distinct_of(h.ones) : 0.0;
    const int64_t* rp = m.rowptr;
    if (m.n_ne < n) {
        GCN_TRY(device_alloc_t(&m.ne_rows, (size_t)m.n_ne));
        GCN_TRY(device_alloc_t(&m.ne_rowptr, (size_t)m.n_ne + 1));
        NonEmpty pred{m.rowptr};
        GCN_TRY(prims::select_indices(n, pred, m.ne_rows, nullptr, s));
        hipLaunchKernelGGL(k_ne_rowptr, dim3(blocks_for(m.n_ne + 1)), dim3(TPB), 0, s, m.n_ne, nnz, m.ne_rows,
                           m.rowptr, m.ne_rowptr);
        GCN_LAUNCH_CHECK();
        GCN_TRY(device_alloc_t(&m.empty_rows, (size_t)(n - m.n_ne)));
        IsEmpty epred{m.rowptr};
        GCN_TRY(prims::select_indices(n, epred, m.empty_rows, nullptr, s));
        rp = m.ne_rowptr;
    }
    const bool given = m.flags != nullptr;                     // by k_part_emit, sub_row with the rows themselves
    if (!given) GCN_TRY(alloc_subs(m, nnz, s));
    if (nnz > 0 && !given) {
        hipLaunchKernelGGL(k_row_flags, dim3(blocks_for(m.n_ne)), dim3(TPB), 0, s, m.n_ne, rp, m.flags);
        GCN_LAUNCH_CHECK();
    }
    if (nnz > 0 && (!given || m.n_ne < n)) {
        hipLaunchKernelGGL(k_sub_rows, dim3(blocks_for(m.nsub)), dim3(TPB), 0, s, m.nsub, m.n_ne, rp, m.sub_row);
        GCN_LAUNCH_CHECK();
    }
    if (nnz > 0) GCN_TRY(build_fix_list(m.flags, m.sub_row, rp, nnz, &m.fix_list, &m.n_fix, &m.n_fix_long, s));
    return GCN_OK;
}

// Four entries of a row per thread.
__global__ __launch_bounds__(256) void k_short_rows(int64_t nrows, int32_t quads, const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                    const float* __restrict__ val, int4* __restrict__ col4, float4* __restrict__ val4,
                                                    int32_t* __restrict__ rows) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, row = t / quads;
    if (row >= nrows) return;
    const int k0 = (int)(t % quads) * 4;
    const int64_t first = rowptr[row];
    const int len = (int)(rowptr[row + 1] - first);
    int32_t c[4];
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        c[e] = k0 + e < len ? colidx[first + k0 + e] : 0;
        v[e] = k0 + e < len ? val[first + k0 + e] : 0.f;
    }
    col4[t] = make_int4(c[0], c[1], c[2], c[3]);
    val4[t] = make_float4(v[0], v[1], v[2], v[3]);
    if (k0 == 0) rows[row] = len | (int32_t)(first % CHUNK) << 16;
}

// A second copy of a matrix of few and short rows, at an equal pitch: a product on it is a chain of memory latencies, and this way the
// indices need not wait for the row pointers (see k_spmm_short).  At most 33 MB.
int build_short(Matrix& m, int64_t nnz, hipStream_t s) {
    if (m.nrows * 2 > SHORT_LANES || m.max_degree > SHORT_ROW || m.max_degree == 0) return GCN_OK;
    const int32_t quads = (m.max_degree + 3) / 4;
    const int64_t threads = m.nrows * quads;
    m.short_pitch = 4 * quads;
    if (!short_copy_pays(m.nrows, m.short_pitch, nnz, m.lengths.from(4).count())) return GCN_OK;
    if (device_alloc_t(&m.short_col, (size_t)threads * 8 + m.nrows) != GCN_OK) return GCN_OK;       // without it the other kernels run
    m.short_val = (float*)(m.short_col + threads * 4);
    m.short_rows = m.short_col + threads * 8;
    hipLaunchKernelGGL(k_short_rows, dim3(blocks_for(threads)), dim3(TPB), 0, s, m.nrows, quads, m.rowptr, m.colidx, m.val, (int4*)m.short_col,
                       (float4*)m.short_val, m.short_rows);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// A^T of `a` from A's sorted keys and values: a stable radix sort by the column bits alone (inside a column the rows keep
// their ascending order) with the values as payload.
static int build_transpose(gcn_csr* a, const uint64_t* keys, unsigned cbits, uint64_t* scratch_keys, hipStream_t s) {
    const int64_t nnz = a->nnz, n = a->ncols;            // A^T has ncols rows
    GCN_TRY(device_alloc_t(&a->At.val, (size_t)nnz));
    if (nnz > 0)
        GCN_TRY((prims::radix_sort<uint64_t, float>(keys, scratch_keys, a->A.val, a->At.val, (size_t)nnz, cbits, false, s, false)));
    a->At.nrows = n;
    a->At.ncols = a->n;
    GCN_TRY(device_alloc_t(&a->At.rowptr, (size_t)n + 1));
    GCN_TRY(device_alloc_t(&a->At.colidx, (size_t)nnz));
    hipLaunchKernelGGL(k_compress, dim3(blocks_for(nnz)), dim3(TPB), 0, s, nnz, n, scratch_keys, 0u, (1ull << cbits) - 1, cbits, ~0ull,
                       a->At.rowptr, a->At.colidx);
    GCN_LAUNCH_CHECK();
    GCN_TRY(build_schedule(a->At, n, nnz, s));
    GCN_TRY(build_short(a->At, nnz, s));
    a->has_t = true;
    return GCN_OK;
}

// The entries of A by the sort of row_sort.h: columns, row pointers and, where they are wanted, the sorted keys.  *done stays false where that
// sort does not take the matrix.
static int entries_by_rows(gcn_csr* a, int64_t n, int64_t m, const int32_t* src, const int32_t* dst, bool sym, bool loops, unsigned cbits,
                           bool want_keys, TempBuf& keys, bool* done, hipStream_t s) {
    using namespace rowsort;
    const int64_t cap = m * (sym ? 2 : 1) + (loops ? n : 0);
    unsigned shift;
    uint32_t nb;
    if (!takes(n, cap, cbits, &shift, &nb)) return GCN_OK;
    const Items items{src, dst, m, n, m + (loops ? n : 0), sym, cbits, shift};
    const int64_t share = (items.items + SHARES - 1) / SHARES;
    const size_t most_tasks = (size_t)nb + (size_t)(cap / PIECE) + 1;
    TempBuf info, table, total, start, tasks, at, count, offset, order, crowded, keys32;
    GCN_TRY(info.alloc(sizeof(Info)));
    GCN_TRY(table.alloc((size_t)SHARES * nb * 4));
    GCN_TRY(total.alloc((size_t)nb * 4));
    GCN_TRY(start.alloc((size_t)nb * 4));
    GCN_TRY(tasks.alloc(most_tasks * sizeof(Task)));
    GCN_TRY(at.alloc(most_tasks * 4));
    GCN_TRY(count.alloc(most_tasks * 4));
    GCN_TRY(offset.alloc(most_tasks * 4));
    GCN_TRY(order.alloc(most_tasks * 4));
    GCN_TRY(crowded.alloc(most_tasks * 4));
    // Both sides of the sort in one block of 8 bytes per key: where the matrix is refused the radix sort takes it for its own keys (two
    // blocks it could not use raised the peak of such a construction from 16 to 24 bytes per key).
    GCN_TRY(keys32.alloc((size_t)cap * 8));
    uint32_t* const k0 = keys32.as<uint32_t>(), * const k1 = k0 + cap;
    GCN_HIP_TRY(hipMemsetAsync(info.p, 0, sizeof(Info), s));
    hipLaunchKernelGGL(k_part_count, dim3(SHARES), dim3(THREADS), 0, s, items, share, nb, table.as<uint32_t>(), info.as<Info>());
    GCN_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_part_shares, dim3((nb + 63) / 64), dim3(THREADS), 0, s, nb, table.as<uint32_t>(), total.as<uint32_t>());
    GCN_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_part_tasks, dim3(1), dim3(THREADS), 0, s, nb, (uint64_t)cap * MOST_AGAIN, total.as<uint32_t>(),
                       start.as<uint32_t>(), tasks.as<Task>(), order.as<uint32_t>(), info.as<Info>());
    GCN_LAUNCH_CHECK();
    launch_lds<k_part_scatter>(dim3(SHARES), THREADS, SCATTER_LDS, s, items, share, nb, (const uint32_t*)start.as<uint32_t>(),
                               (const uint32_t*)table.as<uint32_t>(), (const Info*)info.as<Info>(), k0);
    GCN_LAUNCH_CHECK();
    const SortArgs sort{cbits, shift, tasks.as<Task>(), order.as<uint32_t>(), k0, k1, at.as<uint32_t>(),
                        count.as<uint32_t>(), crowded.as<uint32_t>(), info.as<Info>()};
    launch_lds<k_part_sort>(dim3((unsigned)most_tasks), THREADS, sort_lds(shift), s, sort);
    GCN_LAUNCH_CHECK();
    launch_lds<k_part_sort_digits>(dim3((unsigned)device_info().cus), THREADS, sort_lds(0), s, sort);
    GCN_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_part_offsets, dim3(1), dim3(THREADS), 0, s, (const uint32_t*)count.as<uint32_t>(), offset.as<uint32_t>(), info.as<Info>());
    GCN_LAUNCH_CHECK();
    Info h;
    GCN_HIP_TRY(hipMemcpyAsync(&h, info.p, sizeof h, hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipStreamSynchronize(s));
    if (h.bad) return fail(GCN_ERR_RANGE, "gcn_csr_create: a vertex id is outside [0, %lld)", (long long)n);
    if (h.refused) return GCN_OK;
    a->nnz = h.kept;
    GCN_TRY(device_alloc_t(&a->A.colidx, (size_t)h.kept));
    if (want_keys) GCN_TRY(keys.alloc((size_t)h.kept * 8));
    GCN_TRY(alloc_subs(a->A, h.kept, s));
    hipLaunchKernelGGL(k_part_emit, dim3(h.tasks), dim3(512), 0, s, n, nb, cbits, shift, (const Task*)tasks.as<Task>(), (const uint32_t*)at.as<uint32_t>(),
                       (const uint32_t*)count.as<uint32_t>(), (const uint32_t*)offset.as<uint32_t>(), (const uint32_t*)k1, a->A.rowptr,
                       a->A.colidx, want_keys ? keys.as<uint64_t>() : nullptr, a->A.flags, a->A.sub_row);
    GCN_LAUNCH_CHECK();
    *done = true;
    return GCN_OK;
}

// The same by a radix sort of 64-bit keys, for any matrix.
static int entries_by_keys(gcn_csr* a, int64_t n, int64_t m, const int32_t* src, const int32_t* dst, bool sym, bool loops, unsigned cbits,
                           bool want_keys, TempBuf& keys, hipStream_t s) {
    const int64_t cap = m * (sym ? 2 : 1) + (loops ? n : 0);
    const uint64_t none = (uint64_t)n << cbits;
    TempBuf bad, k1, off;
    GCN_TRY(bad.alloc(sizeof(int)));
    GCN_HIP_TRY(hipMemsetAsync(bad.p, 0, sizeof(int), s));
    int64_t nnz = 0;
    if (cap > 0) {
        GCN_TRY(k1.alloc((size_t)cap * 8));
        GCN_TRY(prims::radix_sort_from(PairKeys{src, dst, m, n, sym, loops, cbits, bad.as<int>()}, k1.as<uint64_t>(), (size_t)cap,
                                       cbits + bits_for(loops ? n : n + 1), s));
        GCN_TRY(prims::select_positions(cap, prims::FirstOfRun{k1.as<uint64_t>()}, off, s));
        TempBuf result;
        GCN_TRY(result.alloc(sizeof(SortResult)));
        hipLaunchKernelGGL(k_sort_result, dim3(1), dim3(1), 0, s, prims::select_total(cap, off), k1.as<uint64_t>() + (cap - 1), bad.as<int>(),
                           result.as<SortResult>());
        GCN_LAUNCH_CHECK();
        SortResult h;
        GCN_HIP_TRY(hipMemcpyAsync(&h, result.p, sizeof h, hipMemcpyDeviceToHost, s));
        GCN_HIP_TRY(hipStreamSynchronize(s));
        if (h.bad) return fail(GCN_ERR_RANGE, "gcn_csr_create: a vertex id is outside [0, %lld)", (long long)n);
        nnz = h.kept - (!loops && h.last == none ? 1 : 0);
    }
    a->nnz = nnz;
    GCN_TRY(device_alloc_t(&a->A.colidx, (size_t)nnz));
    if (cap > 0) {
        if (want_keys) GCN_TRY(keys.alloc((size_t)nnz * 8));
        GCN_TRY(prims::select_store(cap, prims::FirstOfRun{k1.as<uint64_t>()},
                                    EmitEntry{k1.as<uint64_t>(), n, cbits, a->A.rowptr, a->A.colidx, want_keys ? keys.as<uint64_t>() : nullptr}, off, s));
    }
    const unsigned blocks = blocks_for(n < (1 << 19) ? n : (1 << 19), 1024);
    hipLaunchKernelGGL(k_close_rows, dim3(blocks), dim3(256), 0, s, n, nnz, cap > 0 ? k1.as<uint64_t>() + (cap - 1) : nullptr,
                       cbits, a->A.rowptr);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

static int create_impl(gcn_csr* a, int64_t n, int64_t m, const int32_t* src, const int32_t* dst, uint32_t flags,
                       hipStream_t s) {
    const bool sym = flags & GCN_SYMMETRISE, loops = flags & GCN_ADD_SELF_LOOPS;
    const unsigned cbits = bits_for(n);

    const bool transpose = flags & GCN_BUILD_TRANSPOSE;
    // Both directions of every pair are stored and the value formula (1, or 1/sqrt(d_i d_j)) is symmetric: A^T is A,
    // bit by bit, and one set of arrays and schedules serves both.
    a->symmetric = transpose && sym && !(flags & GCN_NORM_ROW);
    a->n = n;
    a->ncols = n;
    a->A.nrows = a->A.ncols = n;
    a->A.terms = (flags & GCN_NORM_SYM) ? Terms::BY_BOTH : ((flags & GCN_NORM_ROW) ? Terms::BY_ROW : Terms::ALIKE);
    a->At.terms = (flags & GCN_NORM_SYM) && sym ? Terms::BY_BOTH : Terms::ALIKE;      // (its rows are as long as a vertex has entries in A's columns)
    GCN_TRY(device_alloc_t(&a->A.rowptr, (size_t)n + 1));
    TempBuf keys;                                          // row << cbits | column of every entry, for the transpose
    const bool want_keys = transpose && !a->symmetric;
    bool done = false;
    GCN_TRY(entries_by_rows(a, n, m, src, dst, sym, loops, cbits, want_keys, keys, &done, s));
    if (!done) GCN_TRY(entries_by_keys(a, n, m, src, dst, sym, loops, cbits, want_keys, keys, s));
    const int64_t nnz = a->nnz;
    GCN_TRY(device_alloc_t(&a->deg, (size_t)n));
    GCN_TRY(device_alloc_t(&a->A.val, (size_t)nnz));
    GCN_TRY(build_schedule(a->A, n, nnz, s, a->deg));
    if (nnz > 0) {
        const dim3 grid(blocks_for((nnz + 3) / 4));
        if ((flags & GCN_NORM_SYM) && a->A.max_degree < (1 << 16)) {
            TempBuf deg16;
            GCN_TRY(deg16.alloc((size_t)n * 2));
            hipLaunchKernelGGL(k_narrow, dim3(blocks_for(n)), dim3(TPB), 0, s, n, a->deg, deg16.as<uint16_t>());
            GCN_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_values<uint16_t>, grid, dim3(TPB), 0, s, nnz, a->A.colidx, a->A.flags, a->A.sub_row, a->A.ne_rows, deg16.as<uint16_t>(), 1, a->A.val);
        } else if (flags & (GCN_NORM_ROW | GCN_NORM_SYM))
            hipLaunchKernelGGL(k_values<int32_t>, grid, dim3(TPB), 0, s, nnz, a->A.colidx, a->A.flags, a->A.sub_row, a->A.ne_rows, a->deg, (flags & GCN_NORM_ROW) ? 2 : 1, a->A.val);
        else hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(nnz)), dim3(TPB), 0, s, nnz, 1.0f, a->A.val);
        GCN_LAUNCH_CHECK();
    }
    if ((flags & GCN_NORM_SYM) && n > 0) {
        GCN_TRY(device_alloc_t(&a->inv_sqrt_deg, (size_t)n));
        GCN_TRY(inv_sqrt_deg_launch(n, a->deg, a->inv_sqrt_deg, s));
    }
    GCN_TRY(build_short(a->A, nnz, s));
    if (a->symmetric) a->has_t = true;
    else if (transpose) {
        TempBuf sorted;
        GCN_TRY(sorted.alloc((size_t)nnz * 8));
        GCN_TRY(build_transpose(a, keys.as<uint64_t>(), cbits, sorted.as<uint64_t>(), s));
    }
    return GCN_OK;
}

static int from_csr_impl(gcn_csr* a, int64_t n, int64_t ncols, const int64_t* rowptr, const int32_t* colidx,
                         const float* val, uint32_t flags, hipStream_t s) {
    TempBuf bad;
    GCN_TRY(bad.alloc(sizeof(int)));
    GCN_HIP_TRY(hipMemsetAsync(bad.p, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_validate_rowptr, dim3(blocks_for(n)), dim3(TPB), 0, s, n, rowptr, bad.as<int>());
    GCN_LAUNCH_CHECK();
    int hbad = 0;
    int64_t nnz = 0;
    GCN_HIP_TRY(hipMemcpyAsync(&hbad, bad.p, sizeof(int), hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipMemcpyAsync(&nnz, rowptr + n, 8, hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipStreamSynchronize(s));
    if (hbad || nnz < 0) return fail(GCN_ERR_UNSORTED, "gcn_csr_create_from_csr: rowptr must start at 0 and not decrease");
    if (nnz > 0 && !colidx) return fail(GCN_ERR_BADARG, "gcn_csr_create_from_csr: NULL colidx");
    a->n = n;
    a->ncols = ncols;
    a->nnz = nnz;
    a->A.nrows = n;
    a->A.ncols = ncols;
    GCN_TRY(device_alloc_t(&a->A.rowptr, (size_t)n + 1));
    GCN_TRY(device_alloc_t(&a->A.colidx, (size_t)nnz));
    GCN_TRY(device_alloc_t(&a->A.val, (size_t)nnz));
    GCN_TRY(device_alloc_t(&a->deg, (size_t)n));
    GCN_HIP_TRY(hipMemcpyAsync(a->A.rowptr, rowptr, ((size_t)n + 1) * 8, hipMemcpyDeviceToDevice, s));
    const unsigned cbits = bits_for(ncols);
    TempBuf keys, k1;
    GCN_TRY(keys.alloc((size_t)nnz * 8));
    if (nnz > 0) {
        GCN_HIP_TRY(hipMemcpyAsync(a->A.colidx, colidx, (size_t)nnz * 4, hipMemcpyDeviceToDevice, s));
        if (val) GCN_HIP_TRY(hipMemcpyAsync(a->A.val, val, (size_t)nnz * 4, hipMemcpyDeviceToDevice, s));
        else {
            hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(nnz)), dim3(TPB), 0, s, nnz, 1.0f, a->A.val);
            GCN_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL(k_keys_from_csr, dim3(blocks_for(nnz)), dim3(TPB), 0, s, nnz, n, ncols, a->A.rowptr, a->A.colidx,
                           cbits, keys.as<uint64_t>(), bad.as<int>());
        GCN_LAUNCH_CHECK();
        GCN_HIP_TRY(hipMemcpyAsync(&hbad, bad.p, sizeof(int), hipMemcpyDeviceToHost, s));
        GCN_HIP_TRY(hipStreamSynchronize(s));
        if (hbad) return fail(GCN_ERR_UNSORTED, "gcn_csr_create_from_csr: columns must be strictly ascending per row and inside [0,n)");
    }
    GCN_TRY(build_schedule(a->A, n, nnz, s, a->deg));
    GCN_TRY(build_short(a->A, nnz, s));
    if (flags & GCN_BUILD_TRANSPOSE) {
        GCN_TRY(k1.alloc((size_t)nnz * 8));
        GCN_TRY(build_transpose(a, keys.as<uint64_t>(), cbits, k1.as<uint64_t>(), s));
    }
    return GCN_OK;
}

}  // namespace gcn

using namespace gcn;

namespace {
struct Pay4 { uint32_t a; };
struct Pay8 { uint32_t a, b; };
struct Pay12 { uint32_t a, b, c; };

template <typename K>
int radix_sort_by_payload(int64_t n, const void* kin, void* kout, int payload_bytes, const void* pin, void* pout,
                          unsigned end_bit, bool desc, hipStream_t s) {
    using namespace gcn::prims;
    const K* ki = (const K*)kin;
    K* ko = (K*)kout;
    switch (payload_bytes) {
        case 0: return radix_sort<K, NoValue>(ki, ko, (const NoValue*)nullptr, (NoValue*)nullptr, (size_t)n, end_bit, desc, s);
        case 4: return radix_sort<K, Pay4>(ki, ko, (const Pay4*)pin, (Pay4*)pout, (size_t)n, end_bit, desc, s);
        case 8: return radix_sort<K, Pay8>(ki, ko, (const Pay8*)pin, (Pay8*)pout, (size_t)n, end_bit, desc, s);
        case 12: return radix_sort<K, Pay12>(ki, ko, (const Pay12*)pin, (Pay12*)pout, (size_t)n, end_bit, desc, s);
        default: return gcn::fail(GCN_ERR_BADARG, "gcn_radix_sort: payload_bytes must be 0, 4, 8 or 12");
    }
}
}  // namespace

extern "C" {

int gcn_csr_create(gcn_csr** out, int64_t n, int64_t n_edges, const int32_t* src, const int32_t* dst,
                   uint32_t flags, void* stream) {
    if (!out) return fail(GCN_ERR_BADARG, "gcn_csr_create: NULL out");
    *out = nullptr;
    if (n <= 0 || n_edges < 0) return fail(GCN_ERR_BADARG, "gcn_csr_create: n must be positive and n_edges non-negative");
    if (n >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_csr_create: n must be below 2^31");
    if (n_edges > 0 && (!src || !dst)) return fail(GCN_ERR_BADARG, "gcn_csr_create: NULL edge arrays");
    if (n_edges > (1ll << 40)) return fail(GCN_ERR_RANGE, "gcn_csr_create: too many edges");
    if ((flags & GCN_NORM_SYM) && (flags & GCN_NORM_ROW)) return fail(GCN_ERR_BADARG, "gcn_csr_create: choose one normalisation");
    gcn_csr* a = new (std::nothrow) gcn_csr();
    if (!a) return fail(GCN_ERR_OOM, "host allocation failed");
    (void)hipGetDevice(&a->device);
    BuildScope scope((hipStream_t)stream);
    int rc = create_impl(a, n, n_edges, src, dst, flags, (hipStream_t)stream);
    if (rc != GCN_OK) {
        gcn_csr_destroy(a);
        return rc;
    }
    *out = a;
    return GCN_OK;
}

int gcn_csr_create_from_csr(gcn_csr** out, int64_t n, const int64_t* rowptr, const int32_t* colidx,
                            const float* val, uint32_t flags, void* stream) {
    if (!out) return fail(GCN_ERR_BADARG, "gcn_csr_create_from_csr: NULL out");
    *out = nullptr;
    if (n <= 0 || !rowptr) return fail(GCN_ERR_BADARG, "gcn_csr_create_from_csr: n must be positive, rowptr non-NULL");
    if (n >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_csr_create_from_csr: n must be below 2^31");
    gcn_csr* a = new (std::nothrow) gcn_csr();
    if (!a) return fail(GCN_ERR_OOM, "host allocation failed");
    (void)hipGetDevice(&a->device);
    BuildScope scope((hipStream_t)stream);
    int rc = from_csr_impl(a, n, n, rowptr, colidx, val, flags, (hipStream_t)stream);
    if (rc != GCN_OK) {
        gcn_csr_destroy(a);
        return rc;
    }
    *out = a;
    return GCN_OK;
}

int gcn_csr_create_from_csr_rect(gcn_csr** out, int64_t n_rows, int64_t n_cols, const int64_t* rowptr,
                                 const int32_t* colidx, const float* val, uint32_t flags, void* stream) {
    if (!out) return fail(GCN_ERR_BADARG, "gcn_csr_create_from_csr_rect: NULL out");
    *out = nullptr;
    if (n_rows <= 0 || n_cols <= 0 || !rowptr) return fail(GCN_ERR_BADARG, "gcn_csr_create_from_csr_rect: sizes must be positive, rowptr non-NULL");
    if (n_rows >= (1ll << 31) || n_cols >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_csr_create_from_csr_rect: sizes must be below 2^31");
    gcn_csr* a = new (std::nothrow) gcn_csr();
    if (!a) return fail(GCN_ERR_OOM, "host allocation failed");
    (void)hipGetDevice(&a->device);
    BuildScope scope((hipStream_t)stream);
    int rc = from_csr_impl(a, n_rows, n_cols, rowptr, colidx, val, flags, (hipStream_t)stream);
    if (rc != GCN_OK) {
        gcn_csr_destroy(a);
        return rc;
    }
    *out = a;
    return GCN_OK;
}

int gcn_radix_sort(int64_t n, int key_bytes, const void* keys_in, void* keys_out, int payload_bytes,
                   const void* payload_in, void* payload_out, int end_bit, int descending, void* stream) {
    using gcn::fail;
    if (n < 0 || end_bit < 0) return fail(GCN_ERR_BADARG, "gcn_radix_sort: negative size");
    if (n == 0) return GCN_OK;
    BuildScope scope((hipStream_t)stream);
    if (!keys_in || !keys_out || keys_in == keys_out) return fail(GCN_ERR_BADARG, "gcn_radix_sort: keys NULL or in place");
    if (payload_bytes != 0 && (!payload_in || !payload_out || payload_in == payload_out))
        return fail(GCN_ERR_BADARG, "gcn_radix_sort: payload NULL or in place");
    if (key_bytes == 8)
        return radix_sort_by_payload<uint64_t>(n, keys_in, keys_out, payload_bytes, payload_in, payload_out,
                                               (unsigned)end_bit, descending != 0, (hipStream_t)stream);
    if (key_bytes == 4)
        return radix_sort_by_payload<uint32_t>(n, keys_in, keys_out, payload_bytes, payload_in, payload_out,
                                               (unsigned)end_bit, descending != 0, (hipStream_t)stream);
    return fail(GCN_ERR_BADARG, "gcn_radix_sort: key_bytes must be 4 or 8");
}

int gcn_exclusive_scan_i64(int64_t n, const int64_t* in, int64_t* out, void* stream) {
    if (n < 0) return gcn::fail(GCN_ERR_BADARG, "gcn_exclusive_scan_i64: negative size");
    if (n == 0) return GCN_OK;
    BuildScope scope((hipStream_t)stream);
    if (!in || !out) return gcn::fail(GCN_ERR_BADARG, "gcn_exclusive_scan_i64: NULL pointer");
    return gcn::prims::exclusive_scan<int64_t>(in, out, (size_t)n, (hipStream_t)stream);
}

int gcn_unique_u64(int64_t n, const uint64_t* keys_in, uint64_t* keys_out, int64_t* count, void* stream) {
    if (n < 0 || !count) return gcn::fail(GCN_ERR_BADARG, "gcn_unique_u64: negative size or NULL count");
    *count = 0;
    if (n == 0) return GCN_OK;
    BuildScope scope((hipStream_t)stream);
    if (!keys_in || !keys_out || keys_in == keys_out) return gcn::fail(GCN_ERR_BADARG, "gcn_unique_u64: keys NULL or in place");
    return gcn::prims::unique_keys(keys_in, keys_out, n, count, (hipStream_t)stream);
}

}  // extern "C"
