// SpMM: Z = op(A) X for a compressed-row matrix and a tall-skinny dense fp32 operand -- the
// "SpMM" of the paper's sections "Graph Neural Networks" and "A One-Dimensional (1D) Algorithm",
// the operation the paper calls the most time consuming.
//
// Main kernel: nonzero-split.  Every wavefront owns CHUNK = 512 consecutive stored entries no
// matter how they fall into rows, so a 20,000-entry row and 20,000 one-entry rows cost the same.
// The wavefront is cut into G = 64/LPR lane groups; a group of LPR lanes covers one gathered row
// of X (VEC floats per lane) and walks its own contiguous slice of the chunk.  Row boundaries come
// from one precomputed 32-bit flag word per 32 entries, so the walk never touches rowptr.
//   * a row that starts and ends inside one group's slice is written directly;
//   * pieces of a row spread over several groups are joined by a segmented suffix scan across the
//     groups (lane shuffles), in a fixed order;
//   * pieces spread over several wavefronts go through a per-chunk carry buffer and a small
//     second kernel that adds them in ascending chunk order.
// No floating-point atomics are used anywhere: results are bit-reproducible run to run.
// Column indices and values are read with coalesced 16-byte loads into LDS first and consumed
// from there; the gathered rows of X are read with one 16-byte load per lane.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <string>

#include "common.h"
#include "launch_rules.h"

namespace gcn {

static constexpr int WAVES_PER_BLOCK = 4;
static constexpr int SUB_STRIDE = SUB + 4;                         // LDS padding: groups hit different banks
static constexpr int LDS_PER_WAVE = SUBS_PER_CHUNK * SUB_STRIDE;   // ints

struct SplitArgs {
    const int32_t* colidx;
    const float* val;         // NULL: value-free product (every stored entry counts as 1)
    const float* row_scale;   // NULL, or one factor per output row applied before the epilogue
    const uint8_t* defer;     // NULL, or 1 for rows whose sum is stored raw (another pass finishes them)
    const uint32_t* flags;
    const int32_t* sub_row;
    const int32_t* ne_rows;   // NULL: row index == non-empty-row index
    const int64_t* rp;        // rowptr over non-empty rows
    const int4* fix_list;     // the rows that cross chunks: n_fix of them (see build_fix_list)
    int64_t n_fix, n_fix_long;  // the first n_fix_long of them cover a whole further chunk
    int64_t nnz, nsub, nchunks;
    int64_t n_ne = 0;         // rows that have entries
    int32_t f;
    const float* X;
    int64_t ldx;
    float* Z;
    int64_t ldz;
    const float* Zprev;
    int64_t ldzprev;
    float* carry;             // [nchunks][f]
    const float* bias = nullptr;        // with EPI_LAYER (see LayerEnd)
    float* H = nullptr;
    int relu = 0;
    int lds_kb = 0;           // host side: GCN_CFG_SPLIT_LDS_KB
    const int32_t* empty_rows = nullptr;        // rows without entries that the product's kernel zeroes (see zero_share)
    int64_t n_empty = 0;
    int32_t empty_share = 0;  // how many of them go with a chunk
    uint32_t per_xcd = 0;     // 0, or how many consecutive groups of chunks an XCD takes (see chunk_group)
};

// The group of WAVES_PER_BLOCK chunks that this workgroup takes.  Workgroups go to the XCDs in turn.  Over column blocks,
// whose chunks come block by block, every XCD takes one stretch of them instead: a block of X is then fetched into the
// one or two L2s whose XCDs walk it and not into all eight, which counts as long as the blocks are short of entries (5 M entries,
// 150 K columns, four blocks: 187 -> 140 us at 64 columns, 95 -> 74 at 32; 6 M, 120 K, two blocks at 64: 126 -> 117; 119 M,
// 233 K, seven blocks: no difference).  The panels of a product follow each other: each of them to its own XCDs took longer
// where X is beyond the L2s (33 M entries, 128 columns: 1.37 -> 1.55 ms).
static constexpr uint32_t XCDS = 8;
__device__ __forceinline__ int64_t chunk_group(const SplitArgs& a) {
    return a.per_xcd ? (int64_t)(blockIdx.x % XCDS) * a.per_xcd + blockIdx.x / XCDS : (int64_t)blockIdx.x;
}
static inline unsigned chunk_groups(const SplitArgs& a) {          // workgroups per panel
    return a.per_xcd ? XCDS * a.per_xcd : (unsigned)((a.nchunks + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
}

// The index/value stream is read exactly once per product: load it with the non-temporal hint so
// it does not push the gathered rows of X out of L2.
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef float fltx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int4 stream_load_i4(const int32_t* p) {
    const intx4 v = __builtin_nontemporal_load(reinterpret_cast<const intx4*>(p));
    return make_int4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 stream_load_f4(const float* p) {
    const fltx4 v = __builtin_nontemporal_load(reinterpret_cast<const fltx4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

struct __attribute__((packed, aligned(4))) f2u { float x, y; };

template <int VEC>
__device__ __forceinline__ void load_vec(float (&d)[VEC], const float* p) {
    if constexpr (VEC == 2) {
        const f2u v = *reinterpret_cast<const f2u*>(p);
        d[0] = v.x; d[1] = v.y;
    } else if constexpr (VEC == 4) {
        const f4u v = *reinterpret_cast<const f4u*>(p);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    } else {
        d[0] = *p;
    }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&d)[VEC]) {
    if constexpr (VEC == 2) {
        *reinterpret_cast<f2u*>(p) = f2u{d[0], d[1]};
    } else if constexpr (VEC == 4) {
        *reinterpret_cast<f4u*>(p) = f4u{d[0], d[1], d[2], d[3]};
    } else {
        *p = d[0];
    }
}

// The columns of one lane in panel `y` of an operand of width f: VEC of them from `col0` (false: none).  A width that is
// no multiple of 4 ends with a lane that repeats columns of its left neighbour, so that its 16 bytes stay inside
// the row; both compute and store the same values.  When fewer than four columns are left for the last panel it
// takes four more from the panel before, so that the repetition stays inside one panel.
template <int LPR, int VEC>
__device__ __forceinline__ bool lane_columns(int f, int y, int ny, int li, int* col0) {
    constexpr int W = LPR * VEC;
    int first = y * W, end = first + W < f ? first + W : f;
    if constexpr (VEC > 1) {
        const bool thin = ny > 1 && f - (ny - 1) * W < VEC;
        if (thin && y == ny - 1) first -= VEC;
        if (thin && y == ny - 2) end -= VEC;
    }
    const int c = first + li * VEC;
    *col0 = c + VEC <= end ? c : end - VEC;
    return c < end;
}

template <int VEC, int EPI>
__device__ __forceinline__ void epilogue_store(float* z, const float* zprev, float (&v)[VEC], float scale = 1.f,
                                               bool raw = false) {
    if (raw) {
        store_vec<VEC>(z, v);
        return;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] *= scale;           // exact for scale = 1
    if constexpr (EPI == GCN_EPI_RELU) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    } else if constexpr (EPI == GCN_EPI_MASK) {
        float m[VEC];
        load_vec<VEC>(m, zprev);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = m[e] > 0.f ? v[e] : 0.f;
    }
    store_vec<VEC>(z, v);
}

// The end of a layer: the same roundings as a product and a pass of its own, so no multiply-add.
template <int VEC>
__device__ __forceinline__ void layer_store(float* z, float* h, const float* bias, int relu, float (&v)[VEC], float scale) {
#pragma clang fp contract(off)
    float b[VEC] = {};
    if (bias) load_vec<VEC>(b, bias);
    float r[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        v[e] = v[e] * scale;
        if (bias) v[e] = v[e] + b[e];
        r[e] = v[e] > 0.f ? v[e] : 0.f;
        if (relu) v[e] = r[e];
    }
    store_vec<VEC>(z, v);
    if (h) store_vec<VEC>(h, r);
}

// Row `row` of a matrix whose rows are `pitch` bytes apart: one multiply-add of 32 by 32 bits.  Pitches of 4 GB and more
// do not come here (see rowwise_only).
__device__ __forceinline__ const float* at_row(const float* base, uint32_t row, uint32_t pitch) {
    return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (uint64_t)row * pitch);
}

// Stages a chunk's column indices and values in LDS (coalesced 16-byte loads); zeros past the end.
__device__ __forceinline__ void stage_chunk(const SplitArgs& a, int64_t k0, int lane, int32_t* lc, float* lv) {
#pragma unroll
    for (int t = 0; t < CHUNK / 256; ++t) {
        const int i = t * 256 + lane * 4;
        const int64_t k = k0 + i;
        int4 cc = make_int4(0, 0, 0, 0);
        float4 vv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k + 4 <= a.nnz) {
            cc = stream_load_i4(a.colidx + k);
            if (a.val) vv = stream_load_f4(a.val + k);
        } else {
            if (k + 0 < a.nnz) { cc.x = a.colidx[k + 0]; if (a.val) vv.x = a.val[k + 0]; }
            if (k + 1 < a.nnz) { cc.y = a.colidx[k + 1]; if (a.val) vv.y = a.val[k + 1]; }
            if (k + 2 < a.nnz) { cc.z = a.colidx[k + 2]; if (a.val) vv.z = a.val[k + 2]; }
        }
        const int p = i + (i >> 5) * (SUB_STRIDE - SUB);
        *reinterpret_cast<int4*>(lc + p) = cc;
        if (a.val) *reinterpret_cast<float4*>(lv + p) = vv;
    }
}

// Zeroes a chunk's share of the rows without entries (any epilogue maps 0 to 0): a launch of its own took 32 us for 0.7 M rows
// of 64 columns, bound by its stores, while the product beside it was short of memory traffic.  Where that pays: see
// share_of_empty_rows.  The list is asked for together with the chunk (empty_row), the stores are sent before its gathers, 64 rows at
// a time.  Called by whole wavefronts.  Forms of the kernels of their own (ZERO): in those of matrices without such rows the code for it
// cost 1 % of products of 11 to 40 us (k_spmm_line<1>, whose chunks take longer, 0.1 % on 90 products: one form).
__device__ __forceinline__ int32_t empty_row(const SplitArgs& a, int64_t c, int i) {
    if (a.empty_share == 0) return 0;
    const int64_t q = c * a.empty_share + i;
    return a.empty_rows[q < a.n_empty ? q : a.n_empty - 1];
}
template <int LPR, int VEC>
__device__ __forceinline__ void zero_share(const SplitArgs& a, int64_t c, int lane, int32_t row, int col0, bool col_ok) {
    constexpr int G = 64 / LPR;
    const int64_t left = a.n_empty - c * a.empty_share;
    const int mine = left < a.empty_share ? (int)left : a.empty_share, g = lane / LPR;
    const float zero[VEC] = {};
    for (int i0 = 0; i0 < mine; i0 += 64) {
        if (i0 > 0) row = empty_row(a, c, i0 + lane);
        const int count = mine - i0 < 64 ? mine - i0 : 64;
        for (int i = 0; i < count; i += G) {
            const int32_t r = __shfl(row, i + g, 64);
            if (i + g < count && col_ok) store_vec<VEC>(a.Z + (int64_t)r * a.ldz + col0, zero);
        }
    }
}

// What a wavefront keeps in LDS for its chunk.
template <int LPR, int VEC, bool MASK>
struct __attribute__((aligned(16))) WaveLds {
    // A bit per column for as many of the rows begun here as leave five workgroups to a compute unit; the rows after them are
    // looked up one by one (all 512 rows a chunk can begin: 12 M entries in rows of 236, 16 columns: 72 -> 78 us).
    static constexpr int MASK_BYTES = VEC == 4 ? LPR / 2 : 4;
    static constexpr int WITHOUT_MASK = 2 * LDS_PER_WAVE * 4 + CHUNK * 4 + (SUBS_PER_CHUNK + 4) * 4 + 64 * VEC * 4;
    static constexpr int MASK_ROWS = MASK ? (8192 - WITHOUT_MASK) / MASK_BYTES : 0;
    int32_t col[LDS_PER_WAVE];
    float val[LDS_PER_WAVE];                    // values; of a value-free product the factors of the rows begun here
    int32_t row[CHUNK];                         // the rows begun here; the sign bit says that their sum is stored raw
    uint32_t flag[SUBS_PER_CHUNK + 4];
    float head[64 * VEC];
    uint8_t mask[MASK_ROWS * MASK_BYTES];       // whether the derivative mask lets the sums of the first rows through
};

// The work of one workgroup: the four chunks 4*grp .. 4*grp+3 of the matrix described by `a`.
// lds: one block per wavefront (owned by the kernel, so that two instantiations of this body in one kernel share them).
//
// The walk is bound by instructions where X fits the caches, so it holds nothing but one multiply-add per address, the gather,
// the sums and a test per entry: what a row needs when it ends (its number, its factor) is in LDS before the walk,
// fetched into registers when the row starts, so that neither a start nor an end waits for memory (with these looked up at
// the end of a row, every end drained the gathers in flight; and 64-bit row addresses took six instructions, four of
// them multiplications).  With fewer than 16 lane groups the gathers of four entries are issued before the four before
// them are summed; with 16 that many rows are in flight anyway, and where the L2s' request rate is the bound more of
// them are slower (119 M entries over column blocks: 611 us, 620 with two sets).  12 M entries in rows of 236 at 64 columns, operand
// in the L2s: 187 -> 168 us; 2 M at 32: 34 -> 27; 33 M, packed hub and rest at 16: 318 -> 293; 9 M in rows of 9 at
// 32: 203 -> 200 (line fills).
template <int LPR, int VEC, int EPI, bool AHEAD, bool ZERO, class Lds>
__device__ __forceinline__ void split_body(const SplitArgs& a, int64_t grp, Lds* lds) {
    constexpr int G = 64 / LPR;                 // lane groups per wavefront
    constexpr int LEN = CHUNK / G, NW = LEN / SUB;              // entries and flag words per group
    constexpr int UNR = 4;                      // entries fetched together
    static_assert(NW >= 1 && G > 1, "a group needs at least one flag word");

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c = grp * WAVES_PER_BLOCK + wave;
    if (c >= a.nchunks) return;                 // whole wavefront leaves; no block-wide barrier below
    const int g = lane / LPR, li = lane % LPR;
    int col0;
    const bool col_ok = lane_columns<LPR, VEC>(a.f, blockIdx.y, gridDim.y, li, &col0);
    const int64_t k0 = c * CHUNK, j0 = c * SUBS_PER_CHUNK;
    const int nk = a.nnz - k0 < CHUNK ? (int)(a.nnz - k0) : CHUNK;
    Lds& L = lds[wave];

    // ---- stage the chunk: indices, values, flags, the rows begun here ----
    uint32_t word = 0;
    if (lane <= SUBS_PER_CHUNK) word = a.flags[j0 + lane];      // padded by a chunk of zero words
    const int32_t q0 = a.sub_row[j0];           // row of the chunk's first entry
    int at = a.sub_row[j0 + g * NW];            // and of this group's first
    int32_t empty = 0;
    if constexpr (ZERO) empty = empty_row(a, c, lane);
    stage_chunk(a, k0, lane, L.col, L.val);
    if constexpr (ZERO) zero_share<LPR, VEC>(a, c, lane, empty, col0, col_ok);
    if (lane <= SUBS_PER_CHUNK) L.flag[lane] = word;
    const int32_t q1 = q0 + 1 - (int32_t)(__builtin_amdgcn_readfirstlane(word) & 1u);       // the first row begun here
    // each wavefront reads only what it wrote; LDS operations of one wavefront complete in order
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int begun = 0;                              // row starts of the chunk
#pragma unroll
    for (int w = 0; w < SUBS_PER_CHUNK; ++w) begun += __popc(L.flag[w]);
    begun = __builtin_amdgcn_readfirstlane(begun);
    at += 1 - (int)(L.flag[g * NW] & 1u) - q1;  // row starts of the chunk before this group's slice
    for (int i = lane; i < begun; i += 64) {
        const int32_t row = a.ne_rows ? a.ne_rows[q1 + i] : q1 + i;
        const bool raw = a.defer && a.defer[row];
        L.row[i] = row | (raw ? (int32_t)0x80000000 : 0);
        if (!a.val) L.val[i] = a.row_scale && !raw ? a.row_scale[row] : 1.f;
    }
    const bool continued = k0 + CHUNK < a.nnz && !(L.flag[SUBS_PER_CHUNK] & 1u);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // The mask of those rows, as bits: fetched when a row starts or ends, it drained the gathers in flight (hub schedule,
    // 33 M entries at 16 columns: 375 -> 333 us; 1.9 M at 64: 75 -> 64; 1.9 M at 41, k_spmm_line: 87 -> 71).  Not AHEAD: see
    // many_row_starts.
    const uint32_t mpitch = (uint32_t)a.ldzprev * 4u;
    if constexpr (EPI == GCN_EPI_MASK && AHEAD) {
        constexpr int AT_ONCE = 4, MB = Lds::MASK_BYTES;
        const int staged = begun < Lds::MASK_ROWS ? begun : Lds::MASK_ROWS;
        for (int i0 = g; i0 < staged; i0 += AT_ONCE * G) {
            float m[AT_ONCE][VEC];
#pragma unroll
            for (int t = 0; t < AT_ONCE; ++t) {
                const int i = i0 + t * G < staged ? i0 + t * G : i0;
                load_vec<VEC>(m[t], at_row(a.Zprev + col0, (uint32_t)L.row[i] & 0x7fffffffu, mpitch));
            }
#pragma unroll
            for (int t = 0; t < AT_ONCE; ++t) {
                const int i = i0 + t * G < staged ? i0 + t * G : i0;     // (the first again, with the same bits)
                if (t > 0 && i == i0) continue;
                if constexpr (VEC == 4) {
                    int bits = 0;
#pragma unroll
                    for (int u = 0; u < VEC; ++u) bits |= m[t][u] > 0.f ? 1 << u : 0;
                    bits |= __builtin_amdgcn_mov_dpp(bits, 0xf5, 0xf, 0xf, true) << 4;         // of the lane to the right
                    if (li % 2 == 0) L.mask[i * MB + li / 2] = (uint8_t)bits;
                } else {
                    const unsigned long long bits = __ballot(m[t][0] > 0.f);
                    if (li == 0) *reinterpret_cast<uint32_t*>(L.mask + i * MB) = (uint32_t)(bits >> (g * LPR));
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // ---- walk this group's slice ----
    float acc[VEC] = {};
    int through = 0;                            // the mask's bits of this lane's columns
    bool owned = false;                         // has this group seen a row start yet?
    int32_t row = 0;
    float scale = 1.f;
    const float* const xbase = a.X + col0;
    const uint32_t xpitch = (uint32_t)a.ldx * 4u, zpitch = (uint32_t)a.ldz * 4u;
    auto z_row = [&]() { return const_cast<float*>(at_row(a.Z + col0, (uint32_t)row & 0x7fffffffu, zpitch)); };
    float bias[VEC] = {};                       // in registers: a row's end must not wait for memory
    if constexpr (EPI == EPI_LAYER) {
        if (a.bias && col_ok) load_vec<VEC>(bias, a.bias + col0);
    }
    auto store_row = [&]() {
#pragma clang fp contract(off)                  // the bias is added to the rounded product (see layer_store)
        float v[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) v[u] = acc[u] * scale;    // exact for scale = 1, which a raw sum has
        if constexpr (EPI == GCN_EPI_RELU) {
#pragma unroll
            for (int u = 0; u < VEC; ++u) v[u] = v[u] > 0.f || row < 0 ? v[u] : 0.f;
        } else if constexpr (EPI == GCN_EPI_MASK && !AHEAD) {
            float m[VEC];
            load_vec<VEC>(m, at_row(a.Zprev + col0, (uint32_t)row & 0x7fffffffu, mpitch));
#pragma unroll
            for (int u = 0; u < VEC; ++u) v[u] = m[u] > 0.f || row < 0 ? v[u] : 0.f;
        } else if constexpr (EPI == GCN_EPI_MASK) {
#pragma unroll
            for (int u = 0; u < VEC; ++u) v[u] = through >> u & 1 || row < 0 ? v[u] : 0.f;
        }
        if constexpr (EPI == EPI_LAYER) {
            float r[VEC];
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                if (a.bias) v[u] = v[u] + bias[u];
                r[u] = v[u] > 0.f ? v[u] : 0.f;
                if (a.relu) v[u] = r[u];
            }
            if (a.H) store_vec<VEC>(const_cast<float*>(at_row(a.H + col0, (uint32_t)row & 0x7fffffffu, zpitch)), r);
        }
        store_vec<VEC>(z_row(), v);
    };
    auto start_row = [&]() {                    // an entry starts a row: close the fragment before it
        if (owned) store_row();
        else {
#pragma unroll
            for (int u = 0; u < VEC; ++u) L.head[lane * VEC + u] = acc[u];
        }
        owned = true;
        row = L.row[at];
        if (!a.val) scale = L.val[at];
        if constexpr (EPI == GCN_EPI_MASK && AHEAD) {
            if (at >= Lds::MASK_ROWS) {
                float m[VEC];
                load_vec<VEC>(m, at_row(a.Zprev + col0, (uint32_t)row & 0x7fffffffu, mpitch));
                through = 0;
#pragma unroll
                for (int u = 0; u < VEC; ++u) through |= m[u] > 0.f ? 1 << u : 0;
            } else if constexpr (VEC == 4) through = L.mask[at * Lds::MASK_BYTES + li / 2] >> (li % 2 * 4);
            else through = (int)(*reinterpret_cast<const uint32_t*>(L.mask + at * Lds::MASK_BYTES) >> li);
        }
        at += 1;
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = 0.f;
    };
    auto fetch = [&](int p, float (&x)[UNR][VEC]) {             // past the end: row 0
        const int4 cc = *reinterpret_cast<const int4*>(L.col + p + p / SUB * (SUB_STRIDE - SUB));
        load_vec<VEC>(x[0], at_row(xbase, (uint32_t)cc.x, xpitch));
        load_vec<VEC>(x[1], at_row(xbase, (uint32_t)cc.y, xpitch));
        load_vec<VEC>(x[2], at_row(xbase, (uint32_t)cc.z, xpitch));
        load_vec<VEC>(x[3], at_row(xbase, (uint32_t)cc.w, xpitch));
    };
    auto sums = [&](int p, const float (&x)[UNR][VEC], int end) {
        const uint32_t bits = L.flag[p / SUB] >> (p % SUB);
        float vs[UNR] = {1.f, 1.f, 1.f, 1.f};
        if (a.val) {
            const float4 vv = *reinterpret_cast<const float4*>(L.val + p + p / SUB * (SUB_STRIDE - SUB));
            vs[0] = vv.x; vs[1] = vv.y; vs[2] = vv.z; vs[3] = vv.w;
        }
#pragma unroll
        for (int e = 0; e < UNR; ++e) {
            if (p + e < end) {
                if (bits >> e & 1u) start_row();
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[u] = fmaf(vs[e], x[e][u], acc[u]);
            }
        }
    };
    if (col_ok) {
        float xa[UNR][VEC], xb[UNR][VEC];
        const int from = g * LEN, to = from + LEN;
        if (LPR > 4 && nk == CHUNK) {
            fetch(from, xa);
#pragma unroll 1
            for (int p = from; p < to; p += 2 * UNR) {
                fetch(p + UNR, xb);
                sums(p, xa, CHUNK);
                if (p + 2 * UNR < to) fetch(p + 2 * UNR, xa);
                sums(p + UNR, xb, CHUNK);
            }
        } else if (nk == CHUNK) {
#pragma unroll 1
            for (int p = from; p < to; p += UNR) { fetch(p, xa); sums(p, xa, CHUNK); }
        } else {                                // the last chunk
#pragma unroll 1
            for (int p = from; p < to; p += UNR) { fetch(p, xa); sums(p, xa, nk); }
        }
    }
    float R[VEC], T[VEC];                       // R: the entries before the first row start, all of them without one
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        R[v] = owned ? L.head[lane * VEC + v] : acc[v];
        if (!owned) acc[v] = 0.f;
        T[v] = 0.f;
    }
    int stop = owned ? 1 : 0, stop_next = 0;

    // ---- join fragments across groups: R_g = head_g + (owned_g ? 0 : R_{g+1}) ----
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
        float Rp[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) Rp[v] = __shfl_down(R[v], d * LPR, 64);
        const int sp = __shfl_down(stop, d * LPR, 64);
        if (g + d < G && !stop) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) R[v] += Rp[v];
            stop = sp;
        }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) T[v] = __shfl_down(R[v], LPR, 64);
    stop_next = __shfl_down(stop, LPR, 64);
    if (g == G - 1) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) T[v] = 0.f;
        stop_next = 0;
    }
    if (g == 0 && col_ok) store_vec<VEC>(a.carry + c * a.f + col0, R);

    if (owned && col_ok) {
        // the row opened last in this slice: add what later groups of this wavefront hold for it
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += T[v];
        if (!stop_next && continued) store_vec<VEC>(z_row(), acc);      // finished by k_spmm_fixup
        else store_row();
    }
}

template <int LPR, int VEC, int EPI, bool AHEAD = true, bool ZERO = false>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) void k_spmm_split(SplitArgs a) {
    __shared__ WaveLds<LPR, VEC, EPI == GCN_EPI_MASK && AHEAD> lds[WAVES_PER_BLOCK];
    split_body<LPR, VEC, EPI, AHEAD, ZERO>(a, chunk_group(a), lds);
}

// The same product for matrices of few chunks, which is a chain of memory latencies, launches and first executions of
// instructions that wait for each other.  A lane group fetches the 32 rows of X of a flag word at once, leaves them in LDS and
// walks them there; in the walk the end of a row is only noted (some of the 16 groups of a wavefront have one at
// nearly every step, and storing it there took longer than everything else), the rows are stored afterwards, one of every
// group at a time.  A row that ends in the chunk after the one it starts in is finished here: a workgroup takes
// three chunks, its fourth wavefront sums the head of the chunk behind them, and heads are passed to the wavefront before
// through LDS; a fix-up launch follows only when a row covers a whole further chunk.  The sums are those of
// k_spmm_split and k_spmm_fixup, term by term.  1000 rows of 17 entries at 16 columns: 9.7 + 3.9 -> 7.7 us.
template <int LPR, int EPI, bool ZERO>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) void k_spmm_few(SplitArgs a) {
    constexpr int VEC = 4;
    constexpr int G = 64 / LPR, NW = SUBS_PER_CHUNK / G, OWN = WAVES_PER_BLOCK - 1;
    extern __shared__ float4 s_x[];                             // [WAVES_PER_BLOCK][SUB][64]: entry e of every lane group
    __shared__ int32_t s_col[WAVES_PER_BLOCK][LDS_PER_WAVE];
    __shared__ float s_val[WAVES_PER_BLOCK][LDS_PER_WAVE];
    __shared__ float s_head[WAVES_PER_BLOCK][LPR * VEC];        // sum of the entries before the chunk's first row start
    __shared__ int s_starts[WAVES_PER_BLOCK];                   // whether the chunk has a row start at all
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane / LPR, li = lane % LPR;
    const int64_t c = (int64_t)blockIdx.x * OWN + wave;
    const bool active = c < a.nchunks, mine = active && wave < OWN;
    int col0;
    const bool col_ok = lane_columns<LPR, VEC>(a.f, blockIdx.y, gridDim.y, li, &col0);
    const int64_t k0 = c * CHUNK, j0 = c * SUBS_PER_CHUNK + (int64_t)g * NW;
    float acc[VEC] = {}, head[VEC] = {}, T[VEC] = {};
    int32_t q = 0;
    bool owned = false, runs_on = false;
    if (active) {
        // (flags is padded by a chunk of zero words)
        const bool continued = k0 + CHUNK < a.nnz && !(a.flags[(c + 1) * SUBS_PER_CHUNK] & 1u);
        uint32_t mask = a.flags[j0];
        q = a.sub_row[j0];
        int32_t empty = 0;
        if constexpr (ZERO) empty = empty_row(a, c, lane);
        int32_t* lc = s_col[wave];
        float* lv = s_val[wave];
#pragma unroll
        for (int t = 0; t < CHUNK / 256; ++t) {
            const int i = t * 256 + lane * 4;
            const int64_t k = k0 + i;
            int4 cc = make_int4(0, 0, 0, 0);
            float4 vv = make_float4(1.f, 1.f, 1.f, 1.f);        // value-free: only the column stream is read
            if (k + 4 <= a.nnz) {
                cc = *reinterpret_cast<const int4*>(a.colidx + k);
                if (a.val) vv = *reinterpret_cast<const float4*>(a.val + k);
            } else {
                if (k + 0 < a.nnz) { cc.x = a.colidx[k + 0]; if (a.val) vv.x = a.val[k + 0]; }
                if (k + 1 < a.nnz) { cc.y = a.colidx[k + 1]; if (a.val) vv.y = a.val[k + 1]; }
                if (k + 2 < a.nnz) { cc.z = a.colidx[k + 2]; if (a.val) vv.z = a.val[k + 2]; }
            }
            const int p = i + (i >> 5) * (SUB_STRIDE - SUB);
            *reinterpret_cast<int4*>(lc + p) = cc;
            *reinterpret_cast<float4*>(lv + p) = vv;
        }
        if (ZERO && wave < OWN) zero_share<LPR, VEC>(a, c, lane, empty, col0, col_ok);
        // each wavefront reads only what it wrote; LDS operations of one wavefront complete in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        q -= (int32_t)(mask & 1u);              // a start bit at the very first entry re-increments q
        float4* const lx = s_x + wave * (SUB * 64) + lane;
        const float* xbase = a.X + col0;
        for (int w = 0; w < NW; ++w) {
            if (w > 0) mask = a.flags[j0 + w];
            const int64_t left = a.nnz - (j0 + w) * SUB;
            const int cnt = left >= SUB ? SUB : (left > 0 ? (int)left : 0);
            const int base = (g * NW + w) * SUB_STRIDE;
            float x[SUB][VEC];
#pragma unroll
            for (int e = 0; e < SUB; ++e) load_vec<VEC>(x[e], at_row(xbase, (uint32_t)lc[base + e], (uint32_t)a.ldx * 4u));   // past the end: row 0
#pragma unroll
            for (int e = 0; e < SUB; ++e)
                lx[e * 64] = e < cnt ? make_float4(x[e][0], x[e][1], x[e][2], x[e][3]) : make_float4(0.f, 0.f, 0.f, 0.f);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // the walk: where an entry starts a row, the fragment before it takes the entry's place in LDS
#pragma unroll 1
            for (int b = 0; b < SUB; b += 8) {
                float4 xe[8];
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) { xe[e] = lx[(b + e) * 64]; v[e] = lv[base + b + e]; }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (mask >> (b + e) & 1u) {
                        lx[(b + e) * 64] = make_float4(acc[0], acc[1], acc[2], acc[3]);
                        acc[0] = acc[1] = acc[2] = acc[3] = 0.f;
                    }
                    acc[0] = fmaf(v[e], xe[e].x, acc[0]); acc[1] = fmaf(v[e], xe[e].y, acc[1]);
                    acc[2] = fmaf(v[e], xe[e].z, acc[2]); acc[3] = fmaf(v[e], xe[e].w, acc[3]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // the fragments: the first belongs to a row begun earlier, the others are whole rows
            for (uint32_t m = mask; m; m &= m - 1) {
                const float4 f4 = lx[(__ffs(m) - 1) * 64];
                float frag[VEC] = {f4.x, f4.y, f4.z, f4.w};
                if (!owned) {
#pragma unroll
                    for (int u = 0; u < VEC; ++u) head[u] = frag[u];
                    owned = true;
                } else if (col_ok && mine) {
                    const int64_t row = a.ne_rows ? a.ne_rows[q] : q;
                    epilogue_store<VEC, EPI>(a.Z + row * a.ldz + col0,
                                             EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col0 : nullptr, frag,
                                             a.row_scale ? a.row_scale[row] : 1.f, a.defer && a.defer[row]);
                }
                q += 1;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (!owned) {                           // the whole slice lies inside one row
#pragma unroll
            for (int v = 0; v < VEC; ++v) { head[v] = acc[v]; acc[v] = 0.f; }
        }
        // join fragments across groups: R_g = head_g + (owned_g ? 0 : R_{g+1}), left in head
        int stop = owned ? 1 : 0;
#pragma unroll
        for (int d = 1; d < G; d <<= 1) {
            float Rp[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) Rp[v] = __shfl_down(head[v], d * LPR, 64);
            const int sp = __shfl_down(stop, d * LPR, 64);
            if (g + d < G && !stop) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) head[v] += Rp[v];
                stop = sp;
            }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) T[v] = __shfl_down(head[v], LPR, 64);
        int stop_next = __shfl_down(stop, LPR, 64);
        if (g == G - 1) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) T[v] = 0.f;
            stop_next = 0;
        }
        runs_on = !stop_next && continued;
        if (g == 0) {
            if (a.n_fix > 0 && col_ok && mine) store_vec<VEC>(a.carry + c * a.f + col0, head);
#pragma unroll
            for (int v = 0; v < VEC; ++v) s_head[wave][li * VEC + v] = head[v];
            if (li == 0) s_starts[wave] = stop;
        }
    }
    __syncthreads();
    if (owned && col_ok && mine) {
        // the row opened last in this slice: add what later groups of this wavefront hold for it, then the next chunk
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += T[v];
        if (runs_on && s_starts[wave + 1]) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] += s_head[wave + 1][li * VEC + v];
            runs_on = false;
        }
        const int64_t row = a.ne_rows ? a.ne_rows[q] : q;
        if (runs_on) store_vec<VEC>(a.Z + row * a.ldz + col0, acc);     // finished by k_spmm_fixup
        else epilogue_store<VEC, EPI>(a.Z + row * a.ldz + col0,
                                      EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col0 : nullptr, acc,
                                      a.row_scale ? a.row_scale[row] : 1.f, a.defer && a.defer[row]);
    }
}

// Matrices of few rows, all of them short (SHORT_ROW entries at the most): a lane group takes a row, one wavefront per
// workgroup so that a thousand rows spread over 63 compute units.  Nothing is staged or joined: the chain is
// indices, gathers, sums, store, and an empty row is simply a sum of nothing.  The rows lie at an equal pitch (build_short),
// so that the indices do not wait for row pointers.  Eight entries a round, the gathers of the next round sent out as those of
// this one are used: a kernel of a few microseconds pays for every line of its code, which no cache holds when it starts, and 32
// entries unrolled took longer for their 6.6 KB than for their one latency.  The sums are those of the nonzero-split kernels,
// term by term: there a row is cut where a lane group's slice of SLICE entries or a chunk ends, and with at most SHORT_ROW entries
// it has three pieces, F + (H1 + H2), or (F + H1) + H2 when H2 is in the next chunk.
// Microseconds at 16 columns, traced: 1000 rows of 17 entries 6.3, k_spmm_few 7.7, k_spmm_split 9.7 and k_spmm_fixup 3.9.  With row
// pointers and 32 entries a round -> now, one of many in a graph, where an empty kernel takes 2.05: 1000 rows of 17 4.9 -> 4.4, of 40
// 7.9 -> 6.0, of 64 9.3 -> 8.0, 30 K of 17 8.1 -> 7.6.  Called one by one the host takes longer (5.8 a call, 4.15 of it a launch).
// The value of lane `l` of every group of LPR lanes (l a constant once the loop around is unrolled).
template <int LPR>
__device__ __forceinline__ int group_lane(int x, int l) {
    if constexpr (LPR == 4) {                   // inside four lanes without the LDS
        switch (l) {
            case 0: return __builtin_amdgcn_mov_dpp(x, 0x00, 0xf, 0xf, true);
            case 1: return __builtin_amdgcn_mov_dpp(x, 0x55, 0xf, 0xf, true);
            case 2: return __builtin_amdgcn_mov_dpp(x, 0xaa, 0xf, 0xf, true);
            default: return __builtin_amdgcn_mov_dpp(x, 0xff, 0xf, 0xf, true);
        }
    }
    return __shfl(x, l, LPR);
}

// What is next to the rows (RowsNext) is done by the wavefront that made them, 16 rows of up to 16 columns: as a kernel of its own it
// would run for four microseconds, most of it its start and one chain of latencies, of which all but the stores happen here beside the walk.
// The matrix instructions and the sums of a row's exponentials are those of k_gemm_tall and k_softmax_nll, bit for bit.  Epochs: 64-16-8 on 4096
// rows of 17 entries 53 -> 42.5 us (11 launches, now 8), 64-16-16-8 on 1000 67 -> 54, 100-16-4 on 30000 63 -> 53.
//
// The weight gradient H^T Z of up to 64 x 16 (MT tiles of 16 columns of H, fetched before the walk) takes workgroups of four of them, whose sums
// are added up as k_gemm_tn and k_gemm_tn_narrow do it over 64 rows.  It makes the kernel 1 to 2 us longer and saves a launch per layer: epochs of
// 64-16-8 on 4096 vertices 38.7 -> 34.4 us, 64-16-16-8 54.7 -> 49.9, 50-16-12 on 10 K 45.9 -> 39.9, 100-16-4 on 30 K 56.6 -> 54.2.  Workgroups of
// eight wavefronts, whose partial results are half as many, took 4 us longer each: fewer compute units fetch the rows.  (The rows of Z, an epoch's S, are stored there
// too, although nothing reads them then.)
struct NoNext {};                                 // (the plain product has nothing to be told of what is next; in time there is no difference)
template <int NEXT>
using NextArgs = std::conditional_t<NEXT == RowsNext::NONE, NoNext, RowsNext>;
template <int LPR, int SLICE, int EPI, int NEXT = RowsNext::NONE, int MT = 1>
__global__ __launch_bounds__(NEXT & RowsNext::GRAD ? 256 : 64) void k_spmm_short(SplitArgs a, int64_t nrows, const int32_t* __restrict__ rows,
                                                                                 int32_t pitch, NextArgs<NEXT> nx) {
    constexpr int VEC = 4;
    constexpr bool GRAD = (NEXT & RowsNext::GRAD) != 0;
    static_assert(NEXT == RowsNext::NONE || LPR == 4, "16 rows of a wavefront");
    static_assert(SHORT_ROW <= 2 * SLICE, "at most three pieces");
    constexpr int U = 8, OWN = LPR < U ? U / LPR : 1;           // entries per round, those that a lane holds the indices of
    const int lane = threadIdx.x & 63, li = lane % LPR, wave = GRAD ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int64_t unit = GRAD ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    const int64_t row = (unit * 64 + lane) / LPR;
    int col0;
    const bool col_ok = lane_columns<LPR, VEC>(a.f, blockIdx.y, gridDim.y, li, &col0);
    const int64_t own = row < nrows ? row : nrows - 1;
    const int32_t* const cols = a.colidx + own * pitch + li * OWN;
    const float* const vals = a.val ? a.val + own * pitch + li * OWN : nullptr;
    const int32_t packed = rows[own];
    struct Round { int32_t c[OWN]; float v[OWN]; };
    auto indices = [&](int base, Round& r) {
#pragma unroll
        for (int t = 0; t < OWN; ++t) { r.c[t] = 0; r.v[t] = 1.f; }
        if (li * OWN < U && base + li * OWN < pitch) {          // (pitch is a multiple of four)
            __builtin_memcpy(r.c, cols + base, sizeof r.c);
            if (vals) __builtin_memcpy(r.v, vals + base, sizeof r.v);
        }
    };
    const float* const xbase = a.X + col0;
    const uint32_t xpitch = (uint32_t)a.ldx * 4u;
    Round now, next;
    float x[U][VEC];
    auto gather = [&](const Round& r, int e) { load_vec<VEC>(x[e], at_row(xbase, (uint32_t)group_lane<LPR>(r.c[e % OWN], e / OWN), xpitch)); };
    indices(0, now);
    indices(U, next);
#pragma unroll
    for (int e = 0; e < U; ++e) gather(now, e);
    // the next product's operands: lane (r, kq) holds rows 4 kq .. 4 kq + 3 of column r of op(W), and four columns of row r of the mask
    const int r = lane & 15, kq = lane >> 4;
    const int64_t next_row = unit * 16 + r;
    float w[4] = {}, mask[4] = {1.f, 1.f, 1.f, 1.f}, h[MT][4];
    int32_t label = -1;
    if constexpr (GRAD) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int64_t hr = unit * 16 + 4 * s + kq;
                h[t][s] = hr < nrows && 16 * t + r < nx.M ? nx.H[hr * nx.ldh + 16 * t + r] : 0.f;
            }
    }
    if constexpr ((NEXT & RowsNext::GEMM) != 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * kq + e < a.f && r < nx.N) w[e] = nx.transposed ? nx.W[r * a.f + 4 * kq + e] : nx.W[(4 * kq + e) * nx.N + r];
        if (nx.mask && next_row < nrows && 4 * kq < nx.N) load_vec<4>(mask, nx.mask + next_row * nx.N + 4 * kq);
    }
    if constexpr (NEXT == RowsNext::LOSS) {
        if (row < nrows) label = nx.labels[row];
    }
    const int len = row < nrows ? packed & 0xffff : 0, rs = packed >> 16;           // rs: modulo CHUNK, and so modulo SLICE
    const int b1 = SLICE - (rs & (SLICE - 1)), b2 = b1 + SLICE;                     // where the second and the third piece begin
    const bool third_apart = ((rs + b2) & (CHUNK - 1)) == 0;
    float acc[VEC] = {}, first[VEC] = {}, second[VEC] = {};
#pragma unroll 1
    for (int base = 0; __any(base < len); base += U) {
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const float ve = __int_as_float(group_lane<LPR>(__float_as_int(now.v[e % OWN]), e / OWN));
            const int k = base + e;
            const bool cut = k == b1 || k == b2;                // (first and second are used where the row goes on beyond b1 and b2)
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                first[u] = k == b1 ? acc[u] : first[u];
                second[u] = cut ? acc[u] : second[u];
                const float sum = fmaf(ve, x[e][u], cut ? 0.f : acc[u]);
                acc[u] = k < len ? sum : acc[u];
            }
            gather(next, e);                    // of the round after this one; past the end: row 0, not used
        }
        now = next;
        indices(base + 2 * U, next);
    }
    if (NEXT == RowsNext::NONE && (row >= nrows || !col_ok)) return;
    if (len > b2) {
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = third_apart ? (first[u] + second[u]) + acc[u] : first[u] + (second[u] + acc[u]);
    } else if (len > b1) {
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = first[u] + acc[u];
    }
    const bool mine = row < nrows && col_ok;
    if (mine) epilogue_store<VEC, EPI>(a.Z + row * a.ldz + col0, EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col0 : nullptr, acc,
                                       a.row_scale ? a.row_scale[row] : 1.f, a.defer && a.defer[row]);
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    if constexpr (GRAD) {
        constexpr int ST = 20;                  // row stride of a wavefront's tile
        __shared__ float s_rows[4][16 * ST];
        __shared__ float4 s_sum[4][MT][64];
        float* const tile = s_rows[wave];
        *reinterpret_cast<float4*>(tile + (lane >> 2) * ST + 4 * li) =
            mine ? make_float4(acc[0], acc[1], acc[2], acc[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float z[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) z[s] = tile[(4 * s + kq) * ST + r];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            floatx4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) y = __builtin_amdgcn_mfma_f32_16x16x4f32(h[t][s], z[s], y, 0, 0, 0);
            s_sum[wave][t][lane] = make_float4(y[0], y[1], y[2], y[3]);
        }
        __syncthreads();
        if (wave < MT) {
            const float4 p = s_sum[0][wave][lane], q = s_sum[1][wave][lane], u = s_sum[2][wave][lane], v = s_sum[3][wave][lane];
            const float sum[4] = {((p.x + q.x) + u.x) + v.x, ((p.y + q.y) + u.y) + v.y, ((p.z + q.z) + u.z) + v.z, ((p.w + q.w) + u.w) + v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 16 * wave + 4 * kq + e;
                if (m < nx.M && r < a.f) nx.ypart[((int64_t)blockIdx.x * nx.M + m) * a.f + r] = sum[e];
            }
        }
    }
    if constexpr ((NEXT & RowsNext::GEMM) != 0) {               // (all lanes)
        floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float ae = __shfl(mine ? acc[e] : 0.f, r * 4 + kq, 64);
            t = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], ae, t, 0, 0, 0);
        }
        if (next_row < nrows && 4 * kq < nx.N) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = mask[e] > 0.f ? t[e] : 0.f;
            store_vec<4>(nx.T + next_row * nx.N + 4 * kq, v);
        }
    }
    if constexpr (NEXT == RowsNext::LOSS) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = mine ? acc[e] : -INFINITY;
        float m = v[0];
#pragma unroll
        for (int e = 1; e < 4; ++e) m = fmaxf(m, v[e]);
        m = fmaxf(m, __shfl_xor(m, 2, 64));
        m = fmaxf(m, __shfl_xor(m, 1, 64));
        float p[4], sum = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = expf(v[e] - m);              // exp(-inf) = 0 behind the last class
            sum += p[e];
        }
        sum += __shfl_xor(sum, 2, 64);
        sum += __shfl_xor(sum, 1, 64);
        const float lse = m + logf(sum);
        const bool labelled = label >= 0;
        const int y = label >= a.f ? a.f - 1 : label;           // labels >= C are the caller's error; stay in bounds
        double loss = 0.0;
        if (mine) {
            float d[4], zy = 0.f;
            const float inv = 1.f / sum;        // (as k_softmax_nll)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d[e] = labelled ? (p[e] * inv - (col0 + e == y ? 1.f : 0.f)) * nx.inv_m : 0.f;
                zy = col0 + e == y ? v[e] : zy;
            }
            store_vec<4>(nx.G + row * a.f + col0, d);
            if (labelled && y >= col0 && y < col0 + 4) loss = (double)lse - (double)zy;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) loss += __shfl_xor(loss, d, 64);
        if (lane == 0) nx.part[unit] = loss;
    }
}

// Widths above 32 that are no multiple of four, few chunks.  They used to run with one float per lane, a wavefront adding up a
// chunk of 512 entries on its own.  Here a workgroup of 256 takes a chunk in two halves: all
// lanes fetch the half's rows of X (16 bytes per lane, `lanes` lanes per row, the last one repeating some columns) into LDS,
// 16 rows per lane group in flight; then the lane groups take the rows of the result, one after another, and walk
// their entries in LDS.  A row's part in a chunk stays one serial sum, as it was, so every sum keeps its order and
// with it the sign that a ReLU further on may decide by.  41 columns, 0.6 M entries: 76 -> 33 us.
static constexpr int HALF = CHUNK / 2;

template <int EPI>
__global__ __launch_bounds__(256, 3) void k_spmm_ragged(SplitArgs a, int lanes) {
    constexpr int VEC = 4, NE = 16;                             // most rows of X a lane group fetches per half
    constexpr int LONG = 24;                                    // parts from here on go to a whole wavefront
    extern __shared__ float4 s_x[];                             // [HALF][lanes]
    __shared__ int32_t s_col[HALF];
    __shared__ float s_val[HALF];
    __shared__ int s_pos[HALF + 2];                             // where the parts of rows begin; their number behind them
    __shared__ int s_cnt[4];
    __shared__ float s_open[3][64];                             // the sum that goes on into a half
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int groups = 256 / lanes, grp = tid / lanes, li = tid - grp * lanes;
    const bool works = grp < groups;
    const int64_t c = blockIdx.x;
    int col0;
    const bool col_ok = lane_columns<16, VEC>(a.f, blockIdx.y, gridDim.y, li, &col0) && works;
    const float* const xbase = a.X + col0;
    // the panel's columns first .. first + width - 1, and where a single lane finds column `lane` of them in a row of s_x
    // (those behind the last whole four sit in the place of the lane that repeats columns)
    int first = 0;
    lane_columns<16, VEC>(a.f, blockIdx.y, gridDim.y, 0, &first);
    int last4 = 0;
    lane_columns<16, VEC>(a.f, blockIdx.y, gridDim.y, lanes - 1, &last4);
    const int width = last4 + VEC - first, pitch = lanes * VEC;
    const int whole = width / VEC * VEC, slot = lane < whole ? lane : whole + lane - (width - VEC);
    if (tid < 64) s_open[0][tid] = 0.f;
    int owned = 0;                                              // row starts of this chunk so far
    int half = 0;
    int32_t q = 0;                                              // row of the half's part 0
    auto store_row = [&](int32_t r, int col, auto& v) {
        constexpr int N = sizeof(v) / sizeof(float);
        const int64_t row = a.ne_rows ? a.ne_rows[r] : r;
        epilogue_store<N, EPI>(a.Z + row * a.ldz + col, EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col : nullptr, v,
                               a.row_scale ? a.row_scale[row] : 1.f, a.defer && a.defer[row]);
    };
    for (; half < 2; ++half) {
        const int64_t k0 = c * CHUNK + half * HALF;
        if (k0 >= a.nnz) break;
        const int cnt = a.nnz - k0 < HALF ? (int)(a.nnz - k0) : HALF;
        const int64_t j0 = k0 / SUB;
        bool start = false;
        if (tid < cnt) {
            s_col[tid] = a.colidx[k0 + tid];
            s_val[tid] = a.val ? a.val[k0 + tid] : 1.f;
            start = a.flags[j0 + (tid >> 5)] >> (tid & 31) & 1u;
        }
        q = a.sub_row[j0] - (int32_t)(a.flags[j0] & 1u);
        const unsigned long long starts = __ballot(start);
        if (lane == 0) s_cnt[wave] = __popcll(starts);
        __syncthreads();
        int before = __popcll(starts & ((1ull << lane) - 1ull)), np = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) before += s_cnt[w];
            np += s_cnt[w];
        }
        if (start) s_pos[before + 1] = tid;
        if (tid == 0) { s_pos[0] = 0; s_pos[np + 1] = cnt; }
        {
            float x[NE][VEC];
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int e = grp + i * groups;
                if (works && e < cnt) load_vec<VEC>(x[i], at_row(xbase, (uint32_t)s_col[e], (uint32_t)a.ldx * 4u));
            }
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int e = grp + i * groups;
                if (works && e < cnt) s_x[e * lanes + li] = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
            }
        }
        __syncthreads();
        // Long parts: a wavefront takes one, a column per lane (one addition per entry instead of four in a row).
        const float* const xs = reinterpret_cast<const float*>(s_x);
        for (int p = wave; p <= np; p += 4) {
            const int beg = s_pos[p], end = s_pos[p + 1];
            if (end - beg < LONG || lane >= width) continue;
            float acc = p == 0 ? s_open[half][lane] : 0.f;
            int e = beg;
            const float* xc = xs + (size_t)e * pitch + slot;
            for (; e + 16 <= end; e += 16, xc += 16 * pitch) {
                float x[16], v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) { x[i] = xc[i * pitch]; v[i] = s_val[e + i]; }
#pragma unroll
                for (int i = 0; i < 16; ++i) acc = fmaf(v[i], x[i], acc);
            }
            for (; e < end; ++e, xc += pitch) acc = fmaf(s_val[e], *xc, acc);
            float out[1] = {acc};
            if (p == np) s_open[half + 1][lane] = acc;
            else if (p > 0 || owned) store_row(q + p, first + lane, out);
            else a.carry[c * a.f + first + lane] = acc;
        }
        // Short parts: a lane group takes one, four columns per lane.
        for (int p = grp; works && p <= np; p += groups) {
            const int end = s_pos[p + 1];
            int e = s_pos[p];
            if (end - e >= LONG) continue;
            float acc[VEC] = {};
            if (p == 0) {
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[u] = s_open[half][col0 - first + u];
            }
#pragma unroll 2
            for (; e < end; ++e) {
                const float4 x = s_x[e * lanes + li];
                const float v = s_val[e];
                acc[0] = fmaf(v, x.x, acc[0]); acc[1] = fmaf(v, x.y, acc[1]);
                acc[2] = fmaf(v, x.z, acc[2]); acc[3] = fmaf(v, x.w, acc[3]);
            }
            if (!col_ok) continue;
            if (p == np) {
#pragma unroll
                for (int u = 0; u < VEC; ++u) s_open[half + 1][col0 - first + u] = acc[u];
            }
            else if (p > 0 || owned) store_row(q + p, col0, acc);
            else store_vec<VEC>(a.carry + c * a.f + col0, acc);         // the entries before the chunk's first row start
        }
        owned += np;
        q += np;
        __syncthreads();
    }
    if (tid >= width) return;
    float acc[1] = {s_open[half][tid]};
    if (!owned) {                                               // the whole chunk lies inside one row
        a.carry[c * a.f + first + tid] = acc[0];
        return;
    }
    const int64_t knext = (c + 1) * CHUNK;
    const bool continued = knext < a.nnz && !(a.flags[(c + 1) * SUBS_PER_CHUNK] & 1u);
    if (continued) {                                            // finished by k_spmm_fixup
        const int64_t row = a.ne_rows ? a.ne_rows[q] : q;
        a.Z[row * a.ldz + first + tid] = acc[0];
    } else store_row(q, first + tid, acc);
}

// The same for more chunks: one wavefront per chunk and panel of 64 * VEC columns, a row of X per instruction.  An entry is
// the same for all lanes, so its index, value, row address and the test for a row start are scalar work (indices and
// values come through the scalar cache, 16 at a time, nothing is staged), and the vector unit has one multiply-add per entry
// and column.  The rows of 16 entries are on their way while the 16 before them are summed.  The rows begun in the chunk are
// kept 64 at a time, one per lane.  Bound by the L2s' rate or line fills where there are a few thousand chunks.  41 columns, 1.9 M
// entries: 85 -> 57 us (16 lanes of 16 bytes per chunk, four chunks per wavefront), 12 M: 236 -> 196, 33 M: 918 -> 897; 67
// columns, 33 M: 1.71 -> 1.32 ms.
template <int VEC, int EPI>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) void k_spmm_line(SplitArgs a) {
    constexpr int UNR = VEC == 2 && EPI == GCN_EPI_MASK ? 8 : 16;      // (with 16 the masked form of two columns runs out of scalar registers)
    typedef int32_t Ints __attribute__((ext_vector_type(UNR)));
    typedef float Floats __attribute__((ext_vector_type(UNR)));
    typedef int32_t i16v __attribute__((ext_vector_type(16)));
    typedef const __attribute__((address_space(4))) int32_t* ConstI;        // read-only while the kernel runs
    typedef const __attribute__((address_space(4))) float* ConstF;
    typedef const __attribute__((address_space(4))) i16v* ConstI16;
    typedef const __attribute__((address_space(4))) Ints* ConstInts;
    typedef const __attribute__((address_space(4))) Floats* ConstFloats;
    typedef const __attribute__((address_space(1))) char* Global;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c = chunk_group(a) * WAVES_PER_BLOCK + wave;
    if (c >= a.nchunks) return;
    int col0;                                   // (lanes without columns follow the last one that has some)
    const bool col_ok = lane_columns<64, VEC>(a.f, blockIdx.y, gridDim.y, lane, &col0);
    if constexpr (VEC == 1) zero_share<64, VEC>(a, c, lane, empty_row(a, c, lane), col0, col_ok);
    const int64_t k0 = c * CHUNK;
    const int nk = a.nnz - k0 < CHUNK ? (int)(a.nnz - k0) : CHUNK;
    const ConstI cols = (ConstI)(uintptr_t)(a.colidx + k0), flags = (ConstI)(uintptr_t)(a.flags + c * SUBS_PER_CHUNK);
    const ConstF vals = (ConstF)(uintptr_t)(a.val ? a.val + k0 : nullptr);
    const bool continued = k0 + CHUNK < a.nnz && !(flags[SUBS_PER_CHUNK] & 1);     // (padded by a chunk of zero words)
    const uint32_t xpitch = (uint32_t)a.ldx * 4u, zpitch = (uint32_t)a.ldz * 4u, mpitch = (uint32_t)a.ldzprev * 4u;
    // rows begun here: numbers, factors and mask bits of 64 of them
    const int32_t q1 = ((ConstI)(uintptr_t)a.sub_row)[c * SUBS_PER_CHUNK] + 1 - (flags[0] & 1);
    int begun = 0;
    if constexpr (EPI == GCN_EPI_MASK) {
        const i16v all = *(ConstI16)flags;
#pragma unroll
        for (int w = 0; w < SUBS_PER_CHUNK; ++w) begun += __popc((uint32_t)all[w]);
    }
    int32_t rows = 0, at = 0, named = 0;        // 64 rows from the named-th on
    float factors = 1.f;
    int32_t low[VEC] = {}, high[VEC] = {};
    auto name_rows = [&]() {
        const int64_t q = (int64_t)q1 + at + lane, last = a.n_ne - 1;
        rows = (int32_t)(q < last ? q : last);
        if (a.ne_rows) rows = a.ne_rows[rows];
        if constexpr (EPI == GCN_EPI_MASK) {    // a lane keeps its row's bits of all lanes
            constexpr int AT_ONCE = 8;
            const int count = begun - at < 64 ? begun - at : 64;
            for (int i = 0; i < count; i += AT_ONCE) {
                float t[AT_ONCE][VEC];
#pragma unroll
                for (int j = 0; j < AT_ONCE; ++j)
                    load_vec<VEC>(t[j], at_row(a.Zprev, (uint32_t)__builtin_amdgcn_readlane(rows, i + j), mpitch) + (uint32_t)col0);
#pragma unroll
                for (int j = 0; j < AT_ONCE; ++j)
#pragma unroll
                    for (int u = 0; u < VEC; ++u) {
                        const unsigned long long bits = __ballot(t[j][u] > 0.f);
                        low[u] = lane == i + j ? (int32_t)bits : low[u];
                        high[u] = lane == i + j ? (int32_t)(bits >> 32) : high[u];
                    }
            }
        }
        const bool raw = a.defer && a.defer[rows];
        factors = a.row_scale && !raw ? a.row_scale[rows] : 1.f;
        rows |= raw ? (int32_t)0x80000000 : 0;
        asm volatile("" : "+v"(rows), "+v"(factors));        // fetched here, so that no later use has to wait for memory
        named = at;
    };
    name_rows();
    float acc[VEC] = {}, head[VEC] = {};
    unsigned long long through[VEC] = {};
    bool owned = false;
    int32_t row = 0;
    float scale = 1.f;
    auto z_row = [&]() { return const_cast<float*>(at_row(a.Z, (uint32_t)row & 0x7fffffffu, zpitch)) + (uint32_t)col0; };
    auto store_row = [&]() {
        if (!col_ok) return;
        float v[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) v[u] = acc[u] * scale;    // exact for scale = 1, which a raw sum has
        if constexpr (EPI == GCN_EPI_RELU) {
#pragma unroll
            for (int u = 0; u < VEC; ++u) v[u] = v[u] > 0.f || row < 0 ? v[u] : 0.f;
        } else if constexpr (EPI == GCN_EPI_MASK) {
#pragma unroll
            for (int u = 0; u < VEC; ++u) v[u] = through[u] >> lane & 1 || row < 0 ? v[u] : 0.f;
        }
        store_vec<VEC>(z_row(), v);
    };
    auto start_row = [&]() {
        if (owned) store_row();
        else {
#pragma unroll
            for (int u = 0; u < VEC; ++u) head[u] = acc[u];
        }
        owned = true;
        row = __builtin_amdgcn_readlane(rows, at - named);
        scale = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(factors), at - named));
        if constexpr (EPI == GCN_EPI_MASK) {
#pragma unroll
            for (int u = 0; u < VEC; ++u)
                through[u] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane(high[u], at - named) << 32 |
                             (uint32_t)__builtin_amdgcn_readlane(low[u], at - named);
        }
        at += 1;
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = 0.f;
    };
    auto load_x = [&](float (&x)[VEC], int32_t j) {             // a scalar address, the lane's column as the offset
        uint64_t row = (uint64_t)(uintptr_t)a.X + (uint64_t)(uint32_t)j * xpitch;
        uint32_t column = (uint32_t)col0 * 4u;
        asm("" : "+s"(row), "+v"(column));
        load_vec<VEC>(x, (const float*)(const Global)((const Global)row + column));
    };
    // A trip's indices, and the values of the trip before it with their row starts, are fetched a trip before they are used: through the
    // scalar cache too they come from memory, and asked for when needed every trip waited for that twice (with the fix-up: 1.9 M entries at 41
    // columns 55 -> 50.5 us, masked 67 -> 61.5; 0.7 M in rows of 7 46 -> 35; 1 M at 101 48 -> 42; 29 M at 45, bound by line fills,
    // 738 -> 727).  (Past the chunk's last whole trip: that one again.)
    const int whole = nk / UNR * UNR;
    struct Scalars { Ints cc; Floats vv; uint32_t bits; };
    Scalars n;
#pragma unroll
    for (int e = 0; e < UNR; ++e) n.vv[e] = 1.f;
    auto ahead = [&](int p) {                                   // indices of trip p, values and starts of the one before
        const int q = p < whole ? p : whole - UNR, r = p - UNR < whole ? p - UNR : whole - UNR;
        n.cc = *(ConstInts)(cols + q);
        if (vals) n.vv = *(ConstFloats)(vals + r);
        n.bits = (uint32_t)flags[r / SUB] >> (r % SUB);
    };
    auto fetch = [&](Ints cc, float (&x)[UNR][VEC]) {
#pragma unroll
        for (int e = 0; e < UNR; ++e) load_x(x[e], cc[e]);
    };
    auto sums = [&](Floats vv, uint32_t bits, const float (&x)[UNR][VEC]) {
        if (at - named + UNR > 64) name_rows();
#pragma unroll
        for (int e = 0; e < UNR; ++e) {
            if (bits >> e & 1u) start_row();
#pragma unroll
            for (int u = 0; u < VEC; ++u) acc[u] = fmaf(vv[e], x[e][u], acc[u]);
        }
    };
    float xa[UNR][VEC], xb[UNR][VEC];
    int p = 0;
    if (whole > 0) {
        const Ints cc = *(ConstInts)cols;
        fetch(cc, xa);
        ahead(UNR);
#pragma unroll 1
        for (;;) {
            auto half = [&](float (&now)[UNR][VEC], float (&next)[UNR][VEC]) {
                const Floats vv = n.vv;
                const uint32_t bits = n.bits;
                if (p + UNR < whole) fetch(n.cc, next);
                ahead(p + 2 * UNR);
                __builtin_amdgcn_sched_barrier(0);
                sums(vv, bits, now);
                p += UNR;
            };
            half(xa, xb);
            if (p == whole) break;
            half(xb, xa);
            if (p == whole) break;
        }
    }
#pragma unroll 1
    for (; p < nk; ++p) {                       // the end of the last chunk
        float x[VEC];
        load_x(x, cols[p]);
        if (at - named == 64) name_rows();
        if ((uint32_t)flags[p / SUB] >> (p % SUB) & 1u) start_row();
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = fmaf(vals ? vals[p] : 1.f, x[u], acc[u]);
    }
    if (!col_ok) return;
    store_vec<VEC>(a.carry + c * a.f + col0, owned ? head : acc);       // without a row start the whole chunk is inside one row
    if (owned) {
        if (continued) store_vec<VEC>(z_row(), acc);            // finished by k_spmm_fixup
        else store_row();
    }
}

// Two matrices in one launch: of every ra + rb consecutive workgroups the first ra work on `a` (with
// the epilogue) and the other rb on `b` (plain sums).  Used when one part is bound by line fills and
// the other by L2 hits, so that both kinds of work are resident on every compute unit together.
template <int LPR, int VEC, int EPI>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) void k_spmm_split_pair(SplitArgs a, SplitArgs b, int ra, int rb) {
    // ra + rb == 8.  Workgroups go to the eight XCDs round-robin; the rotation by q lets every XCD see
    // both kinds of work in turn.
    __shared__ WaveLds<LPR, VEC, EPI == GCN_EPI_MASK> lds[WAVES_PER_BLOCK];
    const unsigned q = blockIdx.x / 8, r = (blockIdx.x + q) % 8;
    if ((int)r < ra) split_body<LPR, VEC, EPI, true, true>(a, (int64_t)q * ra + r, lds);
    else split_body<LPR, VEC, GCN_EPI_NONE, true, false>(b, (int64_t)q * rb + (r - ra), lds);
}

// Adds, in ascending chunk order, the carries of the chunks a row runs on into, then applies the epilogue.  One LPR-lane
// group per such row; its record (x, y: the first and the last chunk it runs on into, z: the row) was worked out when
// the schedule was built, so that the carries and the row's sum so far are fetched right away.  A row of 60 K entries
// has 120 carries: eight are in flight at a time, the additions stay in order.
template <int LPR, int VEC, int EPI>
__device__ __forceinline__ void fixup_body(const SplitArgs& a, int64_t block) {
    const int64_t t = block * 256 + threadIdx.x;
    const int li = (int)(t % LPR);
    if (t / LPR >= a.n_fix) return;
    const int col0 = blockIdx.y * (LPR * VEC) + li * VEC;
    if (col0 >= a.f) return;
    const int4 rec = a.fix_list[t / LPR];
    const int64_t row = a.ne_rows ? a.ne_rows[rec.z] : rec.z;
    float* z = a.Z + row * a.ldz + col0;
    float cur[VEC], sum[VEC];
    load_vec<VEC>(cur, z);
#pragma unroll
    for (int v = 0; v < VEC; ++v) sum[v] = 0.f;
    const float* part = a.carry + (int64_t)rec.x * a.f + col0;
    int left = rec.y - rec.x + 1;
    for (; left >= 8; left -= 8) {
        float x[8][VEC];
#pragma unroll
        for (int e = 0; e < 8; ++e) load_vec<VEC>(x[e], part + (int64_t)e * a.f);
        part += (int64_t)8 * a.f;
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] += x[e][v];
    }
    for (; left > 0; --left) {
        float x[VEC];
        load_vec<VEC>(x, part);
        part += a.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[v] += x[v];
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) cur[v] += sum[v];
    const float scale = a.row_scale ? a.row_scale[row] : 1.f;
    if constexpr (EPI == EPI_LAYER)
        layer_store<VEC>(z, a.H ? a.H + row * a.ldz + col0 : nullptr, a.bias ? a.bias + col0 : nullptr, a.relu, cur, scale);
    else epilogue_store<VEC, EPI>(z, EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col0 : nullptr, cur, scale, a.defer && a.defer[row]);
}

template <int LPR, int VEC, int EPI>
__global__ __launch_bounds__(256) void k_spmm_fixup(SplitArgs a) {
    fixup_body<LPR, VEC, EPI>(a, blockIdx.x);
}

// The rows of two matrices that k_spmm_split_pair multiplied, those of `b` (plain sums) in the workgroups from `blocks_a` on:
// neither list fills the GPU, and one launch takes as long as the slower of two.
template <int LPR, int VEC, int EPI>
__global__ __launch_bounds__(256) void k_spmm_fixup_pair(SplitArgs a, SplitArgs b, uint32_t blocks_a) {
    if (blockIdx.x < blocks_a) fixup_body<LPR, VEC, EPI>(a, blockIdx.x);
    else fixup_body<LPR, VEC, GCN_EPI_NONE>(b, blockIdx.x - blocks_a);
}

// Rows without stored entries produce zeros (any epilogue maps 0 to 0).
__global__ void k_zero_empty_rows(int64_t n, const int64_t* __restrict__ rowptr, int32_t f, float* __restrict__ Z,
                                  int64_t ldz) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / f;
    const int j = (int)(t % f);
    if (i >= n) return;
    if (rowptr[i + 1] == rowptr[i]) Z[i * ldz + j] = 0.f;
}

// The same from the list of empty rows that the schedule keeps (only their elements are touched): `lanes` lanes of 16
// bytes per row, the last one repeating columns where f is no multiple of 4; VEC = 1 below four columns.
template <int VEC>
__global__ __launch_bounds__(256) void k_zero_listed_rows(int64_t count, uint32_t lanes, const int32_t* __restrict__ rows, int32_t f,
                                                          float* __restrict__ Z, int64_t ldz) {
    const uint32_t per = 256 / lanes;                    // rows per workgroup and step (lanes <= 256)
    const uint32_t r = threadIdx.x / lanes, li = threadIdx.x % lanes;
    if (r >= per) return;
    const int step = (int)lanes * VEC;
    const float zero[VEC] = {};
    for (int64_t q = (int64_t)blockIdx.x * per + r; q < count; q += (int64_t)gridDim.x * per) {
        float* z = Z + (int64_t)rows[q] * ldz;
        for (int c = (int)li * VEC; c < f; c += step) store_vec<VEC>(z + (c + VEC <= f ? c : f - VEC), zero);
    }
}

// Reference-shaped kernel: one thread per output element walks its row.  Kept as a selectable
// second implementation (GCN_CFG_SPMM_ALGO = 1) for cross-checks; chosen automatically only for operands that the
// other kernels do not take (see rowwise_only).
template <int EPI>
__global__ void k_spmm_rowwise(int64_t n, const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                               const float* __restrict__ val, const float* __restrict__ row_scale, int32_t f,
                               const float* __restrict__ X, int64_t ldx,
                               float* __restrict__ Z, int64_t ldz, const float* __restrict__ Zprev, int64_t ldzprev) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / f;
    const int j = (int)(t % f);
    if (i >= n) return;
    float acc = 0.f;
    for (int64_t k = rowptr[i]; k < rowptr[i + 1]; ++k)
        acc = fmaf(val ? val[k] : 1.f, X[(int64_t)colidx[k] * ldx + j], acc);
    if (row_scale) acc *= row_scale[i];
    if (EPI == GCN_EPI_RELU) acc = acc > 0.f ? acc : 0.f;
    if (EPI == GCN_EPI_MASK) acc = Zprev[i * ldzprev + j] > 0.f ? acc : 0.f;
    Z[i * ldz + j] = acc;
}

// Dynamic LDS on top of the kernel's own, to lower the number of resident workgroups.  The kernels with 16 lane groups
// per wavefront (rows of up to 64 bytes) keep 64 gathers in flight per wavefront and run slower with eight workgroups
// per compute unit than with five (119 M entries at 16 columns: 0.64 -> 0.62 ms), which the 31 KB of the 16-byte kernel
// leave by themselves; the one-float kernel, with 28 KB of its own, takes four (102 M entries at one column: 612 -> 576
// us) and is padded to 38 KB.  A setting takes the place of both rules.
template <int LPR, int VEC>
static size_t occupancy_pad(int lds_kb, int epilogue) {
    if (LPR != 4) return 0;
    const size_t own = epilogue == GCN_EPI_MASK ? sizeof(WaveLds<LPR, VEC, true>) : sizeof(WaveLds<LPR, VEC, false>);
    const size_t want = (size_t)(lds_kb > 0 ? lds_kb : (VEC == 1 ? 38 : 0)) << 10;
    return want > WAVES_PER_BLOCK * own ? want - WAVES_PER_BLOCK * own : 0;
}

template <int LPR, int VEC>
static int launch_fixup(const SplitArgs& args, int epilogue, hipStream_t s) {
    if (args.n_fix == 0) return GCN_OK;
    const dim3 grid((unsigned)((args.n_fix * LPR + 255) / 256), (unsigned)((args.f + LPR * VEC - 1) / (LPR * VEC)));
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL((k_spmm_fixup<LPR, VEC, GCN_EPI_NONE>), grid, dim3(256), 0, s, args); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL((k_spmm_fixup<LPR, VEC, GCN_EPI_RELU>), grid, dim3(256), 0, s, args); break;
        case EPI_LAYER: hipLaunchKernelGGL((k_spmm_fixup<LPR, VEC, EPI_LAYER>), grid, dim3(256), 0, s, args); break;
        default: hipLaunchKernelGGL((k_spmm_fixup<LPR, VEC, GCN_EPI_MASK>), grid, dim3(256), 0, s, args); break;
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// The fix-up reads and writes rows of Z: where lanes of 16 bytes repeat columns, it takes one column per lane.
template <int LPR, int VEC>
static int fixup_of(const SplitArgs& args, int epilogue, hipStream_t s) {
    if (VEC == 4 && args.f % 4 != 0) return launch_fixup<16, 1>(args, epilogue, s);
    return launch_fixup<LPR, VEC>(args, epilogue, s);
}

// Whether a masked product over 17 columns and more looks its mask up when a row ends instead of keeping bits: chunks that
// begin more rows than there is room for bits read the rest one by one in any case, and the burst for those that fit
// costs more than it saves.  Rows of up to 3.5 entries on average: in rows of 3 at 32 columns 1 M entries take 50 us with
// bits and 41 without, 20 M 686 and 575; in rows of 5 20 M take 347 and 479.  At 16 columns the bits of all rows fit and win.
static bool many_row_starts(const SplitArgs& a) { return 2 * a.nnz <= 7 * a.n_ne; }

template <int LPR>
static int launch_few(const SplitArgs& args, int epilogue, hipStream_t s) {
    const int64_t panels = (args.f + LPR * 4 - 1) / (LPR * 4);
    const dim3 grid((unsigned)((args.nchunks + WAVES_PER_BLOCK - 2) / (WAVES_PER_BLOCK - 1)), (unsigned)panels);
    constexpr size_t lds = WAVES_PER_BLOCK * SUB * 64 * sizeof(float4);
    SplitArgs few = args;
    few.n_fix = args.n_fix_long;                  // they come first in the list
    auto go = [&](auto zero) {
        constexpr bool ZERO = decltype(zero)::value;
        switch (epilogue) {
            case GCN_EPI_NONE: launch_lds<k_spmm_few<LPR, GCN_EPI_NONE, ZERO>>(grid, 64 * WAVES_PER_BLOCK, lds, s, few); break;
            case GCN_EPI_RELU: launch_lds<k_spmm_few<LPR, GCN_EPI_RELU, ZERO>>(grid, 64 * WAVES_PER_BLOCK, lds, s, few); break;
            default: launch_lds<k_spmm_few<LPR, GCN_EPI_MASK, ZERO>>(grid, 64 * WAVES_PER_BLOCK, lds, s, few); break;
        }
    };
    timing_begin(s);
    if (args.empty_share > 0) go(std::true_type());
    else go(std::false_type());
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return fixup_of<LPR, 4>(few, epilogue, s);
}

template <int LPR, int VEC>
static int launch_split(const SplitArgs& args, int epilogue, hipStream_t s) {
    const int tile = LPR * VEC;
    const dim3 grid(chunk_groups(args), (unsigned)((args.f + tile - 1) / tile));
    const dim3 block(64 * WAVES_PER_BLOCK);
    const size_t pad = occupancy_pad<LPR, VEC>(args.lds_kb, epilogue);
    auto go = [&](auto zero) {
        constexpr bool ZERO = decltype(zero)::value;
        switch (epilogue) {
            case GCN_EPI_NONE: hipLaunchKernelGGL((k_spmm_split<LPR, VEC, GCN_EPI_NONE, true, ZERO>), grid, block, pad, s, args); break;
            case GCN_EPI_RELU: hipLaunchKernelGGL((k_spmm_split<LPR, VEC, GCN_EPI_RELU, true, ZERO>), grid, block, pad, s, args); break;
            case EPI_LAYER:                     // (run_matrix; no rows without entries)
                if constexpr (VEC == 4 && !ZERO) hipLaunchKernelGGL((k_spmm_split<LPR, VEC, EPI_LAYER>), grid, block, pad, s, args);
                break;
            default:
                if constexpr (VEC == 4 && LPR == 8) {
                    if (many_row_starts(args)) {
                        hipLaunchKernelGGL((k_spmm_split<LPR, VEC, GCN_EPI_MASK, false, ZERO>), grid, block, pad, s, args);
                        break;
                    }
                }
                hipLaunchKernelGGL((k_spmm_split<LPR, VEC, GCN_EPI_MASK, true, ZERO>), grid, block, pad, s, args);
                break;
        }
    };
    timing_begin(s);
    if (args.empty_share > 0) go(std::true_type());
    else go(std::false_type());
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return fixup_of<LPR, VEC>(args, epilogue, s);
}

template <int VEC>
static int launch_line(const SplitArgs& args, int epilogue, hipStream_t s) {
    const dim3 grid(chunk_groups(args), (unsigned)((args.f + 64 * VEC - 1) / (64 * VEC)));
    const dim3 block(64 * WAVES_PER_BLOCK);
    timing_begin(s);
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL((k_spmm_line<VEC, GCN_EPI_NONE>), grid, block, 0, s, args); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL((k_spmm_line<VEC, GCN_EPI_RELU>), grid, block, 0, s, args); break;
        default: hipLaunchKernelGGL((k_spmm_line<VEC, GCN_EPI_MASK>), grid, block, 0, s, args); break;
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return launch_fixup<16, 1>(args, epilogue, s);
}

static int launch_ragged(const SplitArgs& args, int epilogue, hipStream_t s) {
    const unsigned panels = (unsigned)((args.f + 63) / 64);
    timing_begin(s);
    const int lanes = args.f >= 64 ? 16 : (args.f + 3) / 4;
    const dim3 grid((unsigned)args.nchunks, panels);
    const size_t lds = (size_t)HALF * lanes * sizeof(float4);
    switch (epilogue) {
        case GCN_EPI_NONE: launch_lds<k_spmm_ragged<GCN_EPI_NONE>>(grid, 256, lds, s, args, lanes); break;
        case GCN_EPI_RELU: launch_lds<k_spmm_ragged<GCN_EPI_RELU>>(grid, 256, lds, s, args, lanes); break;
        default: launch_lds<k_spmm_ragged<GCN_EPI_MASK>>(grid, 256, lds, s, args, lanes); break;
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    // the fix-up reads and writes rows of Z: no column may belong to two lanes there
    return launch_fixup<16, 1>(args, epilogue, s);
}

// Whether a matrix goes through k_spmm_short: its rows are all short, and all wavefronts are resident at once (eight per
// compute unit at this kernel's registers).  With more rows the even chunks of k_spmm_split win (rows of 21 entries at 16
// columns: 20 K rows 9.7 against 11.0 us, 50 K rows 17.7 against 14.2).
static int short_lanes(int32_t f) {                // as in choose_split: the pieces of a row follow from them
    return f % 4 == 0 ? (f <= 16 ? 4 : 8) : (f <= 8 ? 2 : (f <= 16 ? 4 : (f <= 32 ? 8 : 16)));
}
static bool short_rows(const Matrix& m, int32_t f) {
    const int lpr = short_lanes(f);
    const int64_t lanes = m.nrows * lpr * ((f + 4 * lpr - 1) / (4 * lpr));
    return f >= 4 && m.short_col && lanes <= SHORT_LANES && lanes <= (int64_t)device_info().cus * 8 * 64;
}

static int launch_short(const SplitArgs& args, const Matrix& m, int epilogue, hipStream_t s, RowsNext* next) {
    const int64_t nrows = m.nrows;
    if (next && next->kind != RowsNext::NONE && epilogue != GCN_EPI_MASK && args.f % 4 == 0 && args.f <= 16) {
        const dim3 grid((unsigned)((nrows + 15) / 16));
        const RowsNext nx = *next;
        auto gradient = [&](auto kinds, auto tiles) {
            hipLaunchKernelGGL((k_spmm_short<4, 32, GCN_EPI_NONE, decltype(kinds)::value, decltype(tiles)::value>),
                               dim3((unsigned)((nrows + 63) / 64)), dim3(256), 0, s, args, nrows, m.short_rows, m.short_pitch, nx);
        };
        constexpr std::integral_constant<int, RowsNext::GRAD> grad{};
        constexpr std::integral_constant<int, RowsNext::GRAD | RowsNext::GEMM> both{};
        constexpr std::integral_constant<int, 1> one{};
        constexpr std::integral_constant<int, 4> four{};
        timing_begin(s);
        if (nx.kind == grad) {
            if (nx.M <= 16) gradient(grad, one);
            else gradient(grad, four);
        } else if (nx.kind == both) {           // (GEMM: M is at most 16)
            gradient(both, one);
        } else if (nx.kind == RowsNext::LOSS)
            hipLaunchKernelGGL((k_spmm_short<4, 32, GCN_EPI_NONE, RowsNext::LOSS>), grid, dim3(64), 0, s, args, nrows, m.short_rows,
                               m.short_pitch, nx);
        else if (epilogue == GCN_EPI_RELU)
            hipLaunchKernelGGL((k_spmm_short<4, 32, GCN_EPI_RELU, RowsNext::GEMM>), grid, dim3(64), 0, s, args, nrows, m.short_rows,
                               m.short_pitch, nx);
        else
            hipLaunchKernelGGL((k_spmm_short<4, 32, GCN_EPI_NONE, RowsNext::GEMM>), grid, dim3(64), 0, s, args, nrows, m.short_rows,
                               m.short_pitch, nx);
        timing_end(s);
        GCN_LAUNCH_CHECK();
        next->done = true;
        return GCN_OK;
    }
    auto go = [&](auto lpr, auto slice) {
        constexpr int LPR = decltype(lpr)::value, SLICE = decltype(slice)::value;
        const dim3 grid((unsigned)((nrows * LPR + 63) / 64), (unsigned)((args.f + 4 * LPR - 1) / (4 * LPR)));
        switch (epilogue) {
            case GCN_EPI_NONE:
                hipLaunchKernelGGL((k_spmm_short<LPR, SLICE, GCN_EPI_NONE>), grid, dim3(64), 0, s, args, nrows, m.short_rows, m.short_pitch, NoNext());
                break;
            case GCN_EPI_RELU:
                hipLaunchKernelGGL((k_spmm_short<LPR, SLICE, GCN_EPI_RELU>), grid, dim3(64), 0, s, args, nrows, m.short_rows, m.short_pitch, NoNext());
                break;
            default:
                hipLaunchKernelGGL((k_spmm_short<LPR, SLICE, GCN_EPI_MASK>), grid, dim3(64), 0, s, args, nrows, m.short_rows, m.short_pitch, NoNext());
                break;
        }
    };
    timing_begin(s);
    // lanes per row as in short_lanes, slices as the nonzero-split kernels cut them at this width
    if (args.f % 4 == 0) {
        if (args.f <= 16) go(std::integral_constant<int, 4>(), std::integral_constant<int, 32>());
        else go(std::integral_constant<int, 8>(), std::integral_constant<int, 64>());
    } else {
        if (args.f <= 8) go(std::integral_constant<int, 2>(), std::integral_constant<int, 64>());
        else if (args.f <= 16) go(std::integral_constant<int, 4>(), std::integral_constant<int, 128>());
        else if (args.f <= 32) go(std::integral_constant<int, 8>(), std::integral_constant<int, 256>());
        else go(std::integral_constant<int, 16>(), std::integral_constant<int, 512>());
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Adds the partial rows of the column-blocked product in ascending block order, then the epilogue.  Bound by reading them, four at a
// time: one by one every partial row waited for its number and then for itself (62 K rows of 100 blocks at 16 columns 121 -> 83 us,
// 4.9 TB/s; 528 K of 15 148 -> 131; 81 K of 8 18 -> 15; 120 K rows of two blocks at 64 columns 16.1 -> 15.4; eight at a time 86, 130, 16 and 17).
template <int VEC, int EPI>
__global__ __launch_bounds__(256) void k_block_reduce(int64_t n, int32_t f, int32_t lanes, const int64_t* __restrict__ rq_ptr,
                                                      const int32_t* __restrict__ rq_idx, const int32_t* __restrict__ row_map,
                                                      const float* __restrict__ row_scale, const float* __restrict__ P,
                                                      float* __restrict__ Z, int64_t ldz, const float* __restrict__ Zprev,
                                                      int64_t ldzprev, int accumulate, LayerEnd end) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / lanes;
    int col0 = (int)(t % lanes) * VEC;
    if (i >= n) return;
    if (col0 + VEC > f) col0 = f - VEC;              // the last lane of a ragged width repeats columns (accumulate: f % VEC == 0)
    const int64_t row = row_map ? row_map[i] : i;    // a row-subset matrix writes only its own rows
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    if (accumulate) load_vec<VEC>(acc, Z + row * ldz + col0);   // what an earlier pass stored raw for this row
    const int64_t first = rq_ptr[i];
    const int32_t* const list = rq_idx + first;
    const int count = (int)(rq_ptr[i + 1] - first);
    constexpr int AT_ONCE = 4;
    for (int k = 0; k < count; k += AT_ONCE) {
        float part[AT_ONCE][VEC];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) load_vec<VEC>(part[e], P + (int64_t)list[k + e < count ? k + e : count - 1] * f + col0);
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) {
            if (k + e < count) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += part[e][v];
            }
        }
    }
    const float scale = row_scale ? row_scale[row] : 1.f;
    if constexpr (EPI == EPI_LAYER)
        layer_store<VEC>(Z + row * ldz + col0, end.H ? end.H + row * ldz + col0 : nullptr, end.bias ? end.bias + col0 : nullptr, end.relu,
                         acc, scale);
    else epilogue_store<VEC, EPI>(Z + row * ldz + col0, EPI == GCN_EPI_MASK ? Zprev + row * ldzprev + col0 : nullptr, acc, scale);
}

template <int VEC>
static int launch_block_reduce(int64_t n, int32_t f, const Blocked& b, const int32_t* row_map, const float* row_scale,
                               int accumulate, const float* P, float* Z,
                               int64_t ldz, int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s,
                               const LayerEnd& end = LayerEnd()) {
    const int lanes = (f + VEC - 1) / VEC;
    const int64_t threads = n * lanes;
    const dim3 grid((unsigned)((threads + 255) / 256));
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL((k_block_reduce<VEC, GCN_EPI_NONE>), grid, dim3(256), 0, s, n, f, lanes, b.rq_ptr, b.rq_idx, row_map, row_scale, P, Z, ldz, Zprev, ldzprev, accumulate, end); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL((k_block_reduce<VEC, GCN_EPI_RELU>), grid, dim3(256), 0, s, n, f, lanes, b.rq_ptr, b.rq_idx, row_map, row_scale, P, Z, ldz, Zprev, ldzprev, accumulate, end); break;
        case EPI_LAYER: hipLaunchKernelGGL((k_block_reduce<VEC, EPI_LAYER>), grid, dim3(256), 0, s, n, f, lanes, b.rq_ptr, b.rq_idx, row_map, row_scale, P, Z, ldz, Zprev, ldzprev, accumulate, end); break;
        default: hipLaunchKernelGGL((k_block_reduce<VEC, GCN_EPI_MASK>), grid, dim3(256), 0, s, n, f, lanes, b.rq_ptr, b.rq_idx, row_map, row_scale, P, Z, ldz, Zprev, ldzprev, accumulate, end); break;
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// ---- column sweep ---------------------------------------------------------------------------------------
// One wavefront owns a task: `rb` consecutive rows whose results live in LDS ((rb + 1) x W floats, W = 16
// or 32) for the whole launch.  Its entries come in ascending column order, so it walks X left to
// right; all wavefronts of a launch start together and have about the same length, so at any moment
// the whole GPU gathers from a narrow band of X, which therefore stays in L2 even when X is far
// larger than every cache.  The stored order puts 2 G entries of different rows into every two steps (see
// Sweep), so the G lane groups of two steps always hold different rows: each multiplies its gathered row by the
// value and adds it to the task's row in LDS with a plain read-modify-write.  Only this wavefront
// touches these accumulators and its LDS operations complete in program order, so the sum order is
// fixed and the result reproducible.
//
// Every launch reads X once per XCD at the least, so few launches (all of the LDS holds accumulators) and wavefronts that stay
// together decide, not the speed of the walk: an L2 turns over in about 5 us, and a task that falls behind the others by more
// than that finds none of their lines.  Hence a workgroup takes a whole compute unit, its wavefronts starting together;
// and a wavefront waits for all it has asked for before it asks for more, which keeps the fast ones from running ahead,
// and adds the trip before while it waits.  Indices are handed round in registers.
// 0.47 G entries over 4.4 M rows of 64 bytes, sweep of one product (and its misses): a wavefront of 256 rows per workgroup, nine per
// compute unit, indices handed round through the LDS: 4.2 ms (176 M); in registers 4.9 (247 M); two trips asked
// for at once 5.5.  Workgroups of 5 x 511 rows, two trips at once: 3.4 to 4.3 (200 to 229 M), depending on where the compiler
// put its waits; this kernel 3.4 (132 M: 138 G entries/s, 39 G misses/s), and the same with four,
// six or seven tasks in the same LDS.  With eight 4.3.  Product: 5.56 -> 4.75 ms; 1.32 G entries, 8.7 M rows 12.1 -> 10.2; 0.12
// G, 1.2 M rows 1.30 -> 0.91, at 32 columns 1.65 -> 1.22.
// What bounds it now is the wait: 127 G L2 requests/s and 38 G misses/s are 0.50 and 0.70 of what a gather loop reaches of either,
// where the hub schedule's pair reaches 0.41 and 0.99 at once.  Nothing is under way when a trip's last gather arrives.
struct SweepArgs {
    const int32_t* colidx;
    const float* val;            // NULL: value-free product
    const float* row_scale;      // NULL, or one factor per output row
    const uint16_t* lrow;
    const int64_t* task_base;
    const int32_t* task_len;
    const int32_t* task_order;
    int64_t n;
    int32_t f, rb;
    int32_t parts;               // how many sums a task's entries are cut into
    int32_t panel, panels;       // of f
    const float* X; int64_t ldx;
    float* Z; int64_t ldz;
    const float* Zprev; int64_t ldzprev;
};

// Entry `q` of the eight that a lane group works through in a trip, of which each of its first four lanes holds two (q a constant
// once the loop around is unrolled).
__device__ __forceinline__ int trip_entry(const int (&x)[2], int q) {
    const int v = x[q & 1];
    switch (q >> 1) {
        case 0: return __builtin_amdgcn_mov_dpp(v, 0x00, 0xf, 0xf, true);
        case 1: return __builtin_amdgcn_mov_dpp(v, 0x55, 0xf, 0xf, true);
        case 2: return __builtin_amdgcn_mov_dpp(v, 0xaa, 0xf, 0xf, true);
        default: return __builtin_amdgcn_mov_dpp(v, 0xff, 0xf, 0xf, true);
    }
}

template <int LPR, int EPI, bool VALUES>
__global__ __launch_bounds__(64 * SWEEP_TASKS) void k_spmm_sweep(SweepArgs a, int64_t first_task, int32_t count) {
    constexpr int G = 64 / LPR;                  // entries per step (16 or 8)
    constexpr int W = LPR * 4;                   // panel width in floats
    constexpr int STEPS = SWEEP_STEPS, TRIP = STEPS * G;
    static_assert(STEPS == 8, "four lanes hold two entries each");
    extern __shared__ float s_acc[];             // per wavefront [rb + 1][W]: the last row takes what padding entries add
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t idx = (int32_t)(blockIdx.x * (blockDim.x >> 6)) + wave;
    if (idx >= count) return;                    // whole wavefront leaves; no block-wide barrier below
    float* const acc = s_acc + wave * ((a.rb + 1) * W);
    const int g = lane / LPR, li = lane % LPR;
    int col0;
    const bool col_ok = lane_columns<LPR, 4>(a.f, a.panel, a.panels, li, &col0);
    const int64_t task = a.task_order[first_task + idx];
    for (int i = lane * 4; i < (a.rb + 1) * W; i += 256) *reinterpret_cast<float4*>(acc + i) = make_float4(0.f, 0.f, 0.f, 0.f);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();

    const int trips = a.task_len[task] / TRIP;
    const int64_t mine = a.task_base[task] + g * STEPS + (lane & 3) * 2;       // this lane's two entries of the first trip
    const float* const xbase = a.X + (col_ok ? col0 : 0);
    const uint32_t xpitch = (uint32_t)a.ldx * 4u;
    const int64_t row0 = task * a.rb;
    struct Index { int c[2], v[2]; uint32_t r; };
    struct Rows { float x[STEPS][4]; int off[STEPS], v[2]; };
    auto load = [&](int t, Index& n) {           // (past the end: the last trip again, not used)
        const int64_t k = mine + (int64_t)(t < trips ? t : trips - 1) * TRIP;
        const intx2 c = __builtin_nontemporal_load(reinterpret_cast<const intx2*>(a.colidx + k));
        n.c[0] = c.x; n.c[1] = c.y;
        n.r = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(a.lrow + k));
        if constexpr (VALUES) {
            const intx2 v = __builtin_nontemporal_load(reinterpret_cast<const intx2*>(a.val + k));
            n.v[0] = v.x; n.v[1] = v.y;
        }
    };
    // Waits for everything on its way, then sends out the gathers of the trip in `n` and loads the indices of trip `next`.
    auto gather = [&](Index& n, int next, Rows& m) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        const float* at[STEPS];
        const int off[2] = {(int)(n.r & 0xffffu) * W, (int)(n.r >> 16) * W};
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            at[q] = at_row(xbase, (uint32_t)trip_entry(n.c, q), xpitch);
            m.off[q] = trip_entry(off, q) + li * 4;
        }
        if constexpr (VALUES) { m.v[0] = n.v[0]; m.v[1] = n.v[1]; }
        __builtin_amdgcn_sched_barrier(0);
        load(next, n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < STEPS; ++q) load_vec<4>(m.x[q], at[q]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto add = [&](const Rows& m) {
        constexpr int P = 2;                     // the entries of two steps hold different rows
#pragma unroll
        for (int q0 = 0; q0 < STEPS; q0 += P) {
            float4 cur[P];
#pragma unroll
            for (int e = 0; e < P; ++e) cur[e] = *reinterpret_cast<const float4*>(acc + m.off[q0 + e]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < P; ++e) {
                const int q = q0 + e;
                const float v = VALUES ? __int_as_float(trip_entry(m.v, q)) : 1.f;
                cur[e].x = fmaf(v, m.x[q][0], cur[e].x);
                cur[e].y = fmaf(v, m.x[q][1], cur[e].y);
                cur[e].z = fmaf(v, m.x[q][2], cur[e].z);
                cur[e].w = fmaf(v, m.x[q][3], cur[e].w);
                *reinterpret_cast<float4*>(acc + m.off[q]) = cur[e];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The task's rows so far, G per pass and 16 bytes per lane: what Z holds of them (nothing at first) plus the sums in LDS.
    bool part_in_z = false;
    auto rows_out = [&](auto last) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 4
        for (int i = g; i < a.rb; i += G) {
            const int64_t row = row0 + i;
            if (row >= a.n || !col_ok) continue;
            float4* const at = reinterpret_cast<float4*>(acc + i * W + li * 4);
            float v[4] = {at->x, at->y, at->z, at->w};
            float* const z = a.Z + row * a.ldz + col0;
            if (part_in_z) {
                float before[4];
                load_vec<4>(before, z);
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] += before[u];
            }
            if constexpr (last) {
                epilogue_store<4, EPI>(z, EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + col0 : nullptr, v,
                                       a.row_scale ? a.row_scale[row] : 1.f);
            } else {
                store_vec<4>(z, v);
                *at = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        part_in_z = true;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    if (trips > 0) {
        const int part = (trips / a.parts + 2) & ~1;            // trips between two of them, even
        int next = part;
        Index n = {};
        Rows xa, xb;
        load(0, n);
        gather(n, 1, xa);
#pragma unroll 1
        for (int t = 0;; t += 2) {
            gather(n, t + 2, xb);                // trip t + 1
            add(xa);
            if (t + 1 >= trips) break;
            gather(n, t + 3, xa);                // trip t + 2
            add(xb);
            if (t + 2 >= trips) break;
            if (t + 2 == next && a.parts > 1) {
                rows_out(std::false_type());
                next += part;
            }
        }
    }
    rows_out(std::true_type());
}

// Rows of a task: what is left of a compute unit's LDS for each of SWEEP_TASKS, less the row of the padding entries.
static int32_t sweep_rows(int panel) { return (160 << 10) / (SWEEP_TASKS * panel * 4) - 1; }
// Tasks that a compute unit works on at once: GCN_CFG_SWEEP_WAVES, as many as there is room for.
static int64_t sweep_tasks(const Config& cfg) { return cfg.sweep_waves < SWEEP_TASKS ? cfg.sweep_waves : SWEEP_TASKS; }

template <int LPR, bool VALUES>
static int launch_sweep(const SweepArgs& args, int64_t ntasks, int64_t per_cu, int epilogue, hipStream_t s) {
    constexpr int W = LPR * 4;
    const unsigned ytiles = (unsigned)((args.f + W - 1) / W);
    // tasks that are resident at once; the launches get equal shares so that the last one is not a stub
    const int64_t cus = device_info().cus, cap = cus * per_cu;
    const int64_t nlaunch = (ntasks + cap - 1) / cap;
    const int64_t gen = (ntasks + nlaunch - 1) / nlaunch;
    const int64_t waves = (gen + cus - 1) / cus;
    const size_t lds = (size_t)waves * (args.rb + 1) * W * sizeof(float);
    timing_begin(s);
    for (unsigned y = 0; y < ytiles; ++y) {
        for (int64_t first = 0; first < ntasks; first += gen) {
            const int32_t count = (int32_t)(ntasks - first < gen ? ntasks - first : gen);
            const dim3 grid((unsigned)((count + waves - 1) / waves));
            const int threads = (int)waves * 64;
            SweepArgs a = args;
            a.panel = (int32_t)y;
            a.panels = (int32_t)ytiles;
            switch (epilogue) {
                case GCN_EPI_NONE: launch_lds<k_spmm_sweep<LPR, GCN_EPI_NONE, VALUES>>(grid, threads, lds, s, a, first, count); break;
                case GCN_EPI_RELU: launch_lds<k_spmm_sweep<LPR, GCN_EPI_RELU, VALUES>>(grid, threads, lds, s, a, first, count); break;
                default: launch_lds<k_spmm_sweep<LPR, GCN_EPI_MASK, VALUES>>(grid, threads, lds, s, a, first, count); break;
            }
        }
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// The kernel and lane layout of one nonzero-split product.
struct SplitChoice {
    enum Kernel { SPLIT, FEW, RAGGED, LINE } kernel = SPLIT;
    int lpr = 0, vec = 0;                         // lanes per row of X (RAGGED: from the width), floats per lane
};

static SplitChoice choose_split(int32_t f, int64_t nchunks, bool any_order, bool wide) {
    const int64_t cus = device_info().cus;
    if (f < 4) return {SplitChoice::SPLIT, 4, 1};
    if (f % 4 != 0 && !any_order) {
        if (f <= 8) return {SplitChoice::SPLIT, 8, 1};
        if (f <= 16) return {SplitChoice::SPLIT, 16, 1};
        if (f <= 32) return {SplitChoice::SPLIT, 32, 1};
        // k_spmm_ragged puts four wavefronts to a chunk: worth it while that is what fills the GPU (0.3 M entries at 41 columns,
        // 620 chunks: 22 us, k_spmm_line 27; 1 M, 1900 chunks: 51 and 49; 0.4 M at 101, 1660 chunks and panels: 52 and 34).
        const int panels = (f + 63) / 64;
        if (nchunks * panels <= cus * 4) return {SplitChoice::RAGGED, 0, 4};
        // two columns per lane where that halves the number of panels: every panel walks all entries
        return {SplitChoice::LINE, 64, (f + 127) / 128 * 2 == panels ? 2 : 1};
    }
    // Wider operands are processed in panels of 32 columns (one 128-byte line per gathered row): the panel of X that the
    // gathers touch is 4x smaller than at f = 128, so far more of it stays in L2, at the price of re-reading the
    // index/value stream once per panel.  Over column blocks (`wide`) 64 unless a plan says otherwise (see SpmmCost::narrow_panels);
    // the products that keep the schedule of their sizes alone have no plan, and with the panels they keep their sums' order.
    // Rows that are not whole 16-byte pieces (only without an order to keep) straddle lines wherever they are cut: one
    // panel up to 64 columns (41 columns, 1 M rows: 1.20 ms in two panels, 0.89 in one).
    int lpr = 8;
    if (f <= 16) lpr = 4;
    else if (f > 32 && ((f >= 64 && wide) || (f % 4 != 0 && f <= 64))) lpr = 16;
    // k_spmm_few as long as its workgroups of three chunks run side by side (their LDS allows one per compute unit)
    const int64_t panels = (f + 4 * lpr - 1) / (4 * lpr);
    return {nchunks * panels <= cus * (WAVES_PER_BLOCK - 1) ? SplitChoice::FEW : SplitChoice::SPLIT, lpr, 4};
}

static std::string kernel_name(const SplitChoice& c) {
    switch (c.kernel) {
        case SplitChoice::FEW: return "k_spmm_few<" + std::to_string(c.lpr) + ">";
        case SplitChoice::RAGGED: return "k_spmm_ragged";
        case SplitChoice::LINE: return "k_spmm_line<" + std::to_string(c.vec) + ">";
        default: return "k_spmm_split<" + std::to_string(c.lpr) + "," + std::to_string(c.vec) + ">";
    }
}

static int run_split(const SplitArgs& args, int epilogue, hipStream_t s, const SplitChoice& c) {
    switch (c.kernel) {
        case SplitChoice::RAGGED: return launch_ragged(args, epilogue, s);
        case SplitChoice::LINE: return c.vec == 2 ? launch_line<2>(args, epilogue, s) : launch_line<1>(args, epilogue, s);
        case SplitChoice::FEW:
            if (c.lpr == 4) return launch_few<4>(args, epilogue, s);
            if (c.lpr == 8) return launch_few<8>(args, epilogue, s);
            return launch_few<16>(args, epilogue, s);
        default: break;
    }
    if (c.vec == 4) {
        if (c.lpr == 4) return launch_split<4, 4>(args, epilogue, s);
        if (c.lpr == 8) return launch_split<8, 4>(args, epilogue, s);
        return launch_split<16, 4>(args, epilogue, s);
    }
    if (c.lpr == 4) return launch_split<4, 1>(args, epilogue, s);
    if (c.lpr == 8) return launch_split<8, 1>(args, epilogue, s);
    if (c.lpr == 16) return launch_split<16, 1>(args, epilogue, s);
    return launch_split<32, 1>(args, epilogue, s);
}

// How many column blocks to cut X into so that one block of the gathered panel stays in one L2
// (4 MB per XCD on this GPU; the size is read from the device).  Blocking costs one partial row per
// non-empty (block,row) pair, so it only pays when rows are long compared with the number of blocks: at
// least `per_block` entries per partial row.  When half-L2 blocks would make the partial rows shorter than
// that, blocks of up to twice the L2 are still worth it (measured on the long rows of config 5: 5.6 MB
// blocks beat 2 MB ones); beyond that 1 (no blocking).
static int64_t choose_blocks(const Config& cfg, int64_t nrows, int64_t ncols, int64_t nnz, int32_t f, int64_t per_block) {
    const int forced = cfg.spmm_blocks;
    if (forced >= 1) return forced;
    const int64_t l2 = device_info().l2_bytes;
    const int64_t panel = f < 32 ? f : 32;
    const int64_t xbytes = ncols * panel * 4;
    if (xbytes <= l2 / 8 * 7) return 1;                    // already L2-resident
    const int64_t block = l2 / 2;
    const int64_t want = (xbytes + block - 1) / block;
    const int64_t cap = (nnz / (nrows > 0 ? nrows : 1)) / per_block;
    if (want <= cap) return want;
    return (cap >= 2 && 4 * cap >= want) ? cap : 1;
}

// The schedule of a product whose order of additions is free, by what the schedules are estimated to cost (spmm_cost.h); worked
// out once per matrix and width.  `usual` is the number of blocks that the sizes alone give.  Small matrices and operands
// that an L2 holds do not ask.
static bool worth_a_plan(const Matrix& m, int32_t f, int64_t nnz) {
    const int64_t panel = f < 32 ? f : 32;
    return f >= 4 && nnz >= PLANNED_NNZ && m.lengths.total() == nnz && m.ncols * panel * 4 > device_info().l2_bytes / 8 * 7;
}

static SpmmPlan& plan_of(gcn_csr* a, Matrix& m, int32_t f, Terms terms, int64_t usual) {
    for (SpmmPlan& p : m.plans)
        if (p.f == f && p.terms == terms) return p;
    SpmmPlan p;
    p.f = f;
    p.terms = terms;
    p.usual = (int32_t)usual;
    const int64_t nnz = m.lengths.total();
    const SpmmCost c{f, device_info().cus, 8.0, (double)device_info().l2_bytes};
    // the columns of a matrix are the rows of its transpose, where that is stored; otherwise taken to be alike
    const Matrix& t = a->symmetric || &m == &a->At ? a->A : a->At;
    const bool known = t.lengths.total() == nnz;
    const Lengths cols = known ? t.lengths : Lengths::equal(m.ncols, nnz), lines = c.lines(cols);
    if (!even_rows(m.lengths, m.nrows, m.order) || (known && !even_rows(cols, m.ncols, t.order)) || !drawn_columns(cols, m.order)) {
        p.blocks = p.usual;
        m.plans.push_back(p);
        return m.plans.back();
    }
    double split = 0;
    p.narrow = c.narrow_panels(lines, (int)usual);
    // (rows beyond 64 columns that are not whole 16-byte pieces: by the sizes, in panels of 64, which are not estimated)
    const double must = f > 64 && f % 4 != 0 && usual >= 2 ? 0.0 : c.must_save(m.lengths, (int)usual, p.narrow);
    p.blocks = c.best_blocks(m.lengths, lines, m.ncols, (int)usual, must, &split);
    p.narrow = p.narrow || p.blocks > usual;
    constexpr int HEAVY = 8, MOST_PARTS = 8;                    // rows of 2^8 entries and more are long
    int heavy_blocks = 1;
    const int32_t W = f <= 16 ? 16 : 32;
    double sweep = c.sweep(m.lengths, lines, m.nrows, m.ncols, HEAVY, sweep_rows(W), SWEEP_TASKS, 1, &heavy_blocks);
    // As many sums per row as keep them as close to the exact ones as the nonzero split's (see as_exact; 30 M pairs, 1 M vertices, 16
    // columns: 10.0e-8 of the norm there, 14.1, 10.5, 9.1 and 8.5e-8 with one to four; another costs 6 % of the product).
    int parts = 1;
    while (parts <= MOST_PARTS && !c.as_exact(m.lengths, p.usual, heavy_blocks, parts, HEAVY, terms)) ++parts;
    if (parts > 1) sweep = parts > MOST_PARTS ? 1e30 : c.sweep(m.lengths, lines, m.nrows, m.ncols, HEAVY, sweep_rows(W), SWEEP_TASKS, parts, &heavy_blocks);
    // Ragged rows in two panels straddle lines twice (41 columns: no gain).
    p.sweep = c.sweep_pays(m.lengths, sweep, split) && (f % 4 == 0 || f < 32);
    if (p.sweep) {
        p.blocks = heavy_blocks;
        p.narrow = true;
        p.parts = parts;
        p.heavy = (1 << HEAVY) - 1;
        p.padding = c.padding(m.lengths.below(HEAVY), m.nrows, sweep_rows(W));
    }
    m.plans.push_back(p);
    return m.plans.back();
}

// The rows without entries go with the chunks of the product, in equal shares, where there is a list of them and share_of_empty_rows says
// so.  Not k_spmm_ragged, whose matrices are small, nor k_spmm_line<2>, whose registers they cost a wavefront.
static bool share_empty_rows(SplitArgs* args, const Matrix& m, const SplitChoice& c) {
    if (!m.empty_rows || c.kernel == SplitChoice::RAGGED || (c.kernel == SplitChoice::LINE && c.vec == 2)) return false;
    const int64_t n_empty = m.nrows - m.n_ne;
    args->empty_share = share_of_empty_rows(m.nrows, n_empty, m.nchunks, CHUNK, c.lpr, c.vec, args->f, args->ldz, (uintptr_t)args->Z);
    if (args->empty_share == 0) return false;
    args->empty_rows = m.empty_rows;
    args->n_empty = n_empty;
    return true;
}

static int zero_empty_rows(const Matrix& m, int32_t f, float* Z, int64_t ldz, hipStream_t s) {
    const int64_t n_empty = m.nrows - m.n_ne;
    if (m.empty_rows && n_empty > 0) {
        const int vec = f >= 4 ? 4 : 1;
        const int lanes = (f + vec - 1) / vec < 256 ? (f + vec - 1) / vec : 256;
        const int64_t per = 256 / lanes, want = (n_empty + per - 1) / per;
        const dim3 grid((unsigned)(want < 16384 ? want : 16384));
        if (vec == 4) hipLaunchKernelGGL(k_zero_listed_rows<4>, grid, dim3(256), 0, s, n_empty, (uint32_t)lanes, m.empty_rows, f, Z, ldz);
        else hipLaunchKernelGGL(k_zero_listed_rows<1>, grid, dim3(256), 0, s, n_empty, (uint32_t)lanes, m.empty_rows, f, Z, ldz);
    } else {
        const int64_t work = m.nrows * f;
        hipLaunchKernelGGL(k_zero_empty_rows, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, s, m.nrows, m.rowptr, f, Z, ldz);
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// The nonzero-split product of one stored matrix -- the whole matrix, or the heavy rows of a sweep
// copy (then row_map gives the row each of its rows stands for) -- with or without column blocks.
static int run_matrix(gcn_csr* a, Matrix& mm, const int32_t* row_map, int64_t nnz, int64_t nblocks, int32_t f,
                      const float* X, int64_t ldx, float* Z, int64_t ldz, int epilogue, const float* Zprev,
                      int64_t ldzprev, const SpmmOpt& o, hipStream_t s, float* carry_given = nullptr) {
    if (mm.nchunks >= (1ll << 31))
        return fail(GCN_ERR_RANGE, "gcn_spmm: too many chunks for one launch");
    // carry_given: a buffer of at least nchunks * f floats that the caller of this function provides
    // (only without column blocks); otherwise the handle's own buffer, grown on demand
    if (!carry_given) GCN_TRY(grow_retire(a, &a->carry, &a->carry_bytes, (size_t)mm.nchunks * (size_t)f * sizeof(float)));
    SplitArgs args;
    args.lds_kb = cfg_of(a).split_lds_kb;
    args.nnz = nnz; args.nsub = mm.nsub; args.nchunks = mm.nchunks; args.f = f;
    args.X = X; args.ldx = ldx; args.carry = carry_given ? carry_given : a->carry;
    args.defer = nullptr;
    if (nblocks >= 2) {
        int64_t cpb = (mm.ncols + nblocks - 1) / nblocks;
        cpb = (cpb + 1023) & ~1023ll;
        GCN_TRY(want_blocked(mm, nnz, cpb, s));
        const Blocked& b = mm.blk;
        GCN_TRY(grow_retire(a, &a->partial, &a->partial_bytes, (size_t)b.nrows * (size_t)f * sizeof(float)));
        const SplitChoice choice = choose_split(f, mm.nchunks, o.any_order, !o.narrow);
        if (o.describe) {
            char t[200];
            snprintf(t, sizeof t, "blocked(blocks=%d,cols_per_block=%lld,partial_rows=%lld,chunks=%lld,kernel=%s)", (int)b.nblocks,
                     (long long)b.cols_per_block, (long long)b.nrows, (long long)mm.nchunks, kernel_name(choice).c_str());
            *o.describe += t;
        }
        if (o.dry) return GCN_OK;
        args.colidx = b.colidx; args.val = o.pattern ? nullptr : b.val; args.flags = b.flags; args.sub_row = b.sub_row;
        args.n_ne = b.nrows;
        args.ne_rows = nullptr; args.rp = b.rp; args.row_scale = nullptr;     // the scale belongs to the reduced row
        args.fix_list = b.fix_list; args.n_fix = b.n_fix; args.n_fix_long = b.n_fix_long;
        args.Z = a->partial; args.ldz = f; args.Zprev = nullptr; args.ldzprev = 0;
        args.per_xcd = (uint32_t)((mm.nchunks + XCDS * WAVES_PER_BLOCK - 1) / (XCDS * WAVES_PER_BLOCK));
        GCN_TRY(run_split(args, GCN_EPI_NONE, s, choice));
        LayerEnd end;
        if (o.end && !row_map) {
            epilogue = EPI_LAYER;
            end = *o.end;
            o.end->done = true;
        }
        if (f >= 4) return launch_block_reduce<4>(mm.nrows, f, b, row_map, o.row_scale, o.accumulate ? 1 : 0, a->partial, Z, ldz, epilogue, Zprev, ldzprev, s, end);
        return launch_block_reduce<1>(mm.nrows, f, b, row_map, o.row_scale, o.accumulate ? 1 : 0, a->partial, Z, ldz, epilogue, Zprev, ldzprev, s, end);
    }
    const bool short_kernel = !row_map && short_rows(mm, f);
    const SplitChoice choice = short_kernel ? SplitChoice() : choose_split(f, mm.nchunks, o.any_order, false);
    if (o.describe) {
        char t[120];
        snprintf(t, sizeof t, "split(chunks=%lld,kernel=%s)", (long long)mm.nchunks,
                 short_kernel ? ("k_spmm_short<" + std::to_string(short_lanes(f)) + ">").c_str() : kernel_name(choice).c_str());
        *o.describe += t;
    }
    if (o.dry) return GCN_OK;
    args.colidx = mm.colidx; args.val = o.pattern ? nullptr : mm.val; args.flags = mm.flags; args.sub_row = mm.sub_row;
    args.row_scale = o.row_scale;
    args.defer = o.defer;
    args.ne_rows = row_map ? row_map : mm.ne_rows;
    args.n_ne = mm.n_ne;
    args.rp = mm.ne_rowptr ? mm.ne_rowptr : mm.rowptr;
    args.fix_list = mm.fix_list; args.n_fix = mm.n_fix; args.n_fix_long = mm.n_fix_long;
    args.Z = Z; args.ldz = ldz; args.Zprev = Zprev; args.ldzprev = ldzprev;
    if (short_kernel) {
        args.colidx = mm.short_col;
        if (args.val) args.val = mm.short_val;
        return launch_short(args, mm, epilogue, s, o.next);
    }
    if (o.end && !row_map && choice.kernel == SplitChoice::SPLIT && choice.vec == 4 && mm.n_ne == mm.nrows) {
        // (rows without entries are their bias alone; the other kernels run where a pass more is a launch more, or on ragged widths)
        epilogue = EPI_LAYER;
        args.bias = o.end->bias; args.H = o.end->H; args.relu = o.end->relu;
        o.end->done = true;
    }
    if (!row_map && mm.n_ne < mm.nrows && !share_empty_rows(&args, mm, choice))
        GCN_TRY(zero_empty_rows(mm, f, Z, ldz, s));
    return run_split(args, epilogue, s, choice);
}

// ---- hub schedule -----------------------------------------------------------------------------------------
// xhot[r,:] = X[hot_col[r],:], 16 bytes per thread.
__global__ __launch_bounds__(256) void k_pack_rows(int64_t H, int32_t lanes, const float* __restrict__ X, int64_t ldx,
                                                   const int32_t* __restrict__ hot_col, float* __restrict__ xhot) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = t / lanes;
    const int j = (int)(t % lanes) * 4;
    if (r >= H) return;
    *reinterpret_cast<float4*>(xhot + r * (int64_t)lanes * 4 + j) =
        *reinterpret_cast<const float4*>(X + (int64_t)hot_col[r] * ldx + j);
}

// Packed-buffer size and block width of the hub copy for operands of width f: blocks of about 2 MB
// of the gathered panel, as many hot columns as fit `budget` bytes (a multiple of the block width).
static void hub_shape(const Config& cfg, int64_t ncols, int32_t f, int64_t* H, int64_t* cpb) {
    const int64_t panel = f < 32 ? f : 32;
    *cpb = cfg.hub_block_cols > 0 ? cfg.hub_block_cols : (device_info().l2_bytes / 2) / (panel * 4);
    const int64_t budget = (int64_t)cfg.hub_mb << 20;
    int64_t h = budget / ((int64_t)f * 4);
    if (h > ncols) h = ncols;
    *H = h / *cpb * *cpb;
}

template <int LPR>
static int launch_pair(const SplitArgs& ra_args, const SplitArgs& rb_args, int epilogue, hipStream_t s) {
    const int tile = LPR * 4;
    const unsigned ytiles = (unsigned)((ra_args.f + tile - 1) / tile);
    const int64_t ga = (ra_args.nchunks + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    const int64_t gb = (rb_args.nchunks + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    // shares of the two matrices among eight consecutive workgroups, in proportion to their chunk groups
    int ra = (int)((8 * ga + (ga + gb) / 2) / (ga + gb));
    ra = ra < 1 ? 1 : (ra > 7 ? 7 : ra);
    const int rb = 8 - ra;
    const int64_t periods = std::max((ga + ra - 1) / ra, (gb + rb - 1) / rb);
    if (periods * 8 >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_spmm: too many chunks for one launch");
    const dim3 grid((unsigned)(periods * 8), ytiles);
    timing_begin(s);
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL((k_spmm_split_pair<LPR, 4, GCN_EPI_NONE>), grid, dim3(64 * WAVES_PER_BLOCK), 0, s, ra_args, rb_args, ra, rb); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL((k_spmm_split_pair<LPR, 4, GCN_EPI_RELU>), grid, dim3(64 * WAVES_PER_BLOCK), 0, s, ra_args, rb_args, ra, rb); break;
        default: hipLaunchKernelGGL((k_spmm_split_pair<LPR, 4, GCN_EPI_MASK>), grid, dim3(64 * WAVES_PER_BLOCK), 0, s, ra_args, rb_args, ra, rb); break;
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    const unsigned fa = (unsigned)((ra_args.n_fix * LPR + 255) / 256), fb = (unsigned)((rb_args.n_fix * LPR + 255) / 256);
    if (fa + fb == 0) return GCN_OK;
    const dim3 fix(fa + fb, ytiles);
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL((k_spmm_fixup_pair<LPR, 4, GCN_EPI_NONE>), fix, dim3(256), 0, s, ra_args, rb_args, fa); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL((k_spmm_fixup_pair<LPR, 4, GCN_EPI_RELU>), fix, dim3(256), 0, s, ra_args, rb_args, fa); break;
        default: hipLaunchKernelGGL((k_spmm_fixup_pair<LPR, 4, GCN_EPI_MASK>), fix, dim3(256), 0, s, ra_args, rb_args, fa); break;
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// Z = A_rest X (long rows stored raw) and the partial rows of A_hot X_hot in one paired launch, then
// the long rows get their partial rows added, are scaled and finished.  Needs 16-byte aligned operands.
static int run_hub(gcn_csr* a, Matrix& m, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz, int epilogue,
                   const float* Zprev, int64_t ldzprev, const SpmmOpt& o, hipStream_t s) {
    Hub& h = m.hub;
    GCN_TRY(grow_retire(a, &h.xhot, &h.xhot_bytes, (size_t)h.H * (size_t)f * sizeof(float)));
    Matrix& rest = *h.rest;
    Matrix& hot = *h.hot;
    const Blocked& b = hot.blk;
    if ((rest.nchunks + hot.nchunks) / WAVES_PER_BLOCK + 16 >= (1ll << 31))
        return fail(GCN_ERR_RANGE, "gcn_spmm: too many chunks for one launch");
    GCN_TRY(grow_retire(a, &a->carry, &a->carry_bytes, (size_t)rest.nchunks * (size_t)f * sizeof(float)));
    GCN_TRY(grow_retire(a, &a->carry2, &a->carry2_bytes, (size_t)hot.nchunks * (size_t)f * sizeof(float)));
    GCN_TRY(grow_retire(a, &a->partial, &a->partial_bytes, (size_t)b.nrows * (size_t)f * sizeof(float)));
    if (o.describe) {
        char t[240];
        snprintf(t, sizeof t, "hub(hot_cols=%lld,cols_per_block=%lld,long_row>=%d,nnz_hot=%lld,nnz_rest=%lld,partial_rows=%lld,kernel=k_spmm_split_pair<%d,4>)",
                 (long long)h.H, (long long)h.cpb, (int)h.dmin, (long long)h.nnz_hot, (long long)h.nnz_rest, (long long)b.nrows, f > 16 ? 8 : 4);
        *o.describe += t;
    }
    if (o.dry) return GCN_OK;
    const int lanes = f / 4;
    hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)((h.H * lanes + 255) / 256)), dim3(256), 0, s, h.H, lanes, X, ldx,
                       h.hot_col, h.xhot);
    GCN_LAUNCH_CHECK();
    SplitArgs ar;                                  // A_rest over X, into Z
    ar.colidx = rest.colidx; ar.val = o.pattern ? nullptr : rest.val; ar.flags = rest.flags; ar.sub_row = rest.sub_row;
    ar.row_scale = o.row_scale; ar.defer = h.defer;
    ar.ne_rows = rest.ne_rows; ar.rp = rest.ne_rowptr ? rest.ne_rowptr : rest.rowptr;
    ar.fix_list = rest.fix_list; ar.n_fix = rest.n_fix; ar.n_fix_long = rest.n_fix_long;
    ar.nnz = h.nnz_rest; ar.nsub = rest.nsub; ar.nchunks = rest.nchunks; ar.f = f;
    ar.X = X; ar.ldx = ldx; ar.Z = Z; ar.ldz = ldz; ar.Zprev = Zprev; ar.ldzprev = ldzprev; ar.carry = a->carry;
    SplitArgs ah;                                  // A_hot over the packed rows, into the partial rows
    ah.colidx = b.colidx; ah.val = o.pattern ? nullptr : b.val; ah.flags = b.flags; ah.sub_row = b.sub_row;
    ah.row_scale = nullptr; ah.defer = nullptr; ah.ne_rows = nullptr; ah.rp = b.rp;
    ah.fix_list = b.fix_list; ah.n_fix = b.n_fix; ah.n_fix_long = b.n_fix_long;
    ah.nnz = h.nnz_hot; ah.nsub = hot.nsub; ah.nchunks = hot.nchunks; ah.f = f;
    ah.X = h.xhot; ah.ldx = f; ah.Z = a->partial; ah.ldz = f; ah.Zprev = nullptr; ah.ldzprev = 0; ah.carry = a->carry2;
    if (rest.n_ne < rest.nrows && !share_empty_rows(&ar, rest, SplitChoice{SplitChoice::SPLIT, f > 16 ? 8 : 4, 4}))
        GCN_TRY(zero_empty_rows(rest, f, Z, ldz, s));
    if (f > 16) GCN_TRY(launch_pair<8>(ar, ah, epilogue, s));
    else GCN_TRY(launch_pair<4>(ar, ah, epilogue, s));
    return launch_block_reduce<4>(hot.nrows, f, b, h.heavy_rows, o.row_scale, 1, a->partial, Z, ldz, epilogue, Zprev,
                                  ldzprev, s);
}

// ---- stored orders kept per key ------------------------------------------------------------------------
int want_blocked(Matrix& m, int64_t nnz, int64_t cpb, hipStream_t s) {
    if (m.blk.cols_per_block == cpb) return GCN_OK;
    if (m.blk.cols_per_block != 0) {
        m.blk_parked.push_back(m.blk);
        m.blk = Blocked();
    }
    for (size_t i = 0; i < m.blk_parked.size(); ++i)
        if (m.blk_parked[i].cols_per_block == cpb) {
            m.blk = m.blk_parked[i];
            m.blk_parked.erase(m.blk_parked.begin() + (long)i);
            return GCN_OK;
        }
    BuildScope scope(s);
    const int rc = build_blocked(m, nnz, cpb, s);
    if (rc != GCN_OK) {
        (void)hipStreamSynchronize(s);
        free_blocked(m.blk);
    }
    return rc;
}

int want_sweep(Matrix& m, int64_t nnz, int32_t groups, int32_t rb, int32_t th, double most, hipStream_t s) {
    auto is = [&](const Sweep& w) {
        return w.groups == groups && w.rb == rb && w.heavy_threshold == th && (w.built || w.sparser(most));
    };
    if (is(m.swp)) return GCN_OK;
    if (m.swp.groups != 0) {
        m.swp_parked.push_back(m.swp);
        m.swp = Sweep();
    }
    for (size_t i = 0; i < m.swp_parked.size(); ++i)
        if (is(m.swp_parked[i])) {
            m.swp = m.swp_parked[i];
            m.swp_parked.erase(m.swp_parked.begin() + (long)i);
            return GCN_OK;
        }
    BuildScope scope(s);
    const int rc = build_sweep(m, nnz, groups, rb, th, most, s);
    if (rc != GCN_OK) {
        (void)hipStreamSynchronize(s);
        free_sweep(m.swp);
    }
    return rc;
}

// The hub copy for the current settings: the one in use, a parked one, or a new attempt (state 1 built,
// -1 rejected for these settings).  A change of operand width reuses the copy.
static int want_hub(Matrix& m, const Config& cfg, int64_t nnz, int64_t H, int64_t cpb, bool forced, hipStream_t s) {
    auto is = [&](const Hub& h) {
        return h.state != 0 && h.dmin == cfg.hub_dmin && h.cfg_mb == cfg.hub_mb && h.cfg_block_cols == cfg.hub_block_cols;
    };
    if (is(m.hub)) return GCN_OK;
    if (m.hub.state != 0) {
        m.hub_parked.push_back(m.hub);
        m.hub = Hub();
    }
    for (size_t i = 0; i < m.hub_parked.size(); ++i)
        if (is(m.hub_parked[i])) {
            m.hub = m.hub_parked[i];
            m.hub_parked.erase(m.hub_parked.begin() + (long)i);
            return GCN_OK;
        }
    BuildScope scope(s);
    const int rc = build_hub(m, nnz, H, cpb, cfg.hub_dmin, s);
    if (rc != GCN_OK) {
        // the copy is an optimisation: without it (for instance out of memory) the plain kernel runs
        if (forced) return rc;
        (void)hipStreamSynchronize(s);
        free_hub(m.hub);
        m.hub.state = -1;
    }
    m.hub.dmin = cfg.hub_dmin;
    m.hub.cfg_mb = cfg.hub_mb;
    m.hub.cfg_block_cols = cfg.hub_block_cols;
    return GCN_OK;
}

// Operands that only the row-wise kernel takes:
//   * rows 4 GB and more apart: it computes its addresses in 64 bits, the others multiply a row's number by its pitch in
//     bytes, both 32 bits wide (see at_row);
//   * a mask that is the output itself: its threads read their element of the mask and then store that element, while the
//     others store a row that crosses chunks, or that the hub schedule defers, before they finish it, and read
//     the mask when they finish it (and two lanes of different wavefronts may compute the last columns of a ragged row).
static bool rowwise_only(const Matrix& m, int64_t ldx, const float* Z, int64_t ldz, int epilogue, const float* Zprev,
                         int64_t ldzprev) {
    constexpr int64_t FAR = 1ll << 30;                          // floats
    if (ldx >= FAR || ldz >= FAR) return true;
    if (epilogue != GCN_EPI_MASK) return false;
    return ldzprev >= FAR || (Zprev == Z && (ldzprev == ldz || m.nrows == 1));
}

static int launch_rowwise(const Matrix& m, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz, int epilogue,
                          const float* Zprev, int64_t ldzprev, const SpmmOpt& o, hipStream_t s) {
    const int64_t n = m.nrows, work = n * f;
    const dim3 grid((unsigned)((work + 255) / 256));
    if (work / 256 >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_spmm: n*f too large for the row-wise kernel");
    timing_begin(s);
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL(k_spmm_rowwise<GCN_EPI_NONE>, grid, dim3(256), 0, s, n, m.rowptr, m.colidx, o.pattern ? nullptr : m.val, o.row_scale, f, X, ldx, Z, ldz, Zprev, ldzprev); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL(k_spmm_rowwise<GCN_EPI_RELU>, grid, dim3(256), 0, s, n, m.rowptr, m.colidx, o.pattern ? nullptr : m.val, o.row_scale, f, X, ldx, Z, ldz, Zprev, ldzprev); break;
        default: hipLaunchKernelGGL(k_spmm_rowwise<GCN_EPI_MASK>, grid, dim3(256), 0, s, n, m.rowptr, m.colidx, o.pattern ? nullptr : m.val, o.row_scale, f, X, ldx, Z, ldz, Zprev, ldzprev); break;
    }
    timing_end(s);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

static void took(gcn_csr* a, int sched) {
    g_last_schedule = sched;
    a->last_schedule = sched;
}

static int launch_product(gcn_csr* a, Matrix& m, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                          int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s, const SpmmOpt& asked, SpmmPlan** plan) {
    SpmmOpt o = asked;
    const int64_t n = m.nrows, ncols = m.ncols, nnz = a->nnz;
    const Config& cfg = cfg_of(a);
    if (nnz == 0) {
        if (o.describe) *o.describe += "empty";
        if (o.dry) return GCN_OK;
        const int64_t work = n * f;
        hipLaunchKernelGGL(k_zero_empty_rows, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, s, n, m.rowptr, f, Z, ldz);
        GCN_LAUNCH_CHECK();
        return GCN_OK;
    }
    int algo = cfg.spmm_algo;
    const bool vec4_all = (f % 4 == 0) && (ldx % 4 == 0) && (ldz % 4 == 0) && aligned16(X) && aligned16(Z) &&
                          (epilogue != GCN_EPI_MASK || ((ldzprev % 4 == 0) && aligned16(Zprev)));
    int64_t nblocks = choose_blocks(cfg, n, ncols, nnz, f, 24);
    int32_t heavy = cfg.sweep_heavy, parts = 1;
    int64_t heavy_blocks = 0;                              // 0: by sizes
    if (algo == 0) {
        // Column sweep when X is far beyond the caches, rows are long enough to give every task a
        // real walk over the columns, and too short for partial-row blocking; else nonzero-split.
        const int64_t panel = f < 32 ? f : 32;
        const bool huge = ncols * panel * 4 > (64ll << 20);
        // one step of a task spans about groups^2 * ncols * rowbytes / (rows_per_task * mean_degree) bytes
        // of X (64 * ncols / degree at width 16); the sweep pays while that stays within an L2
        const int64_t deg = nnz / n;
        const bool narrow_steps = deg >= 64 && 64 * ncols / deg <= (6ll << 20);
        algo = (huge && vec4_all && nblocks < 2 && narrow_steps) ? 3 : 2;
    }
    if (algo == 3 && f < 4) algo = 2;
    bool hub_first = nblocks < 2;
    if (algo == 2 && cfg.spmm_algo == 0 && cfg.spmm_blocks == 0 && asked.any_schedule && worth_a_plan(m, f, nnz)) {
        // (without the stored values the caller's row factors decide; those of this library are 1 / sqrt(d_i))
        const Terms terms = o.pattern && m.terms != Terms::BY_BOTH ? Terms::UNKNOWN : m.terms;
        SpmmPlan& p = plan_of(a, m, f, terms, nblocks);
        *plan = &p;
        if (p.sweep) {
            algo = 3;
            heavy = std::min(heavy, p.heavy);
            parts = p.parts;
            heavy_blocks = p.blocks;
        } else nblocks = p.blocks;
        o.narrow = p.narrow;
    }
    if (rowwise_only(m, ldx, Z, ldz, epilogue, Zprev, ldzprev)) algo = 1;
    const int sweep_lanes = f <= 16 ? 4 : 8;
    const int32_t rb = sweep_rows(4 * sweep_lanes);
    if (algo == 3) {
        // How many places the copy takes shows when it is built, not in the lengths of the rows: where the rows of a task select runs of
        // columns that its other rows do not, few of them fill a set (rows of 41 on columns 41 i on: 8 places per entry, 1834 us
        // where the nonzero split takes 394).  Such a matrix goes on without it, by the sizes.  Planned copies of 700 renamed graphs
        // took 1.03 at the most, those chosen by sizes (rows up to 1024 entries, R-MAT) 1.53; at 2.2 the walk is slower than the gathers it saves.
        const double most = cfg.spmm_algo == 3 ? 0.0 : (*plan ? 1.25 * (*plan)->padding : 2.0);
        GCN_TRY(want_sweep(m, nnz, 64 / sweep_lanes, rb, heavy, most, s));
        if (m.swp.sparser(most)) {
            algo = 2;
            if (*plan) {
                (*plan)->give_way();
                nblocks = (*plan)->blocks;
                o.narrow = (*plan)->narrow;
            }
        }
    }
    if ((algo == 2 && cfg.spmm_algo == 0) || algo == 4) {
        // Hub schedule: for operands beyond the L2s when most entries sit in long rows and hot columns
        // (decided from the matrix itself when the copy is built; a rejected shape is remembered).
        const bool forced = algo == 4;
        algo = 2;
        const int64_t panel = f < 32 ? f : 32;
        int64_t H = 0, cpb = 0;
        hub_shape(cfg, ncols, f, &H, &cpb);
        // Measured: it pays when a gathered row is narrower than a 128-byte line (packing then also puts
        // two hot rows into one line: config 4, width 16, 4.33 -> 3.15 ms) and not at 128 bytes per row
        // (config 2: 1.44 -> 1.48 ms), so the automatic choice is limited to panels below 32 floats.
        const bool eligible = vec4_all && hub_first && H >= 2 * cpb && nnz >= (forced ? 1 : (4ll << 20)) &&
                              (forced || (panel < 32 && ncols * panel * 4 > (32ll << 20)));
        if (eligible) {
            // built once per matrix and settings for the width of the first product that qualifies
            GCN_TRY(want_hub(m, cfg, nnz, H, cpb, forced, s));
            if (m.hub.state == 1) {
                took(a, GCN_SCHED_HUB);
                return run_hub(a, m, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, o, s);
            }
        }
    }
    if (algo == 3) {
        took(a, GCN_SCHED_SWEEP);
        const int LPRs = sweep_lanes, W = LPRs * 4;
        const Sweep& w = m.swp;
        if (o.describe) {
            const int64_t cap = (int64_t)device_info().cus * sweep_tasks(cfg);
            char t[240];
            snprintf(t, sizeof t, "sweep(entries_per_step=%d,rows_per_task=%d,long_row>%d,sums_per_row=%d,tasks=%lld,launches=%lld,stored=%lld,kernel=k_spmm_sweep<%d>)",
                     64 / LPRs, (int)rb, (int)heavy, (int)parts, (long long)w.ntasks,
                     (long long)(((w.ntasks + cap - 1) / cap) * ((f + W - 1) / W)), (long long)w.padded, LPRs);
            *o.describe += t;
        }
        if (!o.dry) {
            SweepArgs sa;
            sa.colidx = w.colidx; sa.val = o.pattern ? nullptr : w.val; sa.row_scale = o.row_scale; sa.lrow = w.lrow; sa.task_base = w.task_base; sa.task_len = w.task_len; sa.task_order = w.task_order;
            sa.n = n; sa.f = f; sa.rb = rb; sa.parts = parts; sa.X = X; sa.ldx = ldx; sa.Z = Z; sa.ldz = ldz; sa.Zprev = Zprev; sa.ldzprev = ldzprev;
            const auto launch = LPRs == 4 ? (o.pattern ? launch_sweep<4, false> : launch_sweep<4, true>)
                                          : (o.pattern ? launch_sweep<8, false> : launch_sweep<8, true>);
            GCN_TRY(launch(sa, w.ntasks, sweep_tasks(cfg), epilogue, s));
        }
        if (w.heavy) {
            // long rows: nonzero-split kernel over the row subset; their rows are long enough for the
            // column-blocked form to pay even with many blocks
            Matrix& h = *w.heavy;
            const int64_t hb = heavy_blocks > 0 ? heavy_blocks : choose_blocks(cfg, h.nrows, ncols, w.nnz_heavy, f, 30);
            if (o.describe) *o.describe += "+long_rows:";
            GCN_TRY(run_matrix(a, h, h.ne_rows, w.nnz_heavy, hb, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, o, s));
        }
        return GCN_OK;
    }
    if (algo == 1) {
        took(a, GCN_SCHED_ROWWISE);
        if (o.describe) *o.describe += "rowwise";
        if (o.dry) return GCN_OK;
        return launch_rowwise(m, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, o, s);
    }
    took(a, nblocks >= 2 ? GCN_SCHED_BLOCKED : GCN_SCHED_SPLIT);
    return run_matrix(a, m, nullptr, nnz, nblocks, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, o, s);
}

int spmm_launch(gcn_csr* a, Matrix& m, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s, const SpmmOpt& asked) {
    const size_t said = asked.describe ? asked.describe->size() : 0;
    return run_or_by_sizes(GCN_ERR_OOM, [&](SpmmPlan** plan) {
        if (asked.describe) asked.describe->resize(said);
        return launch_product(a, m, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, s, asked, plan);
    });
}

// For a matrix this library normalised symmetrically, D^-1/2 (A+I) D^-1/2 X = D^-1/2 ((A+I) (D^-1/2 X))
// (section "Graph Neural Networks"): the product can skip the stored values, which halves the
// index/value stream.  It pays when rows are long (the pre-scaling pass over X is amortised).
bool use_value_free(const gcn_csr* a) {
    const int mode = cfg_of(a).pattern_spmm;
    if (!a->inv_sqrt_deg || mode == 0) return false;
    return mode == 1 || a->nnz / (a->n > 0 ? a->n : 1) >= 64;
}

int spmm_prepare(gcn_csr* a, Matrix& m, int32_t f, hipStream_t s, bool any_schedule, bool pattern) {
    SpmmOpt o;
    o.dry = true;
    o.any_schedule = any_schedule;
    o.pattern = pattern;
    return spmm_launch(a, m, f, nullptr, f, nullptr, f, GCN_EPI_NONE, nullptr, 0, s, o);
}

}  // namespace gcn

using namespace gcn;

static inline hipStream_t s_of(void* stream) { return (hipStream_t)stream; }

static int check_spmm_args(const char* who, const gcn_csr* a, int trans, int32_t f, const float* X, int64_t ldx,
                           const float* Z, int64_t ldz, int epilogue, const float* Zprev, int64_t ldzprev) {
    if (!a || !X || !Z) return fail(GCN_ERR_BADARG, "%s: NULL argument", who);
    if (f <= 0 || ldx < f || ldz < f) return fail(GCN_ERR_BADARG, "%s: need f > 0, ldx >= f, ldz >= f", who);
    if (epilogue < GCN_EPI_NONE || epilogue > GCN_EPI_MASK) return fail(GCN_ERR_BADARG, "%s: unknown epilogue", who);
    if (epilogue == GCN_EPI_MASK && (!Zprev || ldzprev < f)) return fail(GCN_ERR_BADARG, "%s: mask epilogue needs Zprev with ld >= f", who);
    if (trans && !a->has_t) return fail(GCN_ERR_NOTRANSPOSE, "%s: trans=1 needs GCN_BUILD_TRANSPOSE", who);
    // X and Z must not overlap: the product gathers rows of X while rows of Z are written
    const int64_t xrows = trans ? a->n : a->ncols, zrows = trans ? a->ncols : a->n;
    const char* xb = (const char*)X; const char* xe = xb + ((size_t)(xrows - 1) * ldx + f) * sizeof(float);
    const char* zb = (const char*)Z; const char* ze = zb + ((size_t)(zrows - 1) * ldz + f) * sizeof(float);
    if (xb < ze && zb < xe) return fail(GCN_ERR_BADARG, "%s: X and Z overlap", who);
    return GCN_OK;
}

// Whether a stand-alone product may take any schedule: not at the ragged widths, whose kernels all add alike, and not the
// forward product A^T X, plain or with a ReLU, on which the first hidden layer of gcn_epoch_preaggregated (or of the caller's
// own) decides.  A ReLU never changes the sums: A X takes the same schedule with and without one, and so does A^T X.
static bool free_schedule(int32_t f, int trans, int epilogue) { return f % 4 == 0 && !(trans && epilogue != GCN_EPI_MASK); }

extern "C" int gcn_spmm(gcn_csr* a, int trans, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                        int epilogue, const float* Zprev, int64_t ldzprev, void* stream) {
    GCN_TRY(check_spmm_args("gcn_spmm", a, trans, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev));
    PhaseTimer whole(s_of(stream), GCN_PHASE_SPMM);           // the whole product: every kernel it queues
    if (use_value_free(a)) {
        // value-free form: a pre-scaled copy of X in the handle (n x f), then sums of gathered rows, the output
        // rows scaled in the kernels' store path; differs from the valued product by fp32 roundings only
        GCN_TRY(grow_retire(a, &a->xs, &a->xs_bytes, (size_t)a->n * (size_t)f * sizeof(float)));
        GCN_TRY(scale_rows_launch(a->n, f, X, ldx, a->inv_sqrt_deg, a->xs, f, s_of(stream)));
        SpmmOpt o;
        o.pattern = true;
        o.row_scale = a->inv_sqrt_deg;
        o.any_schedule = free_schedule(f, trans, epilogue);
        return spmm_launch(a, matrix_of(a, trans), f, a->xs, f, Z, ldz, epilogue, Zprev, ldzprev, s_of(stream), o);
    }
    SpmmOpt o;
    o.any_schedule = free_schedule(f, trans, epilogue);
    return spmm_launch(a, matrix_of(a, trans), f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, (hipStream_t)stream, o);
}

extern "C" int gcn_spmm_prepare(gcn_csr* a, int trans, int32_t f, void* stream) {
    if (!a || f <= 0) return fail(GCN_ERR_BADARG, "gcn_spmm_prepare: NULL matrix or f <= 0");
    if (trans && !a->has_t) return fail(GCN_ERR_NOTRANSPOSE, "gcn_spmm_prepare: trans=1 needs GCN_BUILD_TRANSPOSE");
    if (use_value_free(a)) GCN_TRY(grow_retire(a, &a->xs, &a->xs_bytes, (size_t)a->n * (size_t)f * sizeof(float)));
    // for the layer calls too: their backward and last products are free at every width; and for gcn_spmm_pattern, whose schedule may be another
    // where the stored values tell more than the caller's row factors (see Terms)
    Matrix& m = matrix_of(a, trans);
    if (!free_schedule(f, trans, GCN_EPI_NONE)) GCN_TRY(spmm_prepare(a, m, f, (hipStream_t)stream, false));
    if (m.terms != Terms::BY_BOTH && m.terms != Terms::UNKNOWN) GCN_TRY(spmm_prepare(a, m, f, (hipStream_t)stream, true, true));
    return spmm_prepare(a, m, f, (hipStream_t)stream, true);
}

extern "C" int gcn_spmm_describe(gcn_csr* a, int trans, int32_t f, char* out, size_t out_bytes, void* stream) {
    if (!a || f <= 0 || !out || out_bytes == 0) return fail(GCN_ERR_BADARG, "gcn_spmm_describe: bad argument");
    if (trans && !a->has_t) return fail(GCN_ERR_NOTRANSPOSE, "gcn_spmm_describe: trans=1 needs GCN_BUILD_TRANSPOSE");
    std::string text;
    SpmmOpt o;
    o.dry = true;
    o.describe = &text;
    o.any_schedule = free_schedule(f, trans, GCN_EPI_NONE);
    o.pattern = use_value_free(a);
    GCN_TRY(spmm_launch(a, matrix_of(a, trans), f, nullptr, f, nullptr, f, GCN_EPI_NONE, nullptr, 0, (hipStream_t)stream, o));
    if (o.pattern) text += "; value-free (operand rows pre-scaled by d^-1/2, output rows scaled)";
    snprintf(out, out_bytes, "%s", text.c_str());
    return GCN_OK;
}

// ---- the product for callers that cannot allocate --------------------------------------------------------
// The nonzero-split kernel needs one row of f floats per 512 stored entries for the pieces of rows that
// cross wavefronts.  gcn_spmm keeps that buffer in the handle and grows it with hipMalloc; this entry point
// keeps it in a fixed array in the library's device image instead, so that it never allocates.  Each GPU
// has its own copy of the array at its own address; the address is looked up once per device.
static constexpr size_t STATIC_SCRATCH_BYTES = GCN_SPMM_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
static constexpr int STATIC_MAX_DEVICES = 64;
static std::mutex g_static_mu;
static void* g_static_ptr[STATIC_MAX_DEVICES] = {};

static int static_scratch(float** out) {
    int dev = -1;
    GCN_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= STATIC_MAX_DEVICES) return fail(GCN_ERR_RANGE, "gcn_spmm_static: device index %d not supported", dev);
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[dev]) {
        void* ptr = nullptr;
        GCN_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));      // with `dev` current: this device's copy
        if (!ptr) return fail(GCN_ERR_HIP, "gcn_spmm_static: no address for the scratch array on device %d", dev);
        g_static_ptr[dev] = ptr;
    }
    *out = (float*)g_static_ptr[dev];
    return GCN_OK;
}

extern "C" int gcn_spmm_static(gcn_csr* a, int trans, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                               int epilogue, const float* Zprev, int64_t ldzprev, void* stream) {
    GCN_TRY(check_spmm_args("gcn_spmm_static", a, trans, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev));
    int dev = -1;
    GCN_HIP_TRY(hipGetDevice(&dev));
    if (dev != a->device) return fail(GCN_ERR_BADARG, "gcn_spmm_static: the matrix lives on device %d, current device is %d", a->device, dev);
    Matrix& m = matrix_of(a, trans);
    const size_t need = (size_t)m.nchunks * (size_t)f * sizeof(float);
    if (need > STATIC_SCRATCH_BYTES)
        return fail(GCN_ERR_WORKSPACE, "gcn_spmm_static: needs %zu bytes of scratch (%lld stored entries / 512, rounded up, x %d floats), the fixed "
                    "array holds %zu; use gcn_spmm", need, (long long)a->nnz, (int)f, STATIC_SCRATCH_BYTES);
    hipStream_t s = (hipStream_t)stream;
    if (a->nnz == 0) return zero_empty_rows(m, f, Z, ldz, s);
    if (rowwise_only(m, ldx, Z, ldz, epilogue, Zprev, ldzprev)) {
        took(a, GCN_SCHED_ROWWISE);
        return launch_rowwise(m, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, SpmmOpt(), s);
    }
    float* carry = nullptr;
    GCN_TRY(static_scratch(&carry));
    took(a, GCN_SCHED_SPLIT);
    return run_matrix(a, m, nullptr, a->nnz, 1, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, SpmmOpt(), s, carry);
}

extern "C" int gcn_spmm_pattern(gcn_csr* a, int trans, int32_t f, const float* X, int64_t ldx, float* Z, int64_t ldz,
                                const float* row_scale, int epilogue, const float* Zprev, int64_t ldzprev,
                                void* stream) {
    GCN_TRY(check_spmm_args("gcn_spmm_pattern", a, trans, f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev));
    SpmmOpt o;
    o.pattern = true;
    o.row_scale = row_scale;
    o.any_schedule = free_schedule(f, trans, epilogue);
    PhaseTimer whole(s_of(stream), GCN_PHASE_SPMM);
    return spmm_launch(a, matrix_of(a, trans), f, X, ldx, Z, ldz, epilogue, Zprev, ldzprev, (hipStream_t)stream, o);
}
