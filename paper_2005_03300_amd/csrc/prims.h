// Device-wide integer primitives for graph construction: exclusive prefix sum, stable
// least-significant-digit radix sort (keys alone or keys with a payload), and ordered selection
// (of which the removal of equal neighbours is one use).  Hand-written for 64-wide wavefronts;
// all of them are used only while a matrix or a schedule is built, never inside an epoch.
//
// The functions queue their work on the stream and return; select waits for the stream when the caller asks for the
// count.  Temporary buffers are reused in stream order by the BuildScope that every caller has open.
#pragma once
#include <type_traits>

#include "common.h"

namespace gcn {
namespace prims {

constexpr int P_TPB = 256;                 // 4 wavefronts
constexpr int P_WAVES = P_TPB / 64;
constexpr int SCAN_ITEMS = 8;              // consecutive elements per thread
constexpr int SCAN_TILE = P_TPB * SCAN_ITEMS;
constexpr int RS_ROUNDS = 32;              // 256 keys per round
constexpr int RS_TILE = P_TPB * RS_ROUNDS;
constexpr int RS_RADIX = 256;              // 8-bit digits

struct NoValue {};

using Scratch = TempBuf;

// ---- wavefront and workgroup scans -----------------------------------------------------------------

template <typename T> __device__ inline T shfl_up_any(T v, int d) {
    if constexpr (sizeof(T) == 8) return (T)__shfl_up((unsigned long long)v, d, 64);
    else return (T)__shfl_up((unsigned)v, d, 64);
}

template <typename T> __device__ inline T wave_inclusive_sum(T v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        T u = shfl_up_any(v, d);
        if (lane >= d) v += u;
    }
    return v;
}

// Exclusive prefix of v over the 256 threads of the workgroup; total receives the workgroup's sum.
// part is P_WAVES elements of LDS; the call ends with a barrier, so part may be reused at once.
template <typename T> __device__ inline T block_exclusive_sum(T v, T* part, T& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const T inc = wave_inclusive_sum(v);
    if (lane == 63) part[w] = inc;
    __syncthreads();
    T base = 0, all = 0;
#pragma unroll
    for (int i = 0; i < P_WAVES; ++i) {
        const T p = part[i];
        if (i < w) base += p;
        all += p;
    }
    __syncthreads();
    total = all;
    return base + inc - v;
}

// ---- exclusive prefix sum --------------------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(P_TPB) void k_scan_tile_sums(const T* __restrict__ in, size_t n, T* __restrict__ sums) {
    __shared__ T part[P_WAVES];
    const size_t base = (size_t)blockIdx.x * SCAN_TILE + (size_t)threadIdx.x * SCAN_ITEMS;
    T a = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k)
        if (base + k < n) a += in[base + k];
    T total;
    block_exclusive_sum(a, part, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// in == out is allowed: a workgroup reads its whole tile before it writes any of it.
template <typename T>
__global__ __launch_bounds__(P_TPB) void k_scan_tiles(const T* in, T* out, size_t n, const T* __restrict__ tile_off) {
    __shared__ T part[P_WAVES];
    const size_t base = (size_t)blockIdx.x * SCAN_TILE + (size_t)threadIdx.x * SCAN_ITEMS;
    T x[SCAN_ITEMS];
    T a = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        x[k] = base + k < n ? in[base + k] : (T)0;
        a += x[k];
    }
    T total;
    T run = block_exclusive_sum(a, part, total) + (tile_off ? tile_off[blockIdx.x] : (T)0);
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        if (base + k < n) out[base + k] = run;
        run += x[k];
    }
}

// out[i] = in[0] + ... + in[i-1]; in == out allowed.
template <typename T> int exclusive_scan(const T* in, T* out, size_t n, hipStream_t s) {
    if (n == 0) return GCN_OK;
    const size_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (ntiles >= (1ull << 31)) return fail(GCN_ERR_RANGE, "exclusive_scan: %zu elements are too many", n);
    if (ntiles == 1) {
        hipLaunchKernelGGL(k_scan_tiles<T>, dim3(1), dim3(P_TPB), 0, s, in, out, n, (const T*)nullptr);
        GCN_LAUNCH_CHECK();
        return GCN_OK;
    }
    Scratch sums;
    GCN_TRY(sums.alloc(ntiles * sizeof(T)));
    hipLaunchKernelGGL(k_scan_tile_sums<T>, dim3((unsigned)ntiles), dim3(P_TPB), 0, s, in, n, sums.as<T>());
    GCN_LAUNCH_CHECK();
    GCN_TRY(exclusive_scan<T>(sums.as<T>(), sums.as<T>(), ntiles, s));
    hipLaunchKernelGGL(k_scan_tiles<T>, dim3((unsigned)ntiles), dim3(P_TPB), 0, s, in, out, n, (const T*)sums.as<T>());
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// ---- ordered selection -----------------------------------------------------------------------------
// pred(i) decides whether index i is kept; emit(i, pos) stores it as the pos-th kept one.  Kept
// indices keep their order.  Both functors are called once per index in each of two passes.
// A tile's indices are dealt out 64 at a time to the wavefronts, so that neighbouring lanes read and write neighbouring
// elements; a wavefront counts and ranks its 64 by ballot (unique over 34.6 M keys: 505 -> 200 us).

// ITEMS: indices per thread.  SEL_ITEMS, or one where a predicate is a chain of loads and the candidates are few: 65 K of them in 16
// tiles took 16 us per pass, in 256 tiles 4.

constexpr int SEL_ITEMS = 16;
template <int ITEMS> constexpr int64_t sel_tiles(int64_t n) { return (n + P_TPB * ITEMS - 1) / (P_TPB * ITEMS); }

template <int SEL_ITEMS, typename Pred>
__global__ __launch_bounds__(P_TPB) void k_select_count(int64_t n, Pred pred, int64_t* __restrict__ tile_cnt) {
    __shared__ int part[P_WAVES];
    const int64_t base = (int64_t)blockIdx.x * (P_TPB * SEL_ITEMS) + threadIdx.x;
    int c = 0;                                     // the same in every lane of a wavefront
#pragma unroll
    for (int k = 0; k < SEL_ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * P_TPB;
        c += __popcll(__ballot(i < n && pred(i)));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < P_WAVES; ++w) t += part[w];
        tile_cnt[blockIdx.x] = t;
    }
}

template <int SEL_ITEMS, typename Pred, typename Emit>
__global__ __launch_bounds__(P_TPB) void k_select_emit(int64_t n, Pred pred, Emit emit,
                                                      const int64_t* __restrict__ tile_off) {
    __shared__ int cnt[SEL_ITEMS * P_WAVES];       // kept indices of every 64, in index order
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * (P_TPB * SEL_ITEMS) + threadIdx.x;
    unsigned long long kept[SEL_ITEMS];
#pragma unroll
    for (int k = 0; k < SEL_ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * P_TPB;
        kept[k] = __ballot(i < n && pred(i));
        if (lane == 0) cnt[k * P_WAVES + w] = __popcll(kept[k]);
    }
    __syncthreads();
    static_assert(SEL_ITEMS * P_WAVES <= 64, "one wavefront scans the counts");
    if (w == 0) {
        const int c = lane < SEL_ITEMS * P_WAVES ? cnt[lane] : 0, before = (int)wave_inclusive_sum((unsigned)c) - c;
        if (lane < SEL_ITEMS * P_WAVES) cnt[lane] = before;
    }
    __syncthreads();
    const int64_t off = tile_off[blockIdx.x];
#pragma unroll
    for (int k = 0; k < SEL_ITEMS; ++k)
        if (kept[k] >> lane & 1ull)
            emit(base + (int64_t)k * P_TPB, off + cnt[k * P_WAVES + w] + __popcll(kept[k] & ((1ull << lane) - 1ull)));
}

// The first pass: tile_off receives the position of each tile's first kept index and, behind them, the number of kept ones.
template <int ITEMS = SEL_ITEMS, typename Pred> int select_positions(int64_t n, Pred pred, Scratch& tile_off, hipStream_t s) {
    const int64_t ntiles = sel_tiles<ITEMS>(n);
    if (ntiles >= (1ll << 31)) return fail(GCN_ERR_RANGE, "select: %lld candidates are too many", (long long)n);
    GCN_TRY(tile_off.alloc((size_t)(ntiles + 1) * 8));
    int64_t* const cnt = tile_off.as<int64_t>();
    GCN_HIP_TRY(hipMemsetAsync(cnt + ntiles, 0, 8, s));
    hipLaunchKernelGGL((k_select_count<ITEMS, Pred>), dim3((unsigned)ntiles), dim3(P_TPB), 0, s, n, pred, cnt);
    GCN_LAUNCH_CHECK();
    return exclusive_scan<int64_t>(cnt, cnt, (size_t)ntiles + 1, s);
}
template <int ITEMS = SEL_ITEMS> const int64_t* select_total(int64_t n, const Scratch& tile_off) { return tile_off.as<int64_t>() + sel_tiles<ITEMS>(n); }

// The second.
template <int ITEMS = SEL_ITEMS, typename Pred, typename Emit> int select_store(int64_t n, Pred pred, Emit emit, const Scratch& tile_off, hipStream_t s) {
    hipLaunchKernelGGL((k_select_emit<ITEMS, Pred, Emit>), dim3((unsigned)sel_tiles<ITEMS>(n)), dim3(P_TPB), 0, s, n, pred, emit,
                       (const int64_t*)tile_off.as<int64_t>());
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

template <typename Pred, typename Emit> int select(int64_t n, Pred pred, Emit emit, int64_t* count, hipStream_t s) {
    if (count) *count = 0;
    if (n <= 0) return GCN_OK;
    Scratch off;
    GCN_TRY(select_positions(n, pred, off, s));
    GCN_TRY(select_store(n, pred, emit, off, s));
    if (!count) return GCN_OK;
    GCN_HIP_TRY(hipMemcpyAsync(count, select_total(n, off), 8, hipMemcpyDeviceToHost, s));
    GCN_HIP_TRY(hipStreamSynchronize(s));
    return GCN_OK;
}

struct EmitIndex32 {   // out[pos] = i
    int32_t* out;
    __device__ void operator()(int64_t i, int64_t pos) const { out[pos] = (int32_t)i; }
};

// The indices 0 <= i < n (n below 2^31) with pred(i), ascending.
template <typename Pred> int select_indices(int64_t n, Pred pred, int32_t* out, int64_t* count, hipStream_t s) {
    if (n >= (1ll << 31)) return fail(GCN_ERR_RANGE, "select_indices: %lld candidates do not fit 32-bit ids", (long long)n);
    return select(n, pred, EmitIndex32{out}, count, s);
}

struct FirstOfRun {
    const uint64_t* in;
    __device__ bool operator()(int64_t i) const { return i == 0 || in[i] != in[i - 1]; }
};
struct EmitKey {
    const uint64_t* in;
    uint64_t* out;
    __device__ void operator()(int64_t i, int64_t pos) const { out[pos] = in[i]; }
};

// Keeps the first key of every run of equal neighbours (in and out must not overlap).
inline int unique_keys(const uint64_t* in, uint64_t* out, int64_t n, int64_t* count, hipStream_t s) {
    return select(n, FirstOfRun{in}, EmitKey{in, out}, count, s);
}

// ---- radix sort ------------------------------------------------------------------------------------
// One pass orders the keys by one 8-bit digit and keeps the order of equal digits, so passes from
// the lowest digit upwards sort the keys and equal keys keep their input order.  A pass takes three
// steps: every workgroup counts the digits of its tile of RS_TILE keys; an exclusive prefix sum of
// the counts laid out digit-major (digit d of tile t at d*ntiles + t) gives each (digit, tile) its
// first output position; the workgroup then reads the tile again and stores it.  There a wavefront owns
// 64 RS_ITEMS consecutive keys and ranks each among its own earlier keys of the same digit (ballots and a counter per
// digit in LDS that only this wavefront touches: no barrier); one prefix sum over digits and wavefronts turns the ranks
// into positions inside the tile, the keys go to those positions in LDS, and leave from there in order, so that the
// keys of one digit are written as one run (32 of them on average).  Bound by memory: 34.6 M 8-byte keys take 391 us per
// pass when every key is stored from where it was read, about 152 us this way.

template <typename K> __device__ inline unsigned digit_of(K key, unsigned shift, unsigned mask, unsigned flip) {
    return ((unsigned)(key >> shift) & mask) ^ flip;
}

// Where the keys of a pass come from: an array, or (first pass) whatever computes the i-th key and may find it wrong, which the
// counting kernel reports once per thread.
template <typename K> struct KeyArray {
    typedef K Key;
    const K* keys;
    __device__ K operator()(size_t i, bool&) const { return keys[i]; }
    __device__ void report() const {}
};

// Whole-key histograms of every digit position at once: hist[p*256 + d] = keys whose p-th byte is d.
template <typename K>
__global__ __launch_bounds__(P_TPB) void k_radix_byte_hist(const K* __restrict__ keys, size_t n,
                                                          unsigned long long* __restrict__ hist) {
    constexpr int NB = sizeof(K);
    __shared__ unsigned h[NB * RS_RADIX];
    for (int i = threadIdx.x; i < NB * RS_RADIX; i += P_TPB) h[i] = 0;
    __syncthreads();
    // a thread adds a run of equal bytes with one LDS atomic: positions at which all keys agree
    // (the unused high bytes of small ids) would otherwise serialise on one counter
    const size_t base = (size_t)blockIdx.x * RS_TILE;
    unsigned last[NB], run[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) { last[p] = 0; run[p] = 0; }
    for (int r = 0; r < RS_ROUNDS; ++r) {
        const size_t i = base + (size_t)r * P_TPB + threadIdx.x;
        if (i < n) {
            const K key = keys[i];
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                const unsigned d = (unsigned)(key >> (8 * p)) & 255u;
                if (run[p] && d != last[p]) { atomicAdd(&h[p * RS_RADIX + last[p]], run[p]); run[p] = 0; }
                last[p] = d;
                ++run[p];
            }
        }
    }
#pragma unroll
    for (int p = 0; p < NB; ++p)
        if (run[p]) atomicAdd(&h[p * RS_RADIX + last[p]], run[p]);
    __syncthreads();
    for (int i = threadIdx.x; i < NB * RS_RADIX; i += P_TPB)
        if (h[i]) atomicAdd(&hist[i], (unsigned long long)h[i]);
}

// Bound by memory: eight keys of a thread are on their way at a time (34.6 M 8-byte keys: 96 us with one, 66 with eight).
template <typename Source, typename Off>
__global__ __launch_bounds__(P_TPB) void k_radix_tile_hist(Source key_at, size_t n, unsigned shift,
                                                          unsigned mask, unsigned flip, size_t ntiles,
                                                          Off* __restrict__ hist) {
    constexpr int AT_ONCE = 8;
    typedef typename Source::Key K;
    __shared__ unsigned h[RS_RADIX];
    h[threadIdx.x] = 0;
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * RS_TILE;
    unsigned last = 0, run = 0;
    bool wrong = false;
    for (int r = 0; r < RS_ROUNDS; r += AT_ONCE) {
        K key[AT_ONCE];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) {
            const size_t i = base + (size_t)(r + e) * P_TPB + threadIdx.x;
            key[e] = key_at(i < n ? i : n - 1, wrong);
        }
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) {
            if (base + (size_t)(r + e) * P_TPB + threadIdx.x >= n) break;
            const unsigned d = digit_of(key[e], shift, mask, flip);
            if (run && d != last) { atomicAdd(&h[last], run); run = 0; }
            last = d;
            ++run;
        }
    }
    if (run) atomicAdd(&h[last], run);
    if (wrong) key_at.report();
    __syncthreads();
    hist[(size_t)threadIdx.x * ntiles + blockIdx.x] = (Off)h[threadIdx.x];
}

constexpr int RS_TPB = 512;
constexpr int RS_WAVES = RS_TPB / 64;
constexpr int RS_ITEMS = RS_TILE / RS_TPB;         // keys per thread

template <typename K, typename V> constexpr size_t radix_lds_bytes() {
    constexpr size_t v = std::is_same<V, NoValue>::value ? 0 : sizeof(V);
    return (size_t)RS_TILE * (sizeof(K) > v ? sizeof(K) : v);
}

template <typename Source, typename V, typename Off>
__global__ __launch_bounds__(RS_TPB) void k_radix_scatter(Source key_at, typename Source::Key* __restrict__ kout,
                                                         const V* __restrict__ vin, V* __restrict__ vout, size_t n,
                                                         unsigned shift, unsigned mask, unsigned flip, size_t ntiles,
                                                         const Off* __restrict__ first) {
    typedef typename Source::Key K;
    extern __shared__ __align__(16) unsigned char s_tile[];    // the tile's keys, then its payload, in output order
    __shared__ unsigned cnt[RS_WAVES][RS_RADIX];    // keys of each digit by wavefront; then their first place in the tile
    __shared__ Off place[RS_RADIX];                 // output position of a digit's keys less their place in the tile
    __shared__ unsigned part[RS_RADIX / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t base = (size_t)blockIdx.x * RS_TILE;
    const int left = n - base < (size_t)RS_TILE ? (int)(n - base) : RS_TILE;
    for (int i = threadIdx.x; i < RS_WAVES * RS_RADIX; i += RS_TPB) (&cnt[0][0])[i] = 0;
    const int t0 = w * 64 * RS_ITEMS + lane;        // the thread's keys are t0 + 64 k
    K key[RS_ITEMS];
    bool wrong = false;                             // (reported by the counting kernel)
#pragma unroll
    for (int k = 0; k < RS_ITEMS; ++k) {
        key[k] = 0;
        if (t0 + 64 * k < left) key[k] = key_at(base + t0 + 64 * k, wrong);
    }
    __syncthreads();
    unsigned rank[RS_ITEMS];
#pragma unroll
    for (int k = 0; k < RS_ITEMS; ++k) {
        const bool valid = t0 + 64 * k < left;
        const unsigned d = digit_of(key[k], shift, mask, flip);
        unsigned long long peers = __ballot(valid);             // lanes of this wavefront that hold the same digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = d >> b & 1u;
            const unsigned long long have = __ballot(valid && bit);
            peers &= bit ? have : ~have;
        }
        const unsigned before = (unsigned)__popcll(peers & ((1ull << lane) - 1ull));
        unsigned seen = 0;
        if (valid) seen = cnt[w][d];
        // the wavefront's LDS operations complete in program order; the fences keep the compiler to it
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) cnt[w][d] = seen + (unsigned)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        rank[k] = seen + before;
    }
    __syncthreads();
    // first place in the tile of every (digit, wavefront)
    unsigned mine = 0, inc = 0;
    if (threadIdx.x < RS_RADIX) {
#pragma unroll
        for (int i = 0; i < RS_WAVES; ++i) {
            const unsigned c = cnt[i][threadIdx.x];
            cnt[i][threadIdx.x] = mine;
            mine += c;
        }
        inc = wave_inclusive_sum(mine);
        if (lane == 63) part[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x < RS_RADIX) {
        unsigned start = inc - mine;
        for (int i = 0; i < w; ++i) start += part[i];
#pragma unroll
        for (int i = 0; i < RS_WAVES; ++i) cnt[i][threadIdx.x] += start;
        place[threadIdx.x] = first[(size_t)threadIdx.x * ntiles + blockIdx.x] - (Off)start;
    }
    __syncthreads();
    K* sk = reinterpret_cast<K*>(s_tile);
#pragma unroll
    for (int k = 0; k < RS_ITEMS; ++k) {
        rank[k] += cnt[w][digit_of(key[k], shift, mask, flip)];
        if (t0 + 64 * k < left) sk[rank[k]] = key[k];
    }
    __syncthreads();
    Off pos[RS_ITEMS];
#pragma unroll
    for (int k = 0; k < RS_ITEMS; ++k) {
        const int j = threadIdx.x + k * RS_TPB;
        pos[k] = 0;
        if (j < left) {
            const K out = sk[j];
            pos[k] = place[digit_of(out, shift, mask, flip)] + (Off)j;
            kout[pos[k]] = out;
        }
    }
    if constexpr (!std::is_same<V, NoValue>::value) {
        V* sv = reinterpret_cast<V*>(s_tile);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RS_ITEMS; ++k)
            if (t0 + 64 * k < left) sv[rank[k]] = vin[base + t0 + 64 * k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RS_ITEMS; ++k) {
            const int j = threadIdx.x + k * RS_TPB;
            if (j < left) vout[pos[k]] = sv[j];
        }
    }
}

template <typename Source, typename V, typename Off>
int radix_pass(Source from, typename Source::Key* kdst, const V* vsrc, V* vdst, size_t n, unsigned shift, unsigned mask, unsigned flip,
               Off* hist, hipStream_t s) {
    typedef typename Source::Key K;
    const size_t ntiles = (n + RS_TILE - 1) / RS_TILE;
    constexpr size_t lds = radix_lds_bytes<K, V>();
    if (lds > 48 * 1024)      // with the static part more than the 64 KB a workgroup gets without asking
        GCN_HIP_TRY(hipFuncSetAttribute((const void*)k_radix_scatter<Source, V, Off>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((k_radix_tile_hist<Source, Off>), dim3((unsigned)ntiles), dim3(P_TPB), 0, s, from, n, shift, mask, flip, ntiles, hist);
    GCN_LAUNCH_CHECK();
    GCN_TRY(exclusive_scan<Off>(hist, hist, ntiles * RS_RADIX, s));
    hipLaunchKernelGGL((k_radix_scatter<Source, V, Off>), dim3((unsigned)ntiles), dim3(RS_TPB), lds, s, from, kdst, vsrc,
                       vdst, n, shift, mask, flip, ntiles, (const Off*)hist);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

template <typename Source, typename V, typename Off>
int radix_passes(Source from, typename Source::Key* kout, const V* vin, V* vout, size_t n, const unsigned* shifts, const unsigned* masks,
                 int npass, bool descending, hipStream_t s) {
    typedef typename Source::Key K;
    constexpr bool HAS_V = !std::is_same<V, NoValue>::value;
    const size_t ntiles = (n + RS_TILE - 1) / RS_TILE;
    Scratch hist, tk, tv;
    GCN_TRY(hist.alloc(ntiles * RS_RADIX * sizeof(Off)));
    if (npass >= 2) {
        GCN_TRY(tk.alloc(n * sizeof(K)));
        if (HAS_V) GCN_TRY(tv.alloc(n * sizeof(V)));
    }
    const K* ksrc = nullptr;
    const V* vsrc = vin;
    for (int p = 0; p < npass; ++p) {
        const bool to_out = ((npass - 1 - p) % 2) == 0;      // the last pass lands in the caller's output
        K* kdst = to_out ? kout : tk.as<K>();
        V* vdst = to_out ? vout : tv.as<V>();
        const unsigned flip = descending ? masks[p] : 0u;
        if (p == 0) GCN_TRY((radix_pass<Source, V, Off>(from, kdst, vsrc, vdst, n, shifts[p], masks[p], flip, hist.as<Off>(), s)));
        else GCN_TRY((radix_pass<KeyArray<K>, V, Off>(KeyArray<K>{ksrc}, kdst, vsrc, vdst, n, shifts[p], masks[p], flip, hist.as<Off>(), s)));
        ksrc = kdst;
        vsrc = vdst;
    }
    return GCN_OK;
}

// The passes over the bits [0, end_bit).
inline int radix_digits(unsigned end_bit, unsigned* shifts, unsigned* masks) {
    int npass = 0;
    for (unsigned lo = 0; lo < end_bit; lo += 8) {
        shifts[npass] = lo;
        masks[npass] = (1u << (end_bit - lo < 8 ? end_bit - lo : 8)) - 1u;
        ++npass;
    }
    return npass;
}

// Ascending sort of n keys that `from` computes (twice each), by their bits [0, end_bit), at least one of them.
template <typename Source>
int radix_sort_from(Source from, typename Source::Key* kout, size_t n, unsigned end_bit, hipStream_t s) {
    typedef typename Source::Key K;
    if (n == 0) return GCN_OK;
    if ((n + RS_TILE - 1) / RS_TILE >= (1ull << 31)) return fail(GCN_ERR_RANGE, "radix_sort: %zu keys are too many", n);
    unsigned shifts[sizeof(K)], masks[sizeof(K)];
    const int npass = radix_digits(end_bit > 8 * sizeof(K) ? 8 * sizeof(K) : end_bit, shifts, masks);
    return radix_passes<Source, NoValue, unsigned long long>(from, kout, nullptr, nullptr, n, shifts, masks, npass, false, s);
}

// Stable sort of n keys by their bits [0, end_bit), ascending or descending; the payload (if V is
// not NoValue) moves with its key.  The inputs are left as they were; outputs must not overlap them.
// Digit positions at which every key holds the same byte are skipped.
// probe == false: every digit position is taken to vary (the caller packed its keys), which saves a pass over them and a
// wait for the stream.
template <typename K, typename V>
int radix_sort(const K* kin, K* kout, const V* vin, V* vout, size_t n, unsigned end_bit, bool descending, hipStream_t s,
               bool probe = true) {
    constexpr bool HAS_V = !std::is_same<V, NoValue>::value;
    constexpr int NB = sizeof(K);
    if (n == 0) return GCN_OK;
    if (end_bit > 8 * NB) end_bit = 8 * NB;
    const size_t ntiles = (n + RS_TILE - 1) / RS_TILE;
    if (ntiles >= (1ull << 31)) return fail(GCN_ERR_RANGE, "radix_sort: %zu keys are too many", n);
    unsigned shifts[NB], masks[NB];
    int npass = 0;
    if (!probe) {
        npass = radix_digits(end_bit, shifts, masks);
    } else {
        Scratch bh;
        GCN_TRY(bh.alloc(NB * RS_RADIX * 8));
        GCN_HIP_TRY(hipMemsetAsync(bh.p, 0, NB * RS_RADIX * 8, s));
        hipLaunchKernelGGL(k_radix_byte_hist<K>, dim3((unsigned)ntiles), dim3(P_TPB), 0, s, kin, n,
                           bh.as<unsigned long long>());
        GCN_LAUNCH_CHECK();
        unsigned long long h[NB * RS_RADIX];
        GCN_HIP_TRY(hipMemcpyAsync(h, bh.p, sizeof(h), hipMemcpyDeviceToHost, s));
        GCN_HIP_TRY(hipStreamSynchronize(s));
        for (int p = 0; p * 8 < (int)end_bit; ++p) {
            const unsigned width = end_bit - 8 * p < 8 ? end_bit - 8 * p : 8;
            const unsigned mask = (1u << width) - 1u;
            // bins of the masked digit: fold the byte histogram
            bool trivial = false;
            for (unsigned d = 0; d <= mask && !trivial; ++d) {
                unsigned long long c = 0;
                for (unsigned hi = d; hi < RS_RADIX; hi += mask + 1) c += h[p * RS_RADIX + hi];
                trivial = (c == n);
            }
            if (trivial) continue;
            shifts[npass] = 8 * p;
            masks[npass] = mask;
            ++npass;
        }
    }
    if (npass == 0) {
        GCN_HIP_TRY(hipMemcpyAsync(kout, kin, n * sizeof(K), hipMemcpyDeviceToDevice, s));
        if (HAS_V) GCN_HIP_TRY(hipMemcpyAsync((void*)vout, (const void*)vin, n * sizeof(V), hipMemcpyDeviceToDevice, s));
        return GCN_OK;
    }
    // positions are 64-bit whatever n is (their table is 1/32 of the keys' size): one code path at every size
    return radix_passes<KeyArray<K>, V, unsigned long long>(KeyArray<K>{kin}, kout, vin, vout, n, shifts, masks, npass, descending, s);
}

template <typename K> int sort_keys(const K* in, K* out, size_t n, unsigned end_bit, hipStream_t s) {
    return radix_sort<K, NoValue>(in, out, (const NoValue*)nullptr, (NoValue*)nullptr, n, end_bit, false, s);
}
template <typename K, typename V>
int sort_pairs(const K* kin, K* kout, const V* vin, V* vout, size_t n, unsigned end_bit, hipStream_t s) {
    return radix_sort<K, V>(kin, kout, vin, vout, n, end_bit, false, s);
}
template <typename K, typename V>
int sort_pairs_descending(const K* kin, K* kout, const V* vin, V* vout, size_t n, unsigned end_bit, hipStream_t s) {
    return radix_sort<K, V>(kin, kout, vin, vout, n, end_bit, true, s);
}

}  // namespace prims
}  // namespace gcn
