// Pairs of vertices -> distinct entries in row-major order, ascending columns: the sort of graph construction for matrices whose
// rows fall into buckets that a compute unit sorts in its LDS.
//
// One pass cuts the entries into buckets of 2^shift consecutive rows (a key inside a bucket fits 32 bits: row in the bucket, then
// column), a workgroup sorts a bucket in LDS and drops the repeated keys, and one last pass writes columns and row pointers.  A
// radix sort of the 8-byte keys (prims.h), which takes over where this does not fit, reads and writes them once per 8 bits and
// once more to drop the repeated ones.  16.8 M pairs of 1 M vertices, R-MAT (34.6 M keys): 1.35 ms that way; here counting 63 us,
// scatter 132, sort 288, columns and row pointers 84 (100 with the schedule's words).  Whole constructions, symmetrised: uniform
// 20 M pairs of 100 K vertices 2.11 -> 1.01 ms, 14 M of 3.9 M 2.17 -> 1.20; R-MAT 38 M of 1 M 3.98 -> 2.18; 100 K pairs of 10 K
// 0.31 -> 0.23.
// It fits up to 4096 buckets, of 2^(32 - bits of a column) rows at the most: 4,194,304 vertices and 83 M keys.  Larger graphs take the
// radix sort from the start.  Entries that lie in a few buckets are refused after the counting; that and the kernels behind it,
// which then do nothing, cost such constructions 30 to 100 us (pairs of one vertex: 32 K 286 -> 310 us, 400 K 373 -> 438, 8 M 835 -> 932,
// 16.8 M 1689 -> 1774; 2 M power-law pairs of 700 vertices 344 -> 403).
#pragma once
#include <type_traits>

#include "common.h"

namespace gcn {
namespace rowsort {

constexpr int THREADS = 1024, WAVES = THREADS / 64;
constexpr int MAX_BUCKETS = 4096;
constexpr unsigned MAX_SHIFT = 11;                 // rows of a bucket: up to 2048
constexpr int ITEMS = 8;                           // pairs of a thread in a tile
constexpr int TILE_KEYS = 2 * ITEMS * THREADS;
constexpr int KEYS = 24;                           // keys of a thread when a bucket is sorted
constexpr uint32_t CAP = KEYS * THREADS;           // keys that are sorted together
constexpr uint32_t PIECE = CAP / 6 * 5;            // larger buckets are cut into pieces of about this many keys
constexpr unsigned BIN_BITS = 12;                  // of the histograms that say where
constexpr int BINS = 1 << BIN_BITS;
constexpr int SHARES = 256;                        // workgroups that count and scatter
// Keys that the pieces of cut buckets read, of all keys: with more the matrix is refused.  With 2 8 M power-law pairs of 100 K vertices were
// refused (982 us, now 834; 943 by keys), with 8 2 M of 700 were not (536; refused 398).
constexpr uint64_t MOST_AGAIN = 4;

// The items that make keys: the pairs, then the diagonal.  A pair of equal ends makes none: with self loops the diagonal's key is
// there anyway.  *bad is set where an id is outside [0, n); such a pair makes no key either.
struct Items {
    const int32_t* src;
    const int32_t* dst;
    int64_t m, n, items;
    bool symmetrise;
    unsigned cbits, shift;
    __device__ void ends(int64_t i, uint32_t& u, uint32_t& v) const {
        if (i < m) { u = (uint32_t)src[i]; v = (uint32_t)dst[i]; }
        else u = v = (uint32_t)(i - m);
    }
    // how many keys: the first has row u, the second row v
    __device__ int count(int64_t i, uint32_t u, uint32_t v, bool& wrong) const {
        if (i >= m) return 1;
        if ((int64_t)u >= n || (int64_t)v >= n) { wrong = true; return 0; }
        if (u == v) return 0;
        return symmetrise ? 2 : 1;
    }
    __device__ uint32_t bucket(uint32_t row) const { return row >> shift; }
    __device__ uint32_t key(uint32_t row, uint32_t col) const { return (row & ((1u << shift) - 1u)) << cbits | col; }
};

// A bucket's keys, or one of the pieces of a large one.
struct Task { uint32_t bucket, part, parts, first, size; };    // first, size: the bucket's keys
// What is known behind the task table: refused says that the buckets are too uneven for this sort.
struct Info { uint32_t tasks, crowded; int32_t refused, bad; int64_t kept; };

template <typename T>
__device__ inline T wave_sum_up(T v) {                          // inclusive
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T u = (T)__shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}
// Exclusive prefix of v over the workgroup.  part: WAVES elements of LDS, free again when the call ends.
template <typename T>
__device__ inline T wg_exclusive(T v, T* part, T& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const T inc = wave_sum_up(v);
    if (lane == 63) part[w] = inc;
    __syncthreads();
    T base = 0, all = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        const T p = part[i];
        if (i < w) base += p;
        all += p;
    }
    __syncthreads();
    total = all;
    return base + inc - v;
}

// The lanes below this one that a ballot names.
__device__ inline uint32_t lanes_below(unsigned long long who) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
}

// How many keys of every bucket a workgroup's share of the items makes: table[share][bucket].  Bound by the LDS's counters (16.8 M pairs: 63
// us, 2.1 TB/s).
__global__ __launch_bounds__(THREADS) void k_part_count(Items p, int64_t share, uint32_t nb, uint32_t* __restrict__ table,
                                                    Info* __restrict__ info) {
    __shared__ uint32_t s_cnt[MAX_BUCKETS];
    for (uint32_t b = threadIdx.x; b < nb; b += THREADS) s_cnt[b] = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * share, end = first + share < p.items ? first + share : p.items;
    bool wrong = false;
    for (int64_t base = first; base < end; base += ITEMS * THREADS) {
        uint32_t u[ITEMS], v[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = base + k * THREADS + threadIdx.x;
            p.ends(i < end ? i : end - 1, u[k], v[k]);
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = base + k * THREADS + threadIdx.x;
            const int c = i < end ? p.count(i, u[k], v[k], wrong) : 0;
            if (c > 0) atomicAdd(&s_cnt[p.bucket(u[k])], 1u);
            if (c > 1) atomicAdd(&s_cnt[p.bucket(v[k])], 1u);
        }
    }
    if (wrong) info->bad = 1;
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nb; b += THREADS) table[(size_t)blockIdx.x * nb + b] = s_cnt[b];
}

// table[share][bucket] becomes the number of the bucket's keys in earlier shares, total[bucket] that of all of them.
__global__ __launch_bounds__(THREADS) void k_part_shares(uint32_t nb, uint32_t* __restrict__ table, uint32_t* __restrict__ total) {
    constexpr int PER = SHARES / WAVES;
    __shared__ uint32_t part[WAVES][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const uint32_t b = blockIdx.x * 64 + lane;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) c[k] = b < nb ? table[(size_t)(g * PER + k) * nb + b] : 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += c[k];
    part[g][lane] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int i = 0; i < g; ++i) run += part[i][lane];
    if (b >= nb) return;
    if (g == WAVES - 1) total[b] = run + sum;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        table[(size_t)(g * PER + k) * nb + b] = run;
        run += c[k];
    }
}

// Where the buckets begin, and the tasks, in ascending order of their keys and (`order`) with the pieces of large buckets first: one
// per bucket, more for those beyond CAP.  Every piece of such a bucket reads all of its keys three times, so matrices whose
// entries lie in a few buckets for the most part are refused (`most`: keys read that way).
__global__ __launch_bounds__(THREADS) void k_part_tasks(uint32_t nb, uint64_t most, const uint32_t* __restrict__ total, uint32_t* __restrict__ start,
                                                    Task* __restrict__ tasks, uint32_t* __restrict__ order, Info* __restrict__ info) {
    constexpr int PER = MAX_BUCKETS / THREADS;
    __shared__ uint32_t part[WAVES];
    __shared__ unsigned long long part64[WAVES];
    uint32_t size[PER], pieces[PER], keys = 0, count = 0, cut = 0;
    unsigned long long again = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint32_t b = threadIdx.x * PER + k;
        size[k] = b < nb ? total[b] : 0;
        pieces[k] = b < nb ? (size[k] > CAP ? (size[k] + PIECE - 1) / PIECE : 1) : 0;
        if (pieces[k] > 1) { again += (unsigned long long)pieces[k] * size[k]; cut += pieces[k]; }
        keys += size[k];
        count += pieces[k];
    }
    uint32_t all, all_tasks, all_cut;
    unsigned long long all_again;
    uint32_t at = wg_exclusive(keys, part, all), t = wg_exclusive(count, part, all_tasks);
    uint32_t c = wg_exclusive(cut, part, all_cut);
    wg_exclusive(again, part64, all_again);
    const bool refused = all_again > most;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint32_t b = threadIdx.x * PER + k;
        if (b >= nb) break;
        start[b] = at;
        for (uint32_t i = 0; i < (refused ? 0 : pieces[k]); ++i) {
            tasks[t + i] = Task{b, i, pieces[k], at, size[k]};
            order[pieces[k] > 1 ? c++ : all_cut + (t + i - c)] = t + i;        // (c: pieces of cut buckets before this task)
        }
        at += size[k];
        t += pieces[k];
    }
    if (threadIdx.x == 0) {
        info->tasks = refused ? 0 : all_tasks;
        info->refused = refused;
    }
}

// Moves the keys to their buckets.  The order inside a bucket is whatever the counters give: the sort does not depend on it.  A tile's
// keys go through LDS, so that those of one bucket are written as one run (eight keys with 2048 buckets: 132 us for 34.6 M; four with 4096: 172).
__global__ __launch_bounds__(THREADS) void k_part_scatter(Items p, int64_t share, uint32_t nb, const uint32_t* __restrict__ start,
                                                      const uint32_t* __restrict__ table, const Info* __restrict__ info,
                                                      uint32_t* __restrict__ out) {
    constexpr int PER = MAX_BUCKETS / THREADS;
    extern __shared__ uint32_t s_tile[];
    uint32_t* const s_key = s_tile;                             // [TILE_KEYS]
    uint32_t* const s_first = s_key + TILE_KEYS;                // [MAX_BUCKETS] keys of the tile's bucket; then its first place in the tile
    uint32_t* const s_move = s_first + MAX_BUCKETS;             // [MAX_BUCKETS] output position less place in the tile
    uint16_t* const s_bucket = (uint16_t*)(s_move + MAX_BUCKETS);       // [TILE_KEYS]
    __shared__ uint32_t part[WAVES];
    if (info->refused) return;
    uint32_t cursor[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint32_t b = threadIdx.x * PER + k;
        cursor[k] = b < nb ? start[b] + table[(size_t)blockIdx.x * nb + b] : 0;
    }
    const int64_t first = (int64_t)blockIdx.x * share, end = first + share < p.items ? first + share : p.items;
    bool wrong = false;
    for (int64_t base = first; base < end; base += ITEMS * THREADS) {
        uint32_t u[ITEMS], v[ITEMS], r[2 * ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = base + k * THREADS + threadIdx.x;
            p.ends(i < end ? i : end - 1, u[k], v[k]);
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) s_first[threadIdx.x * PER + k] = 0;
        __syncthreads();
        uint32_t two = 0, one = 0;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int64_t i = base + k * THREADS + threadIdx.x;
            const int c = i < end ? p.count(i, u[k], v[k], wrong) : 0;
            if (c > 0) { one |= 1u << k; r[2 * k] = atomicAdd(&s_first[p.bucket(u[k])], 1u); }
            if (c > 1) { two |= 1u << k; r[2 * k + 1] = atomicAdd(&s_first[p.bucket(v[k])], 1u); }
        }
        __syncthreads();
        uint32_t cnt[PER], sum = 0, all;
#pragma unroll
        for (int k = 0; k < PER; ++k) { cnt[k] = s_first[threadIdx.x * PER + k]; sum += cnt[k]; }
        uint32_t at = wg_exclusive(sum, part, all);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            s_first[threadIdx.x * PER + k] = at;
            s_move[threadIdx.x * PER + k] = cursor[k] - at;
            cursor[k] += cnt[k];
            at += cnt[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (one >> k & 1u) {
                const uint32_t b = p.bucket(u[k]), j = s_first[b] + r[2 * k];
                s_key[j] = p.key(u[k], v[k]);
                s_bucket[j] = (uint16_t)b;
            }
            if (two >> k & 1u) {
                const uint32_t b = p.bucket(v[k]), j = s_first[b] + r[2 * k + 1];
                s_key[j] = p.key(v[k], u[k]);
                s_bucket[j] = (uint16_t)b;
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < 2 * ITEMS; ++k) {
            const uint32_t j = k * THREADS + threadIdx.x;
            if (j < all) out[s_move[s_bucket[j]] + j] = s_key[j];
        }
        __syncthreads();
    }
}
constexpr size_t SCATTER_LDS = (size_t)TILE_KEYS * 6 + (size_t)MAX_BUCKETS * 8;

// ---- the sort of a task -------------------------------------------------------------------------------------------------------
constexpr uint32_t WINDOW = 15, MOST_IN_WINDOW = 8, MOST_BY_RANK = 512, MOST_RANKED = 64;
struct SortArgs {
    unsigned cbits, shift;
    const Task* tasks;
    const uint32_t* order;
    const uint32_t* in;
    uint32_t* out;
    uint32_t* at_of;             // [task] where its distinct keys begin in `out`
    uint32_t* count_of;          // [task] and how many there are
    uint32_t* crowded;           // tasks that k_part_sort leaves to k_part_sort_digits
    Info* info;
};
struct SortLds {                 // of a workgroup, beside s_key [CAP + 2 WINDOW], s_slot [SLOTS] and s_row [rows + 1]
    uint32_t part[WAVES], bound[2], below[2], bin[2], count, crowded, large, ranked, low_col, high_col, inverse;
    uint16_t large_at[CAP / (MOST_IN_WINDOW + 1) + 1];     // places of more keys than a window takes
};

constexpr uint32_t SLOTS = CAP / 2 + 1;                         // words of s_slot
static_assert(SLOTS >= 2 * BINS && CAP >= 4 * BINS, "histograms");
inline size_t sort_lds(unsigned shift) { return ((size_t)CAP + 2 * WINDOW + SLOTS + (1u << shift) + 1) * 4; }

// The keys of a whole bucket: key[k] is the one at k THREADS + thread.
__device__ __forceinline__ void load_bucket(const SortArgs& a, const Task& t, uint32_t (&key)[KEYS]) {
    const uint32_t* const keys = a.in + t.first;
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
        const uint32_t j = k * THREADS + threadIdx.x;
        key[k] = j < t.size ? keys[j] : 0;
    }
}

// Those of a piece: returns how many there are, up to CAP, and where they begin.
__device__ __forceinline__ uint32_t fetch_piece(const SortArgs& a, uint32_t id, const Task& t, uint32_t* s_key, uint32_t* s_slot, SortLds& L,
                                                uint32_t (&key)[KEYS], uint32_t& from) {
    const int lane = threadIdx.x & 63;
    const uint32_t* const keys = a.in + t.first;
    const uint32_t size = t.size;
    const unsigned kbits = a.shift + a.cbits;
    from = t.first;
    // The keys between two bounds, which every piece works out for itself: the smallest prefix of up to two bin_bits with at least
    // part / parts of the keys below it.
    const unsigned d1 = kbits < BIN_BITS ? kbits : BIN_BITS, d2 = kbits - d1 < BIN_BITS ? kbits - d1 : BIN_BITS;
    const unsigned sh1 = kbits - d1, sh2 = sh1 - d2;
    uint32_t want[2];
    want[0] = (uint32_t)((uint64_t)size * t.part / t.parts);
    want[1] = (uint32_t)((uint64_t)size * (t.part + 1) / t.parts);
    // (the keys of one long row share a few bins: copies of the first histogram, so that fewer lanes add to one counter)
    constexpr int COPIES = 4;
    uint32_t* const h1 = s_key;                                 // [BINS][COPIES]
    uint32_t* const h2 = s_slot;                                // [2][BINS]
    for (int i = threadIdx.x; i < COPIES * BINS; i += THREADS) h1[i] = 0;
    for (int i = threadIdx.x; i < 2 * BINS; i += THREADS) h2[i] = 0;
    if (threadIdx.x < 2) { L.bound[threadIdx.x] = 0; L.below[threadIdx.x] = 0; L.bin[threadIdx.x] = ~0u; }
    if (threadIdx.x == 0) L.count = 0;
    __syncthreads();
    constexpr int AT_ONCE = 16;
    for (uint32_t j0 = threadIdx.x; j0 < size; j0 += AT_ONCE * THREADS) {
        uint32_t x[AT_ONCE];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) x[e] = keys[j0 + e * THREADS < size ? j0 + e * THREADS : size - 1];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e)
            if (j0 + e * THREADS < size) atomicAdd(&h1[(x[e] >> sh1) * COPIES + lane % COPIES], 1u);
    }
    __syncthreads();
    constexpr int PER = BINS / THREADS;
    uint32_t c[PER], sum = 0, all;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const uint4 four = reinterpret_cast<const uint4*>(h1)[threadIdx.x * PER + k];
        c[k] = four.x + four.y + four.z + four.w;
        sum += c[k];
    }
    uint32_t run = wg_exclusive(sum, L.part, all);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (run < want[e] && want[e] <= run + c[k]) { L.bin[e] = threadIdx.x * PER + k; L.below[e] = run; }
        run += c[k];
    }
    __syncthreads();
    const uint32_t b0 = L.bin[0], b1 = L.bin[1];                // ~0: nothing is below the bound
    const uint32_t below0 = L.below[0], below1 = L.below[1];
    for (uint32_t j0 = threadIdx.x; j0 < size; j0 += AT_ONCE * THREADS) {
        uint32_t x[AT_ONCE];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) x[e] = keys[j0 + e * THREADS < size ? j0 + e * THREADS : size - 1];
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) {
            if (j0 + e * THREADS >= size) break;
            const uint32_t bin = x[e] >> sh1, sub = x[e] >> sh2 & ((1u << d2) - 1u);
            if (bin == b0) atomicAdd(&h2[sub], 1u);
            if (bin == b1) atomicAdd(&h2[BINS + sub], 1u);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t bin = e ? b1 : b0;
        sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) { c[k] = h2[e * BINS + threadIdx.x * PER + k]; sum += c[k]; }
        run = (e ? below1 : below0) + wg_exclusive(sum, L.part, all);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (bin != ~0u && run < want[e] && want[e] <= run + c[k]) {
                L.bound[e] = (bin << d2) + threadIdx.x * PER + k + 1;
                L.below[e] = run + c[k];
            }
            run += c[k];
        }
    }
    __syncthreads();
    const uint32_t low = L.bound[0], high = L.bound[1];
    from += L.below[0];
    // More keys than are sorted together: the last prefix has thousands, nearly all of them repeated (sh2 is 8 at the most).  A bit for each of
    // its keys says which are there, and that is all that is wanted of them; the other prefixes hold a PIECE at the most.
    const bool crowded = L.below[1] - L.below[0] > CAP;         // (the same for all)
    uint32_t* const s_bit = s_slot;
    static_assert(PIECE + (1 << (32 - 2 * BIN_BITS)) <= CAP, "a piece and the keys of a prefix");
    auto collect = [&](auto bits) {                             // (a loop of its own: the test of every key took 16 us more for 34.6 M)
        for (uint32_t j0 = 0; j0 < size; j0 += AT_ONCE * THREADS) {
            uint32_t x[AT_ONCE];
#pragma unroll
            for (int e = 0; e < AT_ONCE; ++e) {
                const uint32_t j = j0 + e * THREADS + threadIdx.x;
                x[e] = keys[j < size ? j : size - 1];
            }
            unsigned long long who[AT_ONCE];
            uint32_t found = 0;
#pragma unroll
            for (int e = 0; e < AT_ONCE; ++e) {
                const uint32_t prefix = x[e] >> sh2;
                bool mine = j0 + e * THREADS + threadIdx.x < size && prefix >= low && prefix < high;
                if (decltype(bits)::value && mine && prefix == high - 1) {
                    const uint32_t bit = x[e] & ((1u << sh2) - 1u);
                    if (!(s_bit[bit / 32] >> bit % 32 & 1u)) atomicOr(&s_bit[bit / 32], 1u << bit % 32);
                    mine = false;
                }
                who[e] = __ballot(mine);
                found += (uint32_t)__popcll(who[e]);
            }
            uint32_t base = 0;
            if (lane == 0 && found) base = atomicAdd(&L.count, found);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
            for (int e = 0; e < AT_ONCE; ++e) {
                if (who[e] >> lane & 1ull) s_key[base + lanes_below(who[e])] = x[e];
                base += (uint32_t)__popcll(who[e]);
            }
        }
        __syncthreads();
    };
    if (crowded) {
        if (threadIdx.x < (1u << (32 - 2 * BIN_BITS)) / 32) s_bit[threadIdx.x] = 0;
        __syncthreads();
        collect(std::true_type());
        if (threadIdx.x < 1u << sh2 && s_bit[threadIdx.x / 32] >> threadIdx.x % 32 & 1u)
            s_key[atomicAdd(&L.count, 1u)] = (high - 1) << sh2 | threadIdx.x;
        __syncthreads();
    } else {
        collect(std::false_type());
    }
    const uint32_t here = L.count;
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
        const uint32_t j = k * THREADS + threadIdx.x;
        key[k] = j < here ? s_key[j] : 0;
    }
    __syncthreads();
    return here;
}

// The distinct ones of the sorted keys in s_key, to where the task's keys began: a lane takes consecutive keys, an odd number of them for the
// banks, they move together in LDS and leave from there.
__device__ __forceinline__ void store_distinct(const SortArgs& a, uint32_t id, uint32_t here, uint32_t from, uint32_t* s_key, SortLds& L) {
    const uint32_t per = (here + THREADS - 1) / THREADS | 1u, j0 = threadIdx.x * per;
    static_assert(KEYS % 2 == 0, "one more where all are there");
    uint32_t x[KEYS + 1], own = 0, all;                         // own: a bit per key that stays
    uint32_t last = j0 > 0 && j0 < here ? s_key[j0 - 1] : 0;
#pragma unroll
    for (uint32_t e = 0; e < KEYS + 1; ++e) {
        if (e >= per) break;
        if (j0 + e < here) {
            x[e] = s_key[j0 + e];
            own |= x[e] != last || j0 + e == 0 ? 1u << e : 0u;
            last = x[e];
        }
    }
    uint32_t to = wg_exclusive((uint32_t)__popc(own), L.part, all);
#pragma unroll
    for (uint32_t e = 0; e < KEYS + 1; ++e) {
        if (e >= per) break;
        if (own >> e & 1u) s_key[to++] = x[e];
    }
    if (threadIdx.x == 0) { a.at_of[id] = from; a.count_of[id] = all; }
    __syncthreads();
#pragma unroll 4
    for (uint32_t j = threadIdx.x; j < all; j += THREADS) a.out[from + j] = s_key[j];
}

// Sorts the keys of a task in LDS and writes the distinct ones.
//
// A row's keys are spread over as many places as it has keys, in proportion to the column's position in the task's range of columns, and
// counted place by place: keys in random order of their columns leave one or two in a place, seldom more than eight.  What is out of
// order then is so only inside a place, and windows of 15 keys, which a lane sorts in registers, put it in order: once from 0 on
// and once from 7 on, so that every place of up to eight keys lies in one of them.  The work of a key is a handful of LDS operations,
// where a sort by digits ranks it by eight ballots per digit.  Larger places (columns that lie close together, pairs that repeat) are put
// in order by a wavefront each: up to 64 keys by their ranks, more where no more than 64 of them are distinct, or where few places have
// so many (up to MOST_BY_RANK).  Beyond that the task is left to k_part_sort_digits.
__global__ __launch_bounds__(THREADS) void k_part_sort(SortArgs a) {
    extern __shared__ uint32_t s_mem[];
    uint32_t* const s_key = s_mem;                              // [CAP], and a window's overhang
    uint32_t* const s_slot = s_key + CAP + 2 * WINDOW;          // [SLOTS] two 16-bit counters each; histograms before
    uint32_t* const s_row = s_slot + SLOTS;                     // [rows + 1]
    __shared__ SortLds L;
    const uint32_t rows = 1u << a.shift, cbits = a.cbits, id = a.order[blockIdx.x];     // (there are as many as workgroups)
    if (blockIdx.x >= a.info->tasks) return;
    const Task t = a.tasks[id];
    uint32_t key[KEYS], here = t.size, from = t.first, all;
    if (threadIdx.x == 0) { L.crowded = L.large = L.ranked = L.high_col = 0; L.low_col = ~0u; }
    if (t.parts > 1) here = fetch_piece(a, id, t, s_key, s_slot, L, key, from);
    else load_bucket(a, t, key);

    // ---- keys of every row, and the range of the columns ----
    for (uint32_t i = threadIdx.x; i <= rows; i += THREADS) s_row[i] = 0;
    for (uint32_t i = threadIdx.x; i <= here / 2; i += THREADS) s_slot[i] = 0;
    __syncthreads();
    const uint32_t cmask = (1u << cbits) - 1u;
    uint32_t low = ~0u, high = 0;
#pragma unroll
    for (int k = 0; k < KEYS; ++k)
        if (k * THREADS + threadIdx.x < here) {
            const uint32_t c = key[k] & cmask;
            low = low < c ? low : c;
            high = high > c ? high : c;
            atomicAdd(&s_row[key[k] >> cbits], 1u);
        }
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t l = __shfl_xor(low, d, 64), h = __shfl_xor(high, d, 64);
        low = low < l ? low : l;
        high = high > h ? high : h;
    }
    if ((threadIdx.x & 63) == 0) { atomicMin(&L.low_col, low); atomicMax(&L.high_col, high); }
    __syncthreads();
    // (2^32 / columns of the range, at most; the product with one of them stays below 2^32)
    if (threadIdx.x == 0) L.inverse = L.high_col > L.low_col ? 0xffffffffu / (L.high_col - L.low_col + 1) : 0;
    {
        constexpr int PER = (1 << MAX_SHIFT) / THREADS;
        uint32_t c[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = threadIdx.x * PER + k;
            c[k] = i < rows ? s_row[i] : 0;
            sum += c[k];
        }
        uint32_t run = wg_exclusive(sum, L.part, all);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = threadIdx.x * PER + k;
            if (i < rows) s_row[i] = run;
            run += c[k];
        }
        if (threadIdx.x == 0) s_row[rows] = here;
    }
    __syncthreads();

    // ---- places: row's first + column / range * keys of the row ----
    const uint32_t col0 = L.low_col, inverse = L.inverse;
    uint32_t place[KEYS];                                       // place, and rank in it from bit 16 up
    constexpr int AT_ONCE = 4;
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
        if (k % AT_ONCE == 0) __builtin_amdgcn_sched_barrier(0);
        place[k] = 0;
        if (k * THREADS + threadIdx.x < here) {
            const uint32_t r = key[k] >> cbits, r0 = s_row[r], len = s_row[r + 1] - r0;
            const uint32_t q = r0 + __umulhi(((key[k] & cmask) - col0) * inverse, len);
            const uint32_t old = atomicAdd(&s_slot[q >> 1], q & 1u ? 1u << 16 : 1u);
            const uint32_t rank = q & 1u ? old >> 16 : old & 0xffffu;
            if (rank == MOST_IN_WINDOW) L.large_at[atomicAdd(&L.large, 1u)] = (uint16_t)q;
            place[k] = q | rank << 16;
        }
    }
    __syncthreads();
    uint16_t* const first = (uint16_t*)s_slot;                  // [here + 1]: counts, then first places
    {
        const uint32_t words = here / 2 + 1, per = ((words + THREADS - 1) / THREADS) | 1u;      // an odd stride over the banks
        const uint32_t w0 = threadIdx.x * per, w1 = w0 + per < words ? w0 + per : words;
        uint32_t sum = 0;
        for (uint32_t i = w0; i < w1; ++i) { const uint32_t x = s_slot[i]; sum += (x & 0xffffu) + (x >> 16); }
        uint32_t run = wg_exclusive(sum, L.part, all);
        for (uint32_t i = w0; i < w1; ++i) {
            const uint32_t x = s_slot[i];
            s_slot[i] = run | (run + (x & 0xffffu)) << 16;
            run += (x & 0xffffu) + (x >> 16);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KEYS; ++k)
        if (k * THREADS + threadIdx.x < here) s_key[first[place[k] & 0xffffu] + (place[k] >> 16)] = key[k];
    if (threadIdx.x < 2 * WINDOW) s_key[here + threadIdx.x] = ~0u;      // (what windows take beyond the last key)
    __syncthreads();
    // the order inside a place
#pragma unroll 1
    for (uint32_t shifted = 0; shifted < 2; ++shifted) {
        for (uint32_t base = threadIdx.x * WINDOW + shifted * (WINDOW / 2); base < here; base += THREADS * WINDOW) {
            uint32_t x[16];
#pragma unroll
            for (uint32_t e = 0; e < 16; ++e) x[e] = e < WINDOW ? s_key[base + e] : ~0u;
            // Batcher's odd-even merge sort
#pragma unroll
            for (int p = 1; p < 16; p *= 2)
#pragma unroll
                for (int k = p; k >= 1; k /= 2)
#pragma unroll
                    for (int j = k % p; j + k < 16; j += 2 * k)
#pragma unroll
                        for (int i = 0; i < k; ++i)
                            if (j + i + k < 15 && (j + i) / (2 * p) == (j + i + k) / (2 * p)) {      // (the sixteenth is the largest)
                                const uint32_t u = x[j + i], v = x[j + i + k];
                                x[j + i] = u < v ? u : v;
                                x[j + i + k] = u < v ? v : u;
                            }
#pragma unroll
            for (uint32_t e = 0; e < WINDOW; ++e) s_key[base + e] = x[e];
        }
        __syncthreads();
    }
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t l = threadIdx.x >> 6; l < L.large && !L.crowded; l += WAVES) {
        const uint32_t f = first[L.large_at[l]], len = first[L.large_at[l] + 1] - f;
        uint32_t* const its = s_key + f;
        if (len <= 64) {                                        // a lane's rank: the keys below its own, and the equal ones before it
            const uint32_t x = its[lane < len ? lane : 0];
            uint32_t to = 0;
            for (uint32_t i = 0; i < len; ++i) {
                const uint32_t other = its[i];
                to += i < lane ? other <= x : other < x;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (lane < len) its[to] = x;
            continue;
        }
        // the distinct ones in ascending order, the i-th of them and how often it is there in lane i
        uint32_t value = 0, times = 0, found = 0, distinct = 0, from_on = 0;
        for (; found < len && distinct < 64; ++distinct) {
            uint32_t least = ~0u;
            for (uint32_t i = lane; i < len; i += 64) {
                const uint32_t x = its[i];
                least = x >= from_on && x < least ? x : least;
            }
            for (int d = 32; d >= 1; d >>= 1) {
                const uint32_t o = __shfl_xor(least, d, 64);
                least = least < o ? least : o;
            }
            uint32_t c = 0;
            for (uint32_t i = lane; i - lane < len; i += 64) c += (uint32_t)__popcll(__ballot(i < len && its[i] == least));
            if (lane == distinct) { value = least; times = c; }
            found += c;
            from_on = least + 1;
        }
        if (found < len) {                                      // by ranks, a few places of a task
            constexpr int PER = MOST_BY_RANK / 64;
            uint32_t few = 0;
            if (lane == 0) few = atomicAdd(&L.ranked, 1u);
            if (len > MOST_BY_RANK || (uint32_t)__builtin_amdgcn_readfirstlane((int)few) >= MOST_RANKED) {
                L.crowded = 1;
                break;
            }
            uint32_t x[PER], to[PER];
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                x[e] = its[e * 64 + lane < len ? e * 64 + lane : 0];
                to[e] = 0;
            }
            for (uint32_t i = 0; i < len; ++i) {
                const uint32_t other = its[i];
#pragma unroll
                for (int e = 0; e < PER; ++e) to[e] += i < e * 64 + lane ? other <= x[e] : other < x[e];
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (e * 64 + lane < len) its[to[e]] = x[e];
            continue;
        }
        uint32_t at = 0;
        for (uint32_t d = 0; d < distinct; ++d) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)value, (int)d), c = (uint32_t)__builtin_amdgcn_readlane((int)times, (int)d);
            for (uint32_t i = lane; i < c; i += 64) its[at + i] = x;
            at += c;
        }
    }
    __syncthreads();
    if (L.crowded) {
        if (threadIdx.x == 0) a.crowded[atomicAdd(&a.info->crowded, 1u)] = id;
        return;
    }
    store_distinct(a, id, here, from, s_key, L);
}

// The crowded tasks, by digits of 8 bits: each pass as k_radix_scatter's inside a tile, a wavefront owns 64 KEYS consecutive keys.
__global__ __launch_bounds__(THREADS) void k_part_sort_digits(SortArgs a) {
    extern __shared__ uint32_t s_mem[];
    uint32_t* const s_key = s_mem;                              // [CAP], and a window's overhang
    uint32_t* const s_slot = s_key + CAP + 2 * WINDOW;                       // [WAVES][256] counters; histograms before
    __shared__ SortLds L;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned kbits = a.shift + a.cbits;
    const uint32_t tasks = a.info->crowded;
    for (uint32_t at = blockIdx.x; at < tasks; at += gridDim.x) {
        const uint32_t id = a.crowded[at];
        const Task t = a.tasks[id];
        uint32_t key[KEYS], here = t.size, from = t.first, all;
        if (t.parts > 1) here = fetch_piece(a, id, t, s_key, s_slot, L, key, from);
        else load_bucket(a, t, key);
#pragma unroll
        for (int k = 0; k < KEYS; ++k)
            if (k * THREADS + threadIdx.x < here) s_key[k * THREADS + threadIdx.x] = key[k];
        const uint32_t mine0 = w * 64 * KEYS + lane;
        uint32_t* const cnt = s_slot + w * 256;                 // this wavefront's
#pragma unroll 1
        for (unsigned lo = 0; lo < kbits; lo += 8) {
            for (int i = threadIdx.x; i < WAVES * 256; i += THREADS) s_slot[i] = 0;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KEYS; ++k) {
                const bool valid = mine0 + 64 * k < here;
                key[k] = valid ? s_key[mine0 + 64 * k] : 0;
                if (valid) atomicAdd(&cnt[key[k] >> lo & 255u], 1u);
            }
            __syncthreads();
            uint32_t sum = 0;
            if (threadIdx.x < 256) {
#pragma unroll
                for (int i = 0; i < WAVES; ++i) {
                    const uint32_t c = s_slot[i * 256 + threadIdx.x];
                    s_slot[i * 256 + threadIdx.x] = sum;
                    sum += c;
                }
            }
            const uint32_t base = wg_exclusive(sum, L.part, all);
            if (threadIdx.x < 256) {
#pragma unroll
                for (int i = 0; i < WAVES; ++i) s_slot[i * 256 + threadIdx.x] += base;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KEYS; ++k) {
                const bool valid = mine0 + 64 * k < here;
                const uint32_t d = key[k] >> lo & 255u;
                unsigned long long peers = __ballot(valid);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const bool bit = d >> b & 1u;
                    const unsigned long long have = __ballot(valid && bit);
                    peers &= bit ? have : ~have;
                }
                const uint32_t before = lanes_below(peers);
                uint32_t to = 0;
                if (valid) to = cnt[d];
                // the wavefront's LDS operations complete in program order; the fences keep the compiler to it
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (valid && before == 0) cnt[d] = to + (uint32_t)__popcll(peers);
                if (valid) s_key[to + before] = key[k];
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
        }
        store_distinct(a, id, here, from, s_key, L);
        __syncthreads();
    }
}

// Where the entries of every task go: offset[task], from the numbers in count[task].
__global__ __launch_bounds__(THREADS) void k_part_offsets(const uint32_t* __restrict__ count, uint32_t* __restrict__ offset, Info* __restrict__ info) {
    __shared__ uint32_t part[WAVES];
    const uint32_t tasks = info->tasks;                         // (none where the matrix is refused)
    uint32_t run = 0;
    for (uint32_t base = 0; base < tasks; base += THREADS) {
        const uint32_t t = base + threadIdx.x;
        uint32_t all;
        const uint32_t before = wg_exclusive(t < tasks ? count[t] : 0u, part, all);
        if (t < tasks) offset[t] = run + before;
        run += all;
    }
    if (threadIdx.x == 0) info->kept = run;
}

// Columns and row pointers of a task's entries: an entry opens the rows after that of the entry before it, the last piece of a bucket
// closes the bucket's rows.  Also the schedule's flag words (a bit per entry that starts a row, zeroed before) and the row of every 32nd
// entry: a wavefront takes 64 entries from a multiple of 64 on, so that it owns two words, except for those at the ends of the task.
// (34 M entries: two passes over the row pointers and a bisection per 32 entries took 54 us, this kernel 100 with them and 84
// without.)  keys (or NULL): also row << cbits | column of every entry.
__global__ __launch_bounds__(512) void k_part_emit(int64_t n, uint32_t nb, unsigned cbits, unsigned shift, const Task* __restrict__ tasks,
                                                   const uint32_t* __restrict__ at_of, const uint32_t* __restrict__ count_of,
                                                   const uint32_t* __restrict__ offset, const uint32_t* __restrict__ in,
                                                   int64_t* __restrict__ rowptr, int32_t* __restrict__ colidx, uint64_t* __restrict__ keys,
                                                   uint32_t* __restrict__ flags, int32_t* __restrict__ sub_row) {
    static_assert(SUB == 32, "two words per wavefront");
    const Task t = tasks[blockIdx.x];
    const uint32_t count = count_of[blockIdx.x], off = offset[blockIdx.x], cmask = (1u << cbits) - 1u;
    const uint32_t* const from = in + at_of[blockIdx.x];
    const int64_t row0 = (int64_t)t.bucket << shift;
    const int lane = threadIdx.x & 63;
    int32_t before = -1;                                        // row in the bucket of the entry before the first
    for (uint32_t p = t.part, i = blockIdx.x; p > 0 && before < 0; --p) {
        --i;
        if (count_of[i] > 0) before = (int32_t)(in[at_of[i] + count_of[i] - 1] >> cbits);
    }
    const int32_t lead = (int32_t)(off & 63u);                  // entries of the first 64 that are another task's
    for (int32_t j0 = (int32_t)(threadIdx.x & ~63u) - lead; j0 < (int32_t)count; j0 += 512) {
        const int32_t j = j0 + lane;
        const bool here = j >= 0 && j < (int32_t)count;
        const uint32_t at = off + (uint32_t)j, key = here ? from[j] : 0;
        const int32_t r = (int32_t)(key >> cbits), last = here && j > 0 ? (int32_t)(from[j - 1] >> cbits) : before;
        if (here) {
            for (int32_t q = last + 1; q <= r; ++q) rowptr[row0 + q] = at;
            colidx[at] = (int32_t)(key & cmask);
            if (keys) keys[at] = (uint64_t)(row0 + r) << cbits | (key & cmask);
            if ((lane & 31) == 0) sub_row[at / SUB] = (int32_t)(row0 + r);
        }
        const unsigned long long starts = __ballot(here && r > last);
        if ((lane & 31) == 0 && j < (int32_t)count && j + 31 >= 0) {
            const uint32_t word = (uint32_t)(starts >> lane);
            uint32_t* const f = flags + (int64_t)(off + (int64_t)j) / SUB;
            if (j >= 0 && j + 32 <= (int32_t)count) *f = word;
            else atomicOr(f, word);
        }
    }
    if (t.part + 1 < t.parts) return;
    const int64_t end = t.bucket + 1 < nb ? row0 + (1ll << shift) : n + 1;
    const int32_t last = count > 0 ? (int32_t)(from[count - 1] >> cbits) : before;
    for (int64_t q = row0 + last + 1 + threadIdx.x; q < end; q += 512) rowptr[q] = off + count;
}

// Whether this sort takes n rows and `cap` keys, and the rows of a bucket.  Buckets of four fifths of what is sorted together leave room
// for uneven ones; at least 256 of them where there are rows enough, so that every compute unit has one.
inline bool takes(int64_t n, int64_t cap, unsigned cbits, unsigned* shift, uint32_t* nb) {
    constexpr int64_t ROOM = CAP / 100 * 83;
    auto buckets = [&](unsigned b) { return (n + (1ll << b) - 1) >> b; };
    unsigned s = 32 - cbits < MAX_SHIFT ? 32 - cbits : MAX_SHIFT;
    while (s > 0 && (buckets(s) < SHARES || cap / buckets(s) > ROOM)) --s;
    if (cap <= 0 || buckets(s) > MAX_BUCKETS || cap / buckets(s) > ROOM) return false;
    *shift = s;
    *nb = (uint32_t)buckets(s);
    return true;
}

}  // namespace rowsort
}  // namespace gcn
