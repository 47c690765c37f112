// fp32 MFMA kernels for the dense products around the SpMM (v_mfma_f32_16x16x4_f32; full fp32
// multiply-add, so the 1e-4 bound against the double oracle holds):
//   k_gemm_tall   C[M x N] = A[M x K] op(B)            M = n (millions), K and N small: H W of
//                 "Forward Propagation", S W^T of Equation 2.  Streams A once from HBM; op(B) sits
//                 in LDS; one wavefront owns a 16-row strip and up to four 16-column tiles.
//   k_gemm_tn     C[M x N] = A[K x M]^T B[K x N]        K = n: the weight gradient of Equation 3.
//                 Split over K across workgroups; partial results are reduced in a fixed order.
// At hidden width 16 both are bandwidth-bound (8 flops per byte of A): the matrix cores keep the
// arithmetic off the critical path.
//
// Operand layout of the 16x16x4 instruction (64 lanes): lane l supplies A[i = l%16][k = l/16] and
// B[k = l/16][j = l%16], and holds D[i = 4*(l/16) + v][j = l%16] in element v of its accumulator.
#include <algorithm>

#include "common.h"
#include "launch_rules.h"
#include "sum_parts.h"

namespace gcn {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// 16-byte load of data that is read once: the non-temporal hint keeps the stream from displacing what other
// wavefronts still need in the caches.  Measured on 14 M rows: +10 % on the A^T B kernel when every row of A is
// whole 128-byte lines (256 floats: 2.67 -> 2.39 ms, 128 floats: 1.62 -> 1.42 ms), +2 % on the strip kernel; a loss
// where neighbouring wavefronts share lines (A^T B at 300 floats per row: 4.13 -> 4.22 ms), so the callers decide.
// The address need only be 4-byte aligned: the last columns of a padded row start anywhere.
typedef floatx4 floatx4u __attribute__((aligned(4)));
__device__ __forceinline__ float4 stream4(const float* p) {
    const floatx4 v = __builtin_nontemporal_load(reinterpret_cast<const floatx4u*>(p));
    return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float4 load4(const float* p) {
    const f4u v = *reinterpret_cast<const f4u*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

template <int EPI>
__device__ __forceinline__ float epi(float v, const float* zprev_elem) {
    if (EPI == GCN_EPI_RELU) return v > 0.f ? v : 0.f;
    if (EPI == GCN_EPI_MASK) return *zprev_elem > 0.f ? v : 0.f;
    return v;
}

// Lane quarter q (16 lanes) holds x[e] = m[q][e]; afterwards it holds m[e][q].
__device__ __forceinline__ void quarter_transpose(float (&x)[4]) {
    auto swap = [](float& a, float& b, bool halves) {
        const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
        const auto v = halves ? __builtin_amdgcn_permlane32_swap(ua, ub, false, false)
                              : __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
        a = __uint_as_float(v[0]);
        b = __uint_as_float(v[1]);
    };
    swap(x[0], x[2], true);
    swap(x[1], x[3], true);
    swap(x[0], x[1], false);
    swap(x[2], x[3], false);
}

struct TallArgs {
    int64_t M;
    int32_t N, K;
    const float* A; int64_t lda;
    const float* B; int64_t ldb; int tb;
    float* C; int64_t ldc;
    const float* bias;
    const float* Zprev; int64_t ldzprev;
    int32_t Kpad;      // K rounded up to 16
    int asc;           // add in ascending k
    int32_t S;         // LDS row stride in floats: 16*NT + 4 (bank-conflict-free B reads)
    const float* row_scale;   // NULL, or one factor per row of C, applied after bias and epilogue (wide store path only)
};

// Columns n0 .. n0 + 16 NT of op(B) into LDS, zeros behind its end: 16 bytes per load, four loads of a thread on their way.
template <int NT>
__device__ __forceinline__ void stage_b(const TallArgs& a, int n0, float* Bs) {
    constexpr int C = 16 * NT;
    auto four = [](const float* p, int left) {          // the first `left` of four
        if (left >= 4) return load4(p);
        return make_float4(left > 0 ? p[0] : 0.f, left > 1 ? p[1] : 0.f, left > 2 ? p[2] : 0.f, 0.f);
    };
    if (!a.tb) {
        const int count = a.Kpad * (C / 4);
#pragma unroll 4
        for (int i = threadIdx.x; i < count; i += blockDim.x) {
            const int k = i / (C / 4), j = i % (C / 4) * 4;
            *reinterpret_cast<float4*>(Bs + k * a.S + j) = four(a.B + (int64_t)k * a.ldb + n0 + j, k < a.K ? a.N - n0 - j : 0);
        }
    } else {
        const int count = a.Kpad / 4 * C;
#pragma unroll 4
        for (int i = threadIdx.x; i < count; i += blockDim.x) {
            const int k = i / C * 4, j = i % C;
            const float4 v = four(a.B + (int64_t)(n0 + j) * a.ldb + k, n0 + j < a.N ? a.K - k : 0);
            float* const at = Bs + k * a.S + j;
            at[0] = v.x; at[a.S] = v.y; at[2 * a.S] = v.z; at[3 * a.S] = v.w;
        }
    }
}

// How the rows of C leave.  By the two MFMA operands in turned order a lane ends up with four consecutive columns of one row of C (element v of tile t is
// C[row0 + l%16][16t + 4*(l/16) + v]) and stores them with one instruction.  WIDE: N % 4 == 0 and 16-byte aligned rows of C (and of Zprev for
// the mask); ANY: at any address (SINGLE, the operands
// the other way round and single columns of four rows per lane and store: 1.5 M x 16 x 15 41 -> 33 us, x 41 164 -> 116; 0.2 M x 602 x 41 200 -> 166); SINGLE: up to
// 16 columns where it is the faster, see single_columns.  ANY takes the bias from LDS, and the columns that end
// in their tile are handled once, behind the whole tiles: loads of single biases and code for the end in every tile took registers, and scalar ones were
// saved to memory (with eight tiles 0.2 M x 16 x 127 and bias 35 us, now 27; with sixteen x 255 65 and 44; with four 76 registers, now 63: 0.58 M x 64 x 107 and
// bias 196 and 158).
// ASC: the products of an element of C are added in ascending k, like the chain of the plain kernel: an instruction
// adds its four products in the order of the lane quarters, so quarter kq has to supply k = k0 + 4e + kq to instruction
// e, and the 16 bytes that it loads at k0 + 4 kq are exchanged between the quarters (a 4 x 4 transposition, four
// instructions).  Without it instruction e takes k = k0 + 4 kq + e.  op(B) leaves its workgroups no more than four wavefronts to a SIMD, so that
// the compiler need not save registers for eight (which put fewer reads of it together: 0.2 M x 602 x 41 223 us and 170).  Not with the wide stores: the
// code is the same there, but each wavefront is given the registers of a fourth of a SIMD, and the second column of workgroups comes in later (137 K x 256 x 100 and
// bias 93 us without that, 104 with it; 110 K and no bias 74 and 82).
enum TallStore { SINGLE, ANY, WIDE };
template <int NT, int EPI, int STORE, bool ASC>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, ASC && STORE != WIDE ? 4 : 8))) void k_gemm_tall(TallArgs a) {
    extern __shared__ float Bs[];                       // [Kpad][S], then the bias
    static_assert(STORE != SINGLE || NT == 1, "one tile");
    auto product = [](float b, float x, floatx4 c) {
        return STORE == SINGLE ? __builtin_amdgcn_mfma_f32_16x16x4f32(x, b, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x4f32(b, x, c, 0, 0, 0);
    };
    const int n0 = blockIdx.y * (NT * 16);
    stage_b<NT>(a, n0, Bs);
    if (STORE != WIDE && a.bias)
        for (int j = threadIdx.x; j < 16 * NT; j += blockDim.x) Bs[a.Kpad * a.S + j] = n0 + j < a.N ? a.bias[n0 + j] : 0.f;
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int64_t ntiles = (a.M + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * waves + wave; tile < ntiles; tile += (int64_t)gridDim.x * waves) {
        const int64_t row0 = tile * 16;
        int64_t arow = row0 + r;
        if (arow >= a.M) arow = a.M - 1;                // clamp: loads stay in bounds, stores are masked
        const float* ap = a.A + arow * a.lda + 4 * kq;
        floatx4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = (floatx4){0.f, 0.f, 0.f, 0.f};
        const int kfull = a.K & ~15;
        int k0 = 0;
        for (; k0 + 64 <= kfull; k0 += 64) {            // four 16-deep steps per trip: 4 loads in flight
            float4 av[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) av[s] = load4(ap + k0 + 16 * s);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                float ae[4] = {av[s].x, av[s].y, av[s].z, av[s].w};
                if constexpr (ASC) quarter_transpose(ae);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float* bp = Bs + (k0 + 16 * s + (ASC ? 4 * e + kq : 4 * kq + e)) * a.S + r;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = product(bp[16 * t], ae[e], acc[t]);
                }
            }
        }
        for (; k0 < kfull; k0 += 16) {
            const float4 av = load4(ap + k0);
            float ae[4] = {av.x, av.y, av.z, av.w};
            if constexpr (ASC) quarter_transpose(ae);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* bp = Bs + (k0 + (ASC ? 4 * e + kq : 4 * kq + e)) * a.S + r;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = product(bp[16 * t], ae[e], acc[t]);
            }
        }
        if (k0 < a.K) {                                 // ragged tail (fewer than 16 columns left)
            // whole 16-byte pieces when K is a multiple of 4 (300 = 18*16 + 12), else element-wise guarded loads
            float tail[4] = {0.f, 0.f, 0.f, 0.f};
            if ((a.K & 3) == 0) {
                if (k0 + 4 * kq + 4 <= a.K) {
                    const float4 av = load4(ap + k0);
                    tail[0] = av.x; tail[1] = av.y; tail[2] = av.z; tail[3] = av.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) tail[e] = k0 + 4 * kq + e < a.K ? ap[k0 + e] : 0.f;
            }
            if constexpr (ASC) quarter_transpose(tail);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + (ASC ? 4 * e + kq : 4 * kq + e);
                const float ae = tail[e];
                const float* bp = Bs + k * a.S + r;     // rows K..Kpad-1 of Bs are zero
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = product(bp[16 * t], ae, acc[t]);
            }
        }
        if constexpr (STORE == SINGLE) {                // element v is C[row0 + 4 kq + v][r]
            if (r >= a.N) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = row0 + 4 * kq + v;
                if (row < a.M)
                    a.C[row * a.ldc + r] = epi<EPI>(a.bias ? acc[0][v] + Bs[a.Kpad * a.S + r] : acc[0][v], EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + r : nullptr);
            }
            continue;
        }
        const int64_t row = row0 + r;
        if constexpr (STORE == WIDE) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int col = n0 + 16 * t + 4 * kq;           // N % 4 == 0: the four columns exist together
                if (col >= a.N || row >= a.M) continue;
                float4 o = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
                if (a.bias) {
                    o.x += a.bias[col]; o.y += a.bias[col + 1]; o.z += a.bias[col + 2]; o.w += a.bias[col + 3];
                }
                if (EPI == GCN_EPI_RELU) {
                    o.x = o.x > 0.f ? o.x : 0.f; o.y = o.y > 0.f ? o.y : 0.f;
                    o.z = o.z > 0.f ? o.z : 0.f; o.w = o.w > 0.f ? o.w : 0.f;
                } else if (EPI == GCN_EPI_MASK) {
                    const float4 m = *reinterpret_cast<const float4*>(a.Zprev + row * a.ldzprev + col);
                    o.x = m.x > 0.f ? o.x : 0.f; o.y = m.y > 0.f ? o.y : 0.f;
                    o.z = m.z > 0.f ? o.z : 0.f; o.w = m.w > 0.f ? o.w : 0.f;
                }
                if (a.row_scale) {
                    const float rs = a.row_scale[row];
                    o.x *= rs; o.y *= rs; o.z *= rs; o.w *= rs;
                }
                *reinterpret_cast<float4*>(a.C + row * a.ldc + col) = o;
            }
            continue;
        }
        const int left = a.N - n0, full = left >= 16 * NT ? NT : left / 16;        // tiles of 16 columns
        float* const c = a.C + row * a.ldc + n0 + 4 * kq;
        const float* const z = EPI == GCN_EPI_MASK ? a.Zprev + row * a.ldzprev + n0 + 4 * kq : nullptr;
        const float* const bias = Bs + a.Kpad * a.S + 4 * kq;
        auto store = [&](int at, floatx4 o) {
            float m[4] = {};
            if (EPI == GCN_EPI_MASK) {
                const float4 x = load4(z + at);
                m[0] = x.x; m[1] = x.y; m[2] = x.z; m[3] = x.w;
                __builtin_amdgcn_wave_barrier();        // (the mask may be C: all lanes read before any of them stores what another one reads)
            }
            *reinterpret_cast<floatx4u*>(c + at) = (floatx4){epi<EPI>(o[0], m), epi<EPI>(o[1], m + 1), epi<EPI>(o[2], m + 2), epi<EPI>(o[3], m + 3)};
        };
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t < full) {
                floatx4 o = acc[t];
                if (a.bias) o += *reinterpret_cast<const floatx4*>(bias + 16 * t);
                if (row < a.M) store(16 * t, o);
            }
        }
        if (full == NT || left == 16 * full) continue;
        // The last tile.  The last two or three columns of a row leave with those before them, which another lane stores too, with the same bits
        // (one by one they made 1.5 M x 16 x 31 90 us, now 65; 1 M x 64 x 23 75, now 64).
        floatx4 o = acc[0];
#pragma unroll
        for (int t = 1; t < NT; ++t)
            if (t == full) o = acc[t];
        if (a.bias) o += *reinterpret_cast<const floatx4*>(bias + 16 * full);
        const int tail = a.N & 3, mine = left - 16 * full - 4 * kq;                // columns from this lane's four on
        int at = 16 * full;
        if (tail >= 2 && left - at > 4) {
            const float x = __shfl_up(o[2], 16, 64), y = __shfl_up(o[3], 16, 64);
            if (mine == tail) {
                o = tail == 2 ? (floatx4){x, y, o[0], o[1]} : (floatx4){y, o[0], o[1], o[2]};
                at -= 4 - tail;
            }
        }
        if (row >= a.M || mine <= 0) continue;
        if (mine >= 4 || at < 16 * full) store(at, o);
        else {
#pragma unroll
            for (int v = 0; v < 3; ++v)
                if (v < mine) c[at + v] = epi<EPI>(o[v], EPI == GCN_EPI_MASK ? z + at + v : nullptr);
        }
    }
}

// ---- the same product for dense rows that are not a multiple of a 128-byte line (300 floats = 1200 bytes) ----
// With such rows the strided 64-byte pieces of k_gemm_tall straddle lines and every line is touched by several
// instructions.  Here a wavefront instead copies its whole 16-row strip, which is one contiguous run of 16 K
// floats when lda == K, with fully coalesced 16-byte loads (1 KB per instruction, like a plain copy) into its own
// LDS buffer and takes the MFMA operands from there; the loads of the next strip are in flight (in registers)
// while the current strip is multiplied.  Needs lda == K, K % 4 == 0, 16-byte aligned A, and the wide store path
// (N % 4 == 0, aligned C).  KV = 16-byte loads per lane and strip = ceil(K / 16).
// A wavefront keeps the results of `held` strips in LDS, where they leave room for as many workgroups, and stores them in one burst: single kilobytes
// of writes among the reads of all memory cost more than their share (300 x 16 over 1.8 M rows 429 -> 397 us, 228 x 12 over 3 M 606 -> 540; the
// same reads without any store 2.77 ms of 3.46 on 14 M).
constexpr int flat_held(int NT, int KV) { return NT == 1 && KV == 19 ? 8 : 0; }
template <int NT, int EPI, int KV>
__global__ __launch_bounds__(512) void k_gemm_tall_flat(TallArgs a) {
    extern __shared__ float lds[];
    float* Bs = lds;                                    // [Kpad][S]
    const int strip_floats = 16 * a.K;
    float* As = lds + a.Kpad * a.S + (threadIdx.x >> 6) * (KV * 256);    // this wavefront's strip, flat
    const int n0 = blockIdx.y * (NT * 16);
    stage_b<NT>(a, n0, Bs);
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int r = lane & 15, kq = lane >> 4;
    const int64_t ntiles = (a.M + 15) / 16;
    const int64_t total = a.M * (int64_t)a.K;           // floats of A
    const int64_t stride = (int64_t)gridDim.x * waves;
    constexpr int HELD = flat_held(NT, KV);
    float* const Cs = lds + a.Kpad * a.S + (blockDim.x >> 6) * (KV * 256) + (threadIdx.x >> 6) * (HELD * 256);
    int held = 0;
    int64_t first = 0;                                  // of the strips held
    float4 pre[KV];
    auto fetch = [&](int64_t tile) {
        const int64_t base = tile * strip_floats;
#pragma unroll
        for (int q = 0; q < KV; ++q) {
            const int64_t off = base + (int64_t)(q * 64 + lane) * 4;
            pre[q] = (q * 256 + lane * 4 < strip_floats && off + 4 <= total) ? stream4(a.A + off)
                                                                             : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    int64_t tile = (int64_t)blockIdx.x * waves + wave;
    if (tile < ntiles) fetch(tile);
    for (; tile < ntiles; tile += stride) {
#pragma unroll
        for (int q = 0; q < KV; ++q) *reinterpret_cast<float4*>(As + (q * 64 + lane) * 4) = pre[q];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (tile + stride < ntiles) fetch(tile + stride);      // in flight while this strip is multiplied

        const int64_t row0 = tile * 16;
        const float* ap = As + r * a.K + 4 * kq;
        floatx4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = (floatx4){0.f, 0.f, 0.f, 0.f};
        const int kfull = a.K & ~15;
        int k0 = 0;
        for (; k0 < kfull; k0 += 16) {
            const float4 av = *reinterpret_cast<const float4*>(ap + k0);
            const float ae[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* bp = Bs + (k0 + 4 * kq + e) * a.S + r;
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(bp[16 * t], ae[e], acc[t], 0, 0, 0);
            }
        }
        if (k0 < a.K) {                                 // K % 16 is 4, 8 or 12: whole 16-byte pieces
            float4 av = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k0 + 4 * kq + 4 <= a.K) av = *reinterpret_cast<const float4*>(ap + k0);
            const float ae[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* bp = Bs + (k0 + 4 * kq + e) * a.S + r;     // rows K..Kpad-1 of Bs are zero
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(bp[16 * t], ae[e], acc[t], 0, 0, 0);
            }
        }
        const int64_t row = row0 + r;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = n0 + 16 * t + 4 * kq;               // N % 4 == 0: the four columns exist together
            if (col >= a.N || row >= a.M) continue;
            float4 o = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
            if (a.bias) {
                o.x += a.bias[col]; o.y += a.bias[col + 1]; o.z += a.bias[col + 2]; o.w += a.bias[col + 3];
            }
            if (EPI == GCN_EPI_RELU) {
                o.x = o.x > 0.f ? o.x : 0.f; o.y = o.y > 0.f ? o.y : 0.f;
                o.z = o.z > 0.f ? o.z : 0.f; o.w = o.w > 0.f ? o.w : 0.f;
            } else if (EPI == GCN_EPI_MASK) {
                const float4 m = *reinterpret_cast<const float4*>(a.Zprev + row * a.ldzprev + col);
                o.x = m.x > 0.f ? o.x : 0.f; o.y = m.y > 0.f ? o.y : 0.f;
                o.z = m.z > 0.f ? o.z : 0.f; o.w = m.w > 0.f ? o.w : 0.f;
            }
            if (a.row_scale) {
                const float rs = a.row_scale[row];
                o.x *= rs; o.y *= rs; o.z *= rs; o.w *= rs;
            }
            if constexpr (HELD) *reinterpret_cast<float4*>(Cs + held * 256 + r * 16 + 4 * kq) = o;
            else *reinterpret_cast<float4*>(a.C + row * a.ldc + col) = o;
        }
        if constexpr (HELD) {
            if (held == 0) first = tile;
            if (++held == HELD || tile + stride >= ntiles) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int col = n0 + 4 * (lane & 3);
#pragma unroll 4
                for (int u = 0; u < held; ++u) {
                    const int64_t to = (first + u * stride) * 16 + (lane >> 2);
                    if (col < a.N && to < a.M) *reinterpret_cast<float4*>(a.C + to * a.ldc + col) = *reinterpret_cast<const float4*>(Cs + u * 256 + lane * 4);
                }
                held = 0;
            }
        }
        // the next strip overwrites As: this wavefront's LDS operations complete in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- C = A^T B over a long K ---------------------------------------------------------------------
// A workgroup takes the rows [kb, ke) of A and B.  The columns of A are cut into groups of 64; inside a group lane i
// covers columns 4i..4i+3 with one 16-byte load, which makes four M-tiles {4i+t : i} for t = 0..3.  The groups are
// dealt to `gw` wavefronts (wavefront w owns groups w, w + gw, ... of the workgroup's share, MG of them at most); when
// there are fewer than four groups the workgroup has `rw` such sets of wavefronts, which take its 16-row trips in turn
// and whose sums are added in LDS in a fixed order, so that a narrow product writes no more partial results than a
// wide one.  Each trip consumes 16 rows (four per matrix instruction, one per lane quarter).  blockIdx.y takes 16 NT columns of B, blockIdx.z a share of the
// column groups of A: any M and N.  The partial M x N results go to part[blockIdx.x][M][N].
// Bound by the stream of A and B up to about 32 columns of B (128 x 16 over 4.4 M rows: 0.36 ms, 6.9 TB/s; 300 x 16 over 14.2 M rows: 2.86 ms,
// 6.4 TB/s) and by the fp32 matrix rate and the stream together beyond (256 x 64 over 120 K rows 52 us, 75 TFLOP/s; one
// thread per output element took 16.5 ms).  Without the next trip on its way 3.3 ms, 0.41 ms and 61 us.
struct TnArgs {
    int64_t K;
    int32_t M, N;
    const float* A; int64_t lda;
    const float* B; int64_t ldb;
    float* part;
    int64_t k_per_block;
    int gw, rw;        // wavefronts per workgroup = gw * rw
};

template <int MG, int NT, bool STREAM>
__global__ __launch_bounds__(512) void k_gemm_tn(TnArgs a) {
    extern __shared__ float s_part[];                   // [rw - 1][gw][MG * 4 * NT][64][4]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gwave = wave % a.gw, rwave = wave / a.gw;
    const int i = lane & 15, kq = lane >> 4;
    const int64_t kb = (int64_t)blockIdx.x * a.k_per_block;
    const int64_t ke = kb + a.k_per_block < a.K ? kb + a.k_per_block : a.K;
    const int n0 = blockIdx.y * (16 * NT);
    const int m0 = blockIdx.z * (a.gw * MG * 64);
    floatx4 acc[MG][4][NT], sum[MG][4][NT];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) sum[g][t][u] = acc[g][t][u] = (floatx4){0.f, 0.f, 0.f, 0.f};
    // after every 8 trips: a workgroup may take tens of thousands of rows, too many for one chain of additions (300 x 16 over
    // 14.2 M rows: 29e-7 of the norm off without, 3.6e-7 with, and 7.5e-7 with 8192 workgroups of one chain each)
    auto flush = [&]() {
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    sum[g][t][u] += acc[g][t][u];
                    acc[g][t][u] = (floatx4){0.f, 0.f, 0.f, 0.f};
                }
    };

    // Lanes past the last column repeat the last four columns of A (the last column of B): no load needs a guard, and
    // an element that two lanes compute gets the same bits from both.
    auto mcol = [&](int g, int ii) {
        const int c = m0 + (gwave + a.gw * g) * 64 + 4 * ii;
        return c < a.M - 4 ? c : a.M - 4;
    };
    auto ncol = [&](int u) {
        const int c = n0 + 16 * u + i;
        return c < a.N ? c : a.N - 1;
    };
    const float* ap[MG];
    const float* bp[NT];
    const int64_t kfirst = kb + 16 * rwave;
#pragma unroll
    for (int g = 0; g < MG; ++g) ap[g] = a.A + (kfirst + kq) * a.lda + mcol(g, i);
#pragma unroll
    for (int u = 0; u < NT; ++u) bp[u] = a.B + (kfirst + kq) * a.ldb + ncol(u);
    const int kstep = 16 * a.rw;
    int64_t k0 = kfirst;
    // Wavefronts on neighbouring columns share the lines at their edges when rows are not whole lines: kept within four
    // trips of each other they find them in the caches (300 x 16 over 1.8 M rows 385 us without, 371 with; 500 x 64
    // over 60 K rows 57 and 52).  All of them take the same number of trips.
    const bool in_step = a.rw == 1 && a.gw > 1;
    struct Trip { float a[4][MG][4], b[4][NT]; };
    auto load = [&](Trip& x) {                          // 16 rows from ap, bp on, which move to the next trip
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int u = 0; u < NT; ++u) x.b[s][u] = bp[u][4 * s * a.ldb];
#pragma unroll
            for (int g = 0; g < MG; ++g) {
                const float4 v = STREAM ? stream4(ap[g] + 4 * s * a.lda) : load4(ap[g] + 4 * s * a.lda);
                x.a[s][g][0] = v.x; x.a[s][g][1] = v.y; x.a[s][g][2] = v.z; x.a[s][g][3] = v.w;
            }
        }
#pragma unroll
        for (int g = 0; g < MG; ++g) ap[g] += (int64_t)kstep * a.lda;
#pragma unroll
        for (int u = 0; u < NT; ++u) bp[u] += (int64_t)kstep * a.ldb;
    };
    auto multiply = [&](const Trip& x) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        acc[g][t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.a[s][g][t], x.b[s][u], acc[g][t][u], 0, 0, 0);
    };
    int trip = 0;
    auto step = [&]() { if (in_step && (++trip & 3) == 0) __builtin_amdgcn_s_barrier(); };
    const int64_t full = k0 + 16 <= ke ? (ke - 16 - k0) / kstep + 1 : 0;      // whole trips of this wavefront
    const int64_t all = k0 < ke ? (ke - 1 - k0) / kstep + 1 : 0;        // with the short one
    {                                                   // the next trip is on its way while this one is multiplied
        Trip x, y;
        int64_t t = 0;
        if (full > 0) load(x);
#pragma unroll 1
        for (; t + 2 <= full; t += 2) {
            load(y);
            step();
            multiply(x);
            if (t + 2 < full) load(x);
            step();
            multiply(y);
            if ((t & 6) == 6) flush();
        }
        if (t < full) { step(); multiply(x); }
    }
    if (full < all) {                                   // the short trip: rows past the end count as zero
        k0 += full * kstep;
        step();
        Trip x;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool kok = k0 + 4 * s + kq < ke;
#pragma unroll
            for (int u = 0; u < NT; ++u) x.b[s][u] = kok ? bp[u][4 * s * a.ldb] : 0.f;
#pragma unroll
            for (int g = 0; g < MG; ++g) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (kok) v = load4(ap[g] + 4 * s * a.lda);
                x.a[s][g][0] = v.x; x.a[s][g][1] = v.y; x.a[s][g][2] = v.z; x.a[s][g][3] = v.w;
            }
        }
        multiply(x);
    }
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[g][t][u] += sum[g][t][u];
    // the row sets hold partial sums of the same tiles: added in order 0, 1, 2, 3, from LDS, where all of them lie side by side (put there and
    // added one after another 64 x 41 over 20 K rows took 11.7 us, now 9.8, 64 x 64 over 120 K 21.8 and 19.6)
    if (a.rw > 1) {
        constexpr int TILES = MG * 4 * NT;
        float4* const mine = reinterpret_cast<float4*>(s_part) + (size_t)gwave * TILES * 64 + lane;
        if (rwave > 0) {
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int u = 0; u < NT; ++u) {
                        const floatx4 v = acc[g][t][u];
                        mine[((rwave - 1) * a.gw * TILES + (g * 4 + t) * NT + u) * 64] = make_float4(v[0], v[1], v[2], v[3]);
                    }
        }
        __syncthreads();
        for (int w = 1; w < a.rw && rwave == 0; ++w)
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int u = 0; u < NT; ++u) {
                        const float4 v = mine[((w - 1) * a.gw * TILES + (g * 4 + t) * NT + u) * 64];
                        acc[g][t][u] += (floatx4){v.x, v.y, v.z, v.w};
                    }
    }
    if (rwave != 0) return;
    float* out = a.part + (int64_t)blockIdx.x * a.M * a.N;
    // D[ii = 4*kq + v][j = i] of tile (g, t) is C[m = mcol(g, ii) + t][n = ncol(u)]
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = mcol(g, 4 * kq + v);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) out[(int64_t)(m + t) * a.N + ncol(u)] = acc[g][t][u][v];
        }
}

// The same for M <= 32 and N <= 32: lane i covers columns i and i+16 of A with 4-byte loads (one M-tile each) and the
// four wavefronts split the rows.
template <int MG, int NT>
__global__ __launch_bounds__(256) void k_gemm_tn_narrow(TnArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, kq = lane >> 4;
    const int64_t kb = (int64_t)blockIdx.x * a.k_per_block;
    const int64_t ke = kb + a.k_per_block < a.K ? kb + a.k_per_block : a.K;
    floatx4 acc[MG][NT], total[MG][NT];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int u = 0; u < NT; ++u) total[g][u] = acc[g][u] = (floatx4){0.f, 0.f, 0.f, 0.f};
    bool mok[MG], nok[NT];
#pragma unroll
    for (int g = 0; g < MG; ++g) mok[g] = 16 * g + i < a.M;
#pragma unroll
    for (int u = 0; u < NT; ++u) nok[u] = 16 * u + i < a.N;
    int trip = 0;
    for (int64_t k0 = kb + 16 * wave; k0 < ke; k0 += 64) {
        float av[4][MG], bv[4][NT];
#pragma unroll
        for (int s = 0; s < 4; ++s) {                   // issue every load of the trip first
            const int64_t k = k0 + 4 * s + kq;
            const bool kok = k < ke;
            const float* arow = a.A + (kok ? k : kb) * a.lda;
            const float* brow = a.B + (kok ? k : kb) * a.ldb;
#pragma unroll
            for (int u = 0; u < NT; ++u) bv[s][u] = (kok && nok[u]) ? brow[16 * u + i] : 0.f;
#pragma unroll
            for (int g = 0; g < MG; ++g) av[s][g] = (kok && mok[g]) ? arow[16 * g + i] : 0.f;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int u = 0; u < NT; ++u)
                    acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s][g], bv[s][u], acc[g][u], 0, 0, 0);
        if ((++trip & 7) == 0) {                        // (as in k_gemm_tn)
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int u = 0; u < NT; ++u) { total[g][u] += acc[g][u]; acc[g][u] = (floatx4){0.f, 0.f, 0.f, 0.f}; }
        }
    }
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[g][u] += total[g][u];
    // the four wavefronts hold partial sums of the same tiles: add them in LDS, fixed order
    float* out = a.part + (int64_t)blockIdx.x * a.M * a.N;
    __shared__ float s_red[4][MG][NT][64][4];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) s_red[wave][g][u][lane][v] = acc[g][u][v];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float sum = ((s_red[0][g][u][lane][v] + s_red[1][g][u][lane][v]) + s_red[2][g][u][lane][v]) +
                                      s_red[3][g][u][lane][v];
                    const int m = 16 * g + 4 * kq + v, n = 16 * u + i;
                    if (m < a.M && n < a.N) out[(int64_t)m * a.N + n] = sum;
                }
    }
}

// What backward does with S = A G at width 16 on both sides, in one pass over the rows: Gprev = (S W^T) masked by Zprev > 0, and the
// partial results of Y = Hin^T S (as k_gemm_tn_narrow leaves them: same rows, same order).  Bound by memory: it reads S and H once
// and writes Gprev, where k_gemm_tall and k_gemm_tn_narrow together read S and H twice; the rows of the next two trips are on
// their way (64 KB per compute unit).  The first product takes and leaves four columns of a row per lane, so the mask is the
// lane's own 16 bytes of H; the second contracts over the rows, which are turned round in LDS.  OWN: Zprev is Hin.
// 14.2 M rows: 520 us (5.2 TB/s), 490 + 320 by the two kernels; 1.8 M: 57, 58 + 50.
template <bool OWN>
__global__ __launch_bounds__(256) void k_gemm_back(TnArgs a, const float* __restrict__ W, const float* Zprev, float* Gprev) {
    constexpr int ST = 20;                              // row stride of the tiles
    __shared__ float s_tile[4][2][16 * ST];
    __shared__ float s_red[4][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    float* const hs = s_tile[wave][0];
    float* const ss = s_tile[wave][1];
    const float4 w4 = load4(W + r * 16 + 4 * g);
    const float w[4] = {w4.x, w4.y, w4.z, w4.w};
    const int64_t kb = (int64_t)blockIdx.x * a.k_per_block;
    const int64_t ke = kb + a.k_per_block < a.K ? kb + a.k_per_block : a.K;
    struct Rows { float4 s, h, z; };
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    auto fetch = [&](int64_t k0) {
        Rows x = {zero, zero, zero};
        if (k0 + r < ke) {
            x.s = stream4(a.B + (k0 + r) * 16 + 4 * g);
            x.h = stream4(a.A + (k0 + r) * a.lda + 4 * g);
            if (!OWN) x.z = stream4(Zprev + (k0 + r) * 16 + 4 * g);
        }
        return x;
    };
    floatx4 acc = {0.f, 0.f, 0.f, 0.f}, total = acc;
    int trip = 0;
    int64_t k0 = kb + 16 * wave;
    Rows next = fetch(k0), after = fetch(k0 + 64);
    for (; k0 < ke; k0 += 64) {
        const Rows x = next;
        next = after;
        after = fetch(k0 + 128);
        floatx4 d = {0.f, 0.f, 0.f, 0.f};
        const float s[4] = {x.s.x, x.s.y, x.s.z, x.s.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], s[e], d, 0, 0, 0);
        *reinterpret_cast<float4*>(hs + r * ST + 4 * g) = x.h;
        *reinterpret_cast<float4*>(ss + r * ST + 4 * g) = x.s;
        const float4 m = OWN ? x.h : x.z;
        if (k0 + r < ke)
            *reinterpret_cast<float4*>(Gprev + (k0 + r) * 16 + 4 * g) =
                make_float4(m.x > 0.f ? d[0] : 0.f, m.y > 0.f ? d[1] : 0.f, m.z > 0.f ? d[2] : 0.f, m.w > 0.f ? d[3] : 0.f);
        // each wavefront reads only what it wrote; LDS operations of one wavefront complete in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float av[4], bv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { av[e] = hs[(4 * e + g) * ST + r]; bv[e] = ss[(4 * e + g) * ST + r]; }
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], acc, 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if ((++trip & 7) == 0) { total += acc; acc = (floatx4){0.f, 0.f, 0.f, 0.f}; }      // (as in k_gemm_tn)
    }
    acc += total;
#pragma unroll
    for (int v = 0; v < 4; ++v) s_red[wave][(4 * g + v) * 16 + r] = acc[v];
    __syncthreads();
    const int o = threadIdx.x;
    a.part[(int64_t)blockIdx.x * 256 + o] = ((s_red[0][o] + s_red[1][o]) + s_red[2][o]) + s_red[3][o];
}

// The same for 16, 32 or 64 columns of Hin and up to as many of S.  A wavefront takes 16 rows and 16 MT columns of Hin and Gprev; of 64, a
// pair of wavefronts shares the rows.  The first product takes a row's columns of S four at a time per lane, from memory, and W from LDS; the
// second takes the same rows of S turned round in LDS, and two columns of Hin per lane, from memory.  The next 16 rows are on
// their way.  Bound by memory and the fp32 matrix rate together: S is read once where k_gemm_tall and k_gemm_tn read it twice, and Hin once
// where it is the mask.  Faster than the two at every size (rows 1 K to 1.5 M, 16 to 64 columns of Hin, 2 to 64 of S: 63 layer calls with a
// product of two entries a row, 1.00 to 1.35 times as fast; other widths of Hin have no such kernel): 64 x 41 over 120 K rows 81 -> 75 us, 32 x 32 over 0.5 M 109 -> 87, 16 x 5 over 1.5 M
// 117 -> 101, 64 x 8 over 5 K 14.3 -> 10.9.  256-64-64-41 on 120 K vertices 1016 -> 990 us an epoch.
template <int NT, int MT, int MH>
__global__ __launch_bounds__(256 * MH) void k_gemm_back_wide(TnArgs a, const float* __restrict__ W, const float* __restrict__ Zprev,
                                                             float* __restrict__ Gprev) {
    constexpr int M = 16 * MT * MH, WS = M + 4;              // row strides: the four quarters of a wavefront on banks of their own
    constexpr int SS = NT == 1 ? 16 : (NT == 4 ? 80 : 48);
    constexpr int SETS = 4, TILES = MT * NT;
    constexpr int W_FLOATS = 16 * NT * WS, TILE_FLOATS = SETS * MH * 16 * SS, SUM_FLOATS = (SETS - 1) * MH * TILES * 256;
    constexpr int FLOATS = W_FLOATS + TILE_FLOATS > SUM_FLOATS ? W_FLOATS + TILE_FLOATS : SUM_FLOATS;
    __shared__ __attribute__((aligned(16))) float s_mem[FLOATS];         // W and the rows of S, the partial sums in the end
    float* const s_w = s_mem;
    float* const s_s = s_mem + W_FLOATS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int m0 = 16 * MT * (wave % MH), set = wave / MH;
    const int N = a.N;
    for (int j = threadIdx.x; j < 16 * NT * M; j += 256 * MH) {
        const int m = j / (16 * NT), k = j % (16 * NT);
        s_w[k * WS + m] = k < N ? W[m * N + k] : 0.f;
    }
    __syncthreads();
    float* const ss = s_s + wave * (16 * SS);
    const int64_t kb = (int64_t)blockIdx.x * a.k_per_block;
    const int64_t ke = kb + a.k_per_block < a.K ? kb + a.k_per_block : a.K;
    auto load_cols = [](float (&h)[MT], const float* p) {
        if constexpr (MT == 2) {
            const float2 v = *reinterpret_cast<const float2*>(p);
            h[0] = v.x; h[1] = v.y;
        } else h[0] = *p;
    };
    struct Rows { floatx4 s[NT], z[MT]; float h[4][MT]; };
    auto fetch = [&](int64_t k0, Rows& x) {             // (rows past the end: the last one again)
        const int64_t row = k0 + r < ke ? k0 + r : ke - 1;
        const float* const sp = a.B + row * N + 4 * g;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int left = N - 16 * q - 4 * g;        // columns from this lane's four on
            if (q + 1 < NT || left >= 4) x.s[q] = *reinterpret_cast<const floatx4u*>(sp + 16 * q);
            else x.s[q] = (floatx4){left > 0 ? sp[16 * q] : 0.f, left > 1 ? sp[16 * q + 1] : 0.f, left > 2 ? sp[16 * q + 2] : 0.f, 0.f};
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) x.z[t] = *reinterpret_cast<const floatx4*>(Zprev + row * M + m0 + 16 * t + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t k = k0 + 4 * e + g < ke ? k0 + 4 * e + g : ke - 1;
            load_cols(x.h[e], a.A + k * a.lda + m0 + MT * r);
        }
    };
    floatx4 acc[MT][NT], total[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u) total[t][u] = acc[t][u] = (floatx4){0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int64_t k0, Rows& x) {
        if (k0 + 16 > ke) {
#pragma unroll
            for (int q = 0; q < NT; ++q)
                if (k0 + r >= ke) x.s[q] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    if (k0 + 4 * e + g >= ke) x.h[e][t] = 0.f;
        }
        floatx4 d[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) d[t] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            *reinterpret_cast<floatx4*>(ss + r * SS + 16 * q + 4 * g) = x.s[q];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    d[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(s_w[(16 * q + 4 * g + e) * WS + m0 + 16 * t + r], x.s[q][e], d[t], 0, 0, 0);
        }
        if (k0 + r < ke) {
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                floatx4 o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = x.z[t][v] > 0.f ? d[t][v] : 0.f;
                *reinterpret_cast<floatx4*>(Gprev + (k0 + r) * M + m0 + 16 * t + 4 * g) = o;
            }
        }
        // each wavefront reads only what it wrote; LDS operations of one wavefront complete in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const float b = ss[(4 * e + g) * SS + 16 * u + r];
#pragma unroll
                for (int t = 0; t < MT; ++t) acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.h[e][t], b, acc[t][u], 0, 0, 0);
            }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    constexpr int STEP = 16 * SETS;
    int64_t k0 = kb + 16 * set;
    int trip = 0;
    Rows x, y;
    if (k0 < ke) fetch(k0, x);
#pragma unroll 1
    for (; k0 < ke; k0 += 2 * STEP) {
        if (k0 + STEP < ke) fetch(k0 + STEP, y);
        multiply(k0, x);
        if (k0 + STEP < ke) {
            if (k0 + 2 * STEP < ke) fetch(k0 + 2 * STEP, x);
            multiply(k0 + STEP, y);
        }
        if ((++trip & 3) == 0) {                        // (as in k_gemm_tn)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) { total[t][u] += acc[t][u]; acc[t][u] = (floatx4){0.f, 0.f, 0.f, 0.f}; }
        }
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[t][u] += total[t][u];
    // the sets of rows hold partial sums of the same tiles: added in order 0, 1, 2, 3
    __syncthreads();
    floatx4* const sums = reinterpret_cast<floatx4*>(s_mem) + (wave % MH) * TILES * 64 + lane;
    if (set > 0) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) sums[((set - 1) * MH * TILES + t * NT + u) * 64] = acc[t][u];
    }
    __syncthreads();
    if (set != 0) return;
#pragma unroll
    for (int w = 0; w < SETS - 1; ++w)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[t][u] += sums[(w * MH * TILES + t * NT + u) * 64];
    float* const out = a.part + (int64_t)blockIdx.x * M * N;
    // D[4 g + v][r] of tile (t, u) is Y[m0 + MT (4 g + v) + t][16 u + r]
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * u + r < N) out[(int64_t)(m0 + MT * (4 * g + v) + t) * N + 16 * u + r] = acc[t][u][v];
}

// Stage 1 of the reduction when there are many partials: group g of `groups` sums the partials g, g+groups, ... in
// ascending order (coalesced over the output index).
__global__ __launch_bounds__(256) void k_tn_fold(int64_t count, int parts, int groups, const float* __restrict__ part,
                                                 float* __restrict__ out) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int g = blockIdx.y;
    if (o >= count) return;
    out[(int64_t)g * count + o] = strided_sum(part + o, count, g, groups, parts);
}

// Stage 2 (see sum_of_parts), then bias, epilogue and store.
template <int EPI>
__global__ __launch_bounds__(1024) void k_tn_reduce(int32_t M, int32_t N, int parts, int transposed, const float* __restrict__ part,
                                                    float* __restrict__ C, int64_t ldc, const float* __restrict__ bias,
                                                    const float* __restrict__ Zprev, int64_t ldzprev) {
    __shared__ SumLds lds;
    sum_of_parts(blockIdx.x, M, N, parts, transposed, part, blockDim.x >> 6, lds.s, [&](int m, int n, float s) {
        if (bias) s += bias[n];
        C[(int64_t)m * ldc + n] = epi<EPI>(s, EPI == GCN_EPI_MASK ? Zprev + (int64_t)m * ldzprev + n : nullptr);
    });
}

// What EpochEnd collected, in one launch: the sums of the weight gradients, each with the update of its weights, and the loss.  (A chain of
// three to six launches of 2 to 6 us, most of each the start of a kernel on cold caches.)
__global__ __launch_bounds__(1024) void k_epoch_end(EpochEnd::Args a) {
    __shared__ SumLds lds;
    const int b = (int)blockIdx.x;
    auto update = [&](float* W, int64_t t, float y) {
        if (W) W[t] = W[t] - a.lr * y;
    };
    if (b == a.loss_at) {
        sum_of_losses(a.lpart, a.lparts, a.inv_m, a.loss, lds.l);
        return;
    }
    if (a.fused.part && b >= a.fused.first) {
        sum_of_fused(b - a.fused.first, a.fused.C, a.fused.CP, a.fused.blocks, a.fused.part, lds.y, [&](int e, float y) {
            a.fused.Y[e] = y;
            update(a.fused.W, e, y);
        });
        return;
    }
    int k = 0;
    while (k + 1 < a.count && b >= a.sums[k + 1].first) ++k;
    const EpochEnd::Sum& g = a.sums[k];
    sum_of_parts(b - g.first, g.M, g.N, g.parts, g.transposed, g.part, sum_waves(g.parts), lds.s, [&](int m, int n, float s) {
        const int64_t t = (int64_t)m * g.N + n;
        g.Y[t] = s;
        update(g.W, t, s);
    });
}

int EpochEnd::finish(float lr, hipStream_t s) {
    args.lr = lr;
    int blocks = 0, waves = args.fused.part || args.loss ? 16 : 1;        // (the other two take all of them)
    for (int k = 0; k < args.count; ++k) {
        waves = std::max(waves, sum_waves(args.sums[k].parts));
        args.sums[k].first = blocks;
        if (lr == 0.f) args.sums[k].W = nullptr;
        blocks += (int)(((int64_t)args.sums[k].M * args.sums[k].N + 63) / 64);
    }
    if (args.fused.part) {
        args.fused.first = blocks;
        if (lr == 0.f) args.fused.W = nullptr;
        blocks += args.fused.CP;
    }
    if (args.loss) args.loss_at = blocks++;
    if (blocks == 0) return GCN_OK;
    hipLaunchKernelGGL(k_epoch_end, dim3((unsigned)blocks), dim3(64 * waves), 0, s, args);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

static inline bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

template <int NT, int STORE, bool ASC>
static void launch_tall_epi(const TallArgs& args, int epilogue, dim3 grid, int threads, size_t lds, hipStream_t s) {
    switch (epilogue) {
        case GCN_EPI_NONE: launch_lds<k_gemm_tall<NT, GCN_EPI_NONE, STORE, ASC>>(grid, threads, lds, s, args); break;
        case GCN_EPI_RELU: launch_lds<k_gemm_tall<NT, GCN_EPI_RELU, STORE, ASC>>(grid, threads, lds, s, args); break;
        default: launch_lds<k_gemm_tall<NT, GCN_EPI_MASK, STORE, ASC>>(grid, threads, lds, s, args); break;
    }
}

template <int NT>
static void launch_tall(const TallArgs& args, int epilogue, dim3 grid, int threads, size_t lds, hipStream_t s) {
    // 16-byte stores when every row of C (and of the mask operand) allows them
    const bool wide = (args.N % 4 == 0) && (args.ldc % 4 == 0) && al16(args.C) &&
                      (epilogue != GCN_EPI_MASK || ((args.ldzprev % 4 == 0) && al16(args.Zprev)));
    if constexpr (NT <= 4) {
        if (args.asc) {
            if (wide) launch_tall_epi<NT, WIDE, true>(args, epilogue, grid, threads, lds, s);
            else launch_tall_epi<NT, ANY, true>(args, epilogue, grid, threads, lds, s);
            return;
        }
    }
    if constexpr (NT == 1) {
        if (!wide && single_columns((args.M + 15) / 16, args.K, device_info().cus)) {
            launch_tall_epi<NT, SINGLE, false>(args, epilogue, grid, threads, lds, s);
            return;
        }
    }
    if (wide) launch_tall_epi<NT, WIDE, false>(args, epilogue, grid, threads, lds, s);
    else launch_tall_epi<NT, ANY, false>(args, epilogue, grid, threads, lds, s);
}

template <int NT, int KV>
static void launch_flat_epi(const TallArgs& args, int waves, int epilogue, dim3 grid, size_t lds, hipStream_t s) {
    switch (epilogue) {
        case GCN_EPI_NONE: launch_lds<k_gemm_tall_flat<NT, GCN_EPI_NONE, KV>>(grid, 64 * waves, lds, s, args); break;
        case GCN_EPI_RELU: launch_lds<k_gemm_tall_flat<NT, GCN_EPI_RELU, KV>>(grid, 64 * waves, lds, s, args); break;
        default: launch_lds<k_gemm_tall_flat<NT, GCN_EPI_MASK, KV>>(grid, 64 * waves, lds, s, args); break;
    }
}

// KV is a compile-time bound of the per-lane loads: the instantiations cover K <= 112 (7), <= 208 (13), <= 304 (19)
static bool launch_tall_flat(const TallArgs& args, int NT, int KV, int waves, int epilogue, dim3 grid, size_t lds, hipStream_t s) {
    if (NT == 1 && KV <= 7) launch_flat_epi<1, 7>(args, waves, epilogue, grid, lds, s);
    else if (NT == 1 && KV <= 13) launch_flat_epi<1, 13>(args, waves, epilogue, grid, lds, s);
    else if (NT == 1 && KV <= 19) launch_flat_epi<1, 19>(args, waves, epilogue, grid, lds, s);
    else if (NT == 2 && KV <= 7) launch_flat_epi<2, 7>(args, waves, epilogue, grid, lds, s);
    else if (NT == 2 && KV <= 13) launch_flat_epi<2, 13>(args, waves, epilogue, grid, lds, s);
    else if (NT == 2 && KV <= 19) launch_flat_epi<2, 19>(args, waves, epilogue, grid, lds, s);
    else return false;
    return true;
}

template <int MG, int NT>
static void launch_tn(const TnArgs& args, bool stream, dim3 grid, hipStream_t s) {
    const size_t lds = (size_t)(args.rw - 1) * args.gw * MG * 4 * NT * 64 * sizeof(floatx4);
    if (stream) launch_lds<k_gemm_tn<MG, NT, true>>(grid, 64 * args.gw * args.rw, lds, s, args);
    else launch_lds<k_gemm_tn<MG, NT, false>>(grid, 64 * args.gw * args.rw, lds, s, args);
}

// C = the sum of `parts` partial results (each M x N, or N x M when transposed) in a fixed order, plus bias, epilogue.
int reduce_parts_launch(int32_t M, int32_t N, int parts, bool transposed, const float* part, float* C, int64_t ldc,
                        const float* bias, int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s) {
    const int64_t count = (int64_t)M * N;
    const dim3 grid((unsigned)((count + 63) / 64)), block(64 * sum_waves(parts));
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL(k_tn_reduce<GCN_EPI_NONE>, grid, block, 0, s, M, N, parts, (int)transposed, part, C, ldc, bias, Zprev, ldzprev); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL(k_tn_reduce<GCN_EPI_RELU>, grid, block, 0, s, M, N, parts, (int)transposed, part, C, ldc, bias, Zprev, ldzprev); break;
        default: hipLaunchKernelGGL(k_tn_reduce<GCN_EPI_MASK>, grid, block, 0, s, M, N, parts, (int)transposed, part, C, ldc, bias, Zprev, ldzprev); break;
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// The partial results that are left to add, after the first stage where there is one (in the same scratch, behind them).
static const float* folded(const TnShape& g, int64_t count, float* part, hipStream_t s, int* parts) {
    *parts = g.fold ? g.fold : (int)g.blocks;
    if (!g.fold) return part;
    float* const out = part + g.blocks * count;
    hipLaunchKernelGGL(k_tn_fold, dim3((unsigned)((count + 255) / 256), (unsigned)g.fold), dim3(256), 0, s, count, (int)g.blocks, g.fold,
                       (const float*)part, out);
    return out;
}

int gemm_mfma_launch(int ta, int tb, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                     int64_t ldb, float* C, int64_t ldc, const float* bias, int epilogue, const float* Zprev,
                     int64_t ldzprev, hipStream_t s, bool* handled, const float* row_scale, bool* scaled, bool few) {
    *handled = false;
    *scaled = false;
    if (!ta) {
        if (K > 4096 || N > 65535 * 16 || M < 64) return GCN_OK;
        const int nt_total = (int)((N + 15) / 16);
        // tiles per wavefront: as many as fit (whole rows of C from one wavefront when N <= 256), while op(B) for them
        // stays within 40 KB of LDS; up to four tiles in any case, as long as op(B) fits a compute unit's LDS at all
        const int64_t kpad = (K + 15) & ~15ll;
        auto b_bytes = [&](int tiles) { return (size_t)(kpad * (16 * tiles + 4)) * sizeof(float); };
        int NT = nt_total >= 4 ? 4 : nt_total;
        if (nt_total >= 16 && b_bytes(16) <= 40 * 1024) NT = 16;
        else if (nt_total >= 8 && b_bytes(8) <= 40 * 1024) NT = 8;
        // Second operands beyond 64 KB are multiplied in ascending k: 256 x 64 on 120 K rows took 704 us with one thread
        // per element in that order; keeping the order keeps the bits of the hidden activations, on whose signs
        // the ReLU decides.
        const bool ascending = b_bytes(NT) > 64 * 1024;
        const bool wide_c = (N % 4 == 0) && (ldc % 4 == 0) && al16(C) &&
                            (epilogue != GCN_EPI_MASK || ((ldzprev % 4 == 0) && al16(Zprev)));
        // Rows of C that are no whole 16 bytes, beyond the memory-side cache: up to 128 columns leave from one wavefront too while two workgroups fit a
        // compute unit.  In two columns of workgroups the lines that these share are written twice, at different times, and then four columns
        // at a time are slower than single ones (1.2 M x 128 x 95 411 us with single columns, 535 with four, 340 in one piece; x 44 x 90 278, 316
        // and 195; 0.5 M x 128 x 127 237, 217 and 167; from 145 rows of op(B) on four in two pieces are the faster, 0.5 M x 160 x 90 299 and 226).  In
        // whole 16 bytes two pieces stay: 0.5 M x 44 x 96 76, in one 83.
        if (!wide_c && nt_total > 4 && nt_total <= 8 && M * (K + N) * 4 >= (192ll << 20) && b_bytes(8) <= 80 * 1024) NT = 8;
        while (NT > 1 && b_bytes(NT) > 150 * 1024) --NT;
        if (const int tiles = equal_shares(M, N, K, epilogue == GCN_EPI_MASK, NT)) NT = tiles;
        TallArgs args;
        args.M = M; args.N = (int32_t)N; args.K = (int32_t)K;
        args.A = A; args.lda = lda; args.B = B; args.ldb = ldb; args.tb = tb;
        args.C = C; args.ldc = ldc; args.bias = bias; args.Zprev = Zprev; args.ldzprev = ldzprev;
        args.Kpad = (int32_t)kpad;
        args.asc = ascending;
        args.S = 16 * NT + 4;
        args.row_scale = wide_c ? row_scale : nullptr;       // the 16-byte store path applies it; else the caller does
        *scaled = args.row_scale != nullptr;
        const size_t lds = b_bytes(NT) + (bias && !wide_c ? 16 * NT * sizeof(float) : 0);
        if (lds > 150 * 1024) { *scaled = false; return GCN_OK; }
        const int64_t ntiles = (M + 15) / 16;
        {   // Rows that are not whole 128-byte lines, and short rows (up to 208 floats, where the coalesced copy also beats
            // the strided 64-byte pieces: 128 floats 1.02 -> 0.96 ms on 8.7 M rows; at 256 floats it loses, 3.14 -> 3.23 ms):
            // contiguous strips through LDS (see k_gemm_tall_flat), where the operand is beyond the memory-side cache.  Below, the strided
            // kernel is faster, with the operand in the cache and from memory (300 x 16: 40 K rows 18 and 21 us, 160 K 45 and 48, 320 K 89
            // and 87, 1.3 M 341 and 316; 128 x 16: 40 K 8.3 and 10.1, 320 K 36 and 39, 640 K 78 and 73), except on short rows that end
            // inside 64 bytes (100 x 16: 40 K 8.3 and 8.3, 80 K 12.0 and 10.8; eight widths from 68 to 108 on 33 K, 45 K and 65 K rows: 0.78 to
            // 0.98 of the strips' time).  With two tiles of columns it is faster at every size
            // from 128 floats on (128 x 32: 40 K 9.6 and 12.3, 1.3 M 158 and 160; 300 x 32: 1.3 M 369 and 390; 64 x 32: 640 K
            // 44.5 and 46.6, 1.3 M 94 and 87).
            const bool beyond = M * K * 4 >= (224ll << 20);
            const bool strips = K <= 112 ? beyond || (K % 16 != 0 && M >= 65536) : NT == 1 && beyond;
            const bool wide = (N % 4 == 0) && (ldc % 4 == 0) && al16(C) &&
                              (epilogue != GCN_EPI_MASK || ((ldzprev % 4 == 0) && al16(Zprev)));
            const int kv_need = (int)((K + 15) / 16);
            const int KV = kv_need <= 7 ? 7 : (kv_need <= 13 ? 13 : 19);     // the compiled per-lane load counts
            // wavefronts per workgroup: up to four, as the strips leave room beside op(B); measured on 14 M rows of
            // 300 floats: 2: 4.15, 3: 4.29, 4: 3.57, 5: 3.87, 6: 3.74 ms (the same ranking at 64, 128 and 192 floats)
            int fw = (int)((150 * 1024 - (int64_t)lds) / ((int64_t)KV * 256 * sizeof(float)));
            fw = fw > 4 ? 4 : fw;
            const size_t lds_flat = lds + (size_t)(fw > 0 ? fw : 1) * (KV + flat_held(NT, KV)) * 256 * sizeof(float);
            if (strips && fw >= 2 && wide && !ascending && lda == K && (K % 4) == 0 && (((K * 4) % 128) != 0 || K <= 208) && K >= 64 && kv_need <= 19 && NT <= 2 && al16(A) &&
                lds_flat <= 150 * 1024) {
                int64_t fb = (ntiles + fw - 1) / fw;
                const int per_cu = (int)((160 * 1024) / lds_flat);
                const int64_t fcap = 256 * (int64_t)(per_cu < 1 ? 1 : per_cu);
                if (fb > fcap) fb = fcap;
                const dim3 fgrid((unsigned)fb, (unsigned)((nt_total + NT - 1) / NT));
                if (launch_tall_flat(args, NT, KV, fw, epilogue, fgrid, lds_flat, s)) {
                    GCN_LAUNCH_CHECK();
                    *handled = true;
                    return GCN_OK;
                }
            }
        }
        // Eight wavefronts share op(B), and no more workgroups than two per compute unit (one where op(B) allows no two) put it into
        // LDS: 128 x 64 on 200 K rows 59 us with 1536 workgroups of four, 40 with 512 of eight; 64 x 64 on 120 K rows 21 and
        // 17; 16 x 16 on 4.4 M 110 and 100.  Four per compute unit where a strip leaves in two tiles while
        // operand and result are in the memory-side cache (32 x 32 on 400 K 20.6 and 18.5, on 820 K 37.0 and 34.4; on 1.8 M
        // 98 and 105; 64 x 31 on 1 M 87 and 93).
        const int64_t panels = (nt_total + NT - 1) / NT;
        const int waves = tall_waves(ntiles, panels, K, device_info().cus);
        int64_t bx = (ntiles + waves - 1) / waves;
        const bool four = NT == 2 && lds <= 40 * 1024 && M * (K + N) * 4 < (192ll << 20);
        const int64_t cap = (int64_t)device_info().cus * (lds > 80 * 1024 ? 1 : (four ? 4 : 2));
        if (bx > cap) bx = cap;
        const dim3 grid((unsigned)bx, (unsigned)panels);
        switch (NT) {
            case 1: launch_tall<1>(args, epilogue, grid, 64 * waves, lds, s); break;
            case 2: launch_tall<2>(args, epilogue, grid, 64 * waves, lds, s); break;
            case 3: launch_tall<3>(args, epilogue, grid, 64 * waves, lds, s); break;
            case 4: launch_tall<4>(args, epilogue, grid, 64 * waves, lds, s); break;
            case 8: launch_tall<8>(args, epilogue, grid, 64 * waves, lds, s); break;
            default: launch_tall<16>(args, epilogue, grid, 64 * waves, lds, s); break;
        }
        GCN_LAUNCH_CHECK();
        *handled = true;
        return GCN_OK;
    }
    // ta: C = A^T B with K long
    if (tb) return GCN_OK;
    const TnShape g = tn_shape(M, N, K, few);
    if (g.blocks >= (1ll << 31) || g.ny > 65535 || g.nz > 65535 || M * N >= (1ll << 36)) return fail(GCN_ERR_RANGE, "gcn_gemm: output too large");
    EpochEnd* const end = !bias && epilogue == GCN_EPI_NONE && ldc == N ? epoch_end() : nullptr;
    ScratchLease lease;
    void* scratch = end ? end->room.grad[end->layer] : nullptr;
    const bool later = scratch != nullptr;
    if (!later) GCN_TRY(lease.get(&scratch, g.scratch_bytes, s));
    TnArgs args;
    args.K = K; args.M = (int32_t)g.Mw; args.N = (int32_t)g.Nw;
    args.A = g.swap ? B : A; args.lda = g.swap ? ldb : lda;
    args.B = g.swap ? A : B; args.ldb = g.swap ? lda : ldb;
    args.part = (float*)scratch; args.k_per_block = g.kpb;
    // rows of A that are whole 128-byte lines, read once: non-temporal loads
    const bool stream = (args.lda % 32 == 0) && (((uintptr_t)args.A & 127u) == 0) && g.ny == 1;
    args.gw = g.gw; args.rw = g.rw;
    const dim3 grid((unsigned)g.blocks, (unsigned)g.ny, (unsigned)g.nz);
    if (g.narrow) {
        if (g.MG == 1) hipLaunchKernelGGL((k_gemm_tn_narrow<1, 1>), grid, dim3(256), 0, s, args);
        else if (g.NT == 1) hipLaunchKernelGGL((k_gemm_tn_narrow<2, 1>), grid, dim3(256), 0, s, args);
        else hipLaunchKernelGGL((k_gemm_tn_narrow<2, 2>), grid, dim3(256), 0, s, args);
    }
#define GCN_TN_CASE(mg, nt) else if (g.MG == mg && g.NT == nt) launch_tn<mg, nt>(args, stream, grid, s)
    GCN_TN_CASE(1, 1); GCN_TN_CASE(2, 1); GCN_TN_CASE(3, 1);
    GCN_TN_CASE(1, 2); GCN_TN_CASE(1, 3); GCN_TN_CASE(1, 4);
#undef GCN_TN_CASE
    GCN_LAUNCH_CHECK();
    int red_parts;
    const float* const red_src = folded(g, M * N, (float*)scratch, s, &red_parts);
    GCN_LAUNCH_CHECK();
    *handled = true;
    if (later) {
        end->add(red_src, C, (int32_t)M, (int32_t)N, red_parts, g.swap);
        return GCN_OK;
    }
    GCN_TRY(reduce_parts_launch((int32_t)M, (int32_t)N, red_parts, g.swap, red_src, C, ldc, bias, epilogue, Zprev, ldzprev, s));
    return GCN_OK;
}

bool gradient_next(RowsNext& next, int64_t n, int32_t f, const float* H, int64_t ldh, int32_t M) {
    const EpochEnd* const end = epoch_end();
    if (!end || !end->room.few[end->layer] || f > 16 || f % 4 != 0 || M > 64) return false;
    next.ypart = (float*)end->room.grad[end->layer];
    next.kind |= RowsNext::GRAD;
    next.H = H; next.ldh = ldh; next.M = M;
    return true;
}

void gradient_made(const RowsNext& next, int64_t n, int32_t f, float* Y) {
    epoch_end()->add(next.ypart, Y, next.M, f, (int)((n + 63) / 64), false);
}

// Whether Gprev (n rows of 16 floats) shares no memory with a matrix of n rows of 16 floats, `ld` apart, that the same kernel
// reads, or lies on it row by row: then a row is read and written by one wavefront, in that order.
static bool row_by_row(int64_t n, const float* Gprev, const float* M, int64_t ld) {
    return (M == Gprev && ld == 16) || M + (n - 1) * ld + 16 <= Gprev || Gprev + n * 16 <= M;
}

// Whether Gprev (n rows of M floats) shares no memory with a matrix of n rows of `cols` floats, `ld` apart.
static bool no_rows_shared(int64_t n, int32_t M, const float* Gprev, const float* other, int32_t cols, int64_t ld) {
    return other + (n - 1) * ld + cols <= Gprev || Gprev + n * M <= other;
}

// Gprev = (S W^T) masked by Zprev, Y = Hin^T S in one kernel, or *handled stays false: Hin 16, 32 or 64 wide, S up to as wide, rows of
// Hin, Zprev and Gprev 16-byte aligned.  It also
// stays false where Gprev lies across rows of an operand that another workgroup may not have read yet: the
// two products one after the other read all of Hin before they write Gprev.
int gemm_back_launch(int64_t n, int32_t f_in, int32_t f_out, const float* Hin, int64_t ldh, const float* S, const float* W,
                     const float* Zprev, float* Y, float* Gprev, bool few, hipStream_t s, bool* handled) {
    *handled = false;
    const bool wide = f_in != 16 || f_out != 16 || !al16(S);          // (k_gemm_back takes rows of S in whole pieces)
    if (n < 64 || ldh % 4 != 0 || !al16(Hin) || !al16(Zprev) || !al16(Gprev)) return GCN_OK;
    if (wide) {
        if ((f_in != 16 && f_in != 32 && f_in != 64) || f_out > f_in) return GCN_OK;
        if (!no_rows_shared(n, f_in, Gprev, Hin, f_in, ldh) || !no_rows_shared(n, f_in, Gprev, S, f_out, f_out) ||
            !no_rows_shared(n, f_in, Gprev, Zprev, f_in, f_in)) return GCN_OK;
        if (Y < W + f_in * f_out && W < Y + f_in * f_out) return GCN_OK;
    } else {
        if (!row_by_row(n, Gprev, Hin, ldh) || !row_by_row(n, Gprev, S, 16) || !row_by_row(n, Gprev, Zprev, 16)) return GCN_OK;
    }
    const TnShape g = tn_shape(f_in, f_out, n, few);
    EpochEnd* const end = epoch_end();
    ScratchLease lease;
    void* scratch = end ? end->room.grad[end->layer] : nullptr;
    const bool later = scratch != nullptr;
    if (!later) GCN_TRY(lease.get(&scratch, g.scratch_bytes, s));
    TnArgs args;
    args.K = n; args.M = f_in; args.N = f_out;
    args.A = Hin; args.lda = ldh; args.B = S; args.ldb = f_out;
    args.part = (float*)scratch; args.k_per_block = g.kpb;
    args.gw = args.rw = 1;
    const dim3 grid((unsigned)g.blocks);
    if (wide) {
        const int nt = (f_out + 15) / 16;
        if (f_in == 16) hipLaunchKernelGGL((k_gemm_back_wide<1, 1, 1>), grid, dim3(256), 0, s, args, W, Zprev, Gprev);
        else if (f_in == 32) {
            if (nt == 1) hipLaunchKernelGGL((k_gemm_back_wide<1, 2, 1>), grid, dim3(256), 0, s, args, W, Zprev, Gprev);
            else hipLaunchKernelGGL((k_gemm_back_wide<2, 2, 1>), grid, dim3(256), 0, s, args, W, Zprev, Gprev);
        } else {
            if (nt == 1) hipLaunchKernelGGL((k_gemm_back_wide<1, 2, 2>), grid, dim3(512), 0, s, args, W, Zprev, Gprev);
            else if (nt == 2) hipLaunchKernelGGL((k_gemm_back_wide<2, 2, 2>), grid, dim3(512), 0, s, args, W, Zprev, Gprev);
            else if (nt == 3) hipLaunchKernelGGL((k_gemm_back_wide<3, 2, 2>), grid, dim3(512), 0, s, args, W, Zprev, Gprev);
            else hipLaunchKernelGGL((k_gemm_back_wide<4, 2, 2>), grid, dim3(512), 0, s, args, W, Zprev, Gprev);
        }
    } else if (Zprev == Hin && ldh == 16) hipLaunchKernelGGL(k_gemm_back<true>, grid, dim3(256), 0, s, args, W, Zprev, Gprev);
    else hipLaunchKernelGGL(k_gemm_back<false>, grid, dim3(256), 0, s, args, W, Zprev, Gprev);
    GCN_LAUNCH_CHECK();
    const float* part = (const float*)scratch;
    int parts = (int)g.blocks;
    if (wide) part = folded(g, (int64_t)f_in * f_out, (float*)scratch, s, &parts);
    GCN_LAUNCH_CHECK();
    *handled = true;
    if (later) {
        end->add(part, Y, f_in, f_out, parts, false);
        return GCN_OK;
    }
    return reduce_parts_launch(f_in, f_out, parts, false, part, Y, f_out, nullptr, GCN_EPI_NONE, nullptr, 0, s);
}

}  // namespace gcn
