// Device functions that add up the partial results of reductions over the vertices, for the kernels that do it one reduction at a
// time and for the one that does it for a whole epoch.  Workgroups of up to 1024 threads; every sum has a fixed order.
#pragma once
#include "common.h"

namespace gcn {

union SumLds {
    float s[16][64];
    float y[64][16];
    double l[256];
};

// Sum of part[p * count] over p = first, first + step, ... below parts, in ascending order; the loads of eight terms
// are in flight together (the additions are a serial chain, the loads need not be), and so are the last of them: with 64 partial results and 16
// wavefronts there are no others (one after another: epoch of 64-16-8 on 4096 vertices 35.0 us, now 34.4; 1000 x 1000 over 1000 rows 90 us, now 80).
// Where a term is not there nothing is loaded for it, and a single term goes first: large results have many workgroups, and few terms each (1000 x 1000
// over 600 rows, a layer call: with the first of the last terms loaded in place of those that are not there 126 us, one after another 118, now 119).
__device__ __forceinline__ float strided_sum(const float* __restrict__ part, int64_t count, int first, int step, int parts) {
    if (first + step >= parts) return first < parts ? 0.f + part[(int64_t)first * count] : 0.f;
    float s = 0.f;
    int p = first;
    for (; p + 7 * step < parts; p += 8 * step) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = part[(int64_t)(p + e * step) * count];
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[e];
    }
    if (p < parts) {                                            // the last ones too: few partial results have no others
        float v[7] = {};
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (p + e * step < parts) v[e] = part[(int64_t)(p + e * step) * count];
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (p + e * step < parts) s += v[e];
    }
    return s;
}

// `group` of 64 results: wavefront w of `waves` sums the partial results w, w + waves, ... in ascending order, the wavefronts are added in order.
// `transposed` means that a partial result is N x M row-major.  store(m, n, sum)
template <typename Store>
__device__ __forceinline__ void sum_of_parts(int group, int32_t M, int32_t N, int parts, int transposed, const float* __restrict__ part,
                                             int waves, float (&s_sum)[16][64], Store store) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t count = (int64_t)M * N;
    const int64_t src = (int64_t)group * 64 + lane;
    if (src < count && wave < waves) s_sum[wave][lane] = strided_sum(part + src, count, wave, waves, parts);
    __syncthreads();
    if (wave != 0 || src >= count) return;
    float s = s_sum[0][lane];
    for (int w = 1; w < waves; ++w) s += s_sum[w][lane];
    store((int)(transposed ? src % M : src / N), (int)(transposed ? src / M : src % N), s);
}

// `group` of 16 numbers of the fused last layer's weight gradient, 16 x C out of 16 x CP: a partial result each for the 64 groups
// of threads, eight of them in flight (one after another, as the compiler left them, 64 waits for memory made 24 us of 2048
// partial results of 512 numbers), every group's sum, then the 64 of them in pairs.  store(index, sum)
template <typename Store>
__device__ __forceinline__ void sum_of_fused(int group, int C, int CP, int blocks, const float* __restrict__ part, float (&s_y)[64][16],
                                             Store store) {
    constexpr int GROUPS = 64, AHEAD = 8;
    const int i = threadIdx.x % 16, j = threadIdx.x / 16;
    const int e = group * 16 + i;                               // of 16 CP numbers
    const size_t count = (size_t)16 * CP;
    const float* p = part + e;
    float acc = 0.f;
    int b = j;
    for (; b + (AHEAD - 1) * GROUPS < blocks; b += AHEAD * GROUPS) {
        float x[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) x[u] = p[(size_t)(b + u * GROUPS) * count];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) acc += x[u];
    }
    if (b < blocks) {
        float x[AHEAD - 1] = {};
#pragma unroll
        for (int u = 0; u < AHEAD - 1; ++u)
            if (b + u * GROUPS < blocks) x[u] = p[(size_t)(b + u * GROUPS) * count];
#pragma unroll
        for (int u = 0; u < AHEAD - 1; ++u)
            if (b + u * GROUPS < blocks) acc += x[u];
    }
    s_y[j][i] = acc;
    __syncthreads();
    for (int d = GROUPS / 2; d >= 1; d >>= 1) {
        if (j < d) s_y[j][i] += s_y[j + d][i];
        __syncthreads();
    }
    const int k = e / CP, c = e % CP;
    if (j == 0 && c < C) store(k * C + c, s_y[0][i]);
}

// The loss: strided sums of 256 threads, then a fixed tree.  Eight terms of a thread are in flight together, but one or two are added as they come: the code for
// eight took a small loss 0.3 us (loss of 800 rows of 300 classes 7.2 us with it, 6.9 without; 8000 of 8, 63 terms in all, 4.8 and 4.5).
__device__ __forceinline__ void sum_of_losses(const double* __restrict__ part, int64_t parts, double inv_m, float* __restrict__ loss,
                                              double (&s)[256]) {
    if (threadIdx.x < 256) {
        double acc = 0.0;
        if (parts <= 512) {
            for (int64_t p = threadIdx.x; p < parts; p += 256) acc += part[p];
        } else {
            for (int64_t p = threadIdx.x; p < parts; p += 8 * 256) {    // (up to 2048: all of them on their way at once)
                double v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = part[p + e * 256 < parts ? p + e * 256 : p];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (p + e * 256 < parts) acc += v[e];
            }
        }
        s[threadIdx.x] = acc;
    }
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) s[threadIdx.x] += s[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(s[0] * inv_m);
}

}  // namespace gcn
