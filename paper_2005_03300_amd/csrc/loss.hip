// Last-layer activation and loss: row-wise log-softmax (the non-elementwise activation the paper
// discusses under "Block Two-Dimensional (2D) Algorithms", Equation H = sigma(Z)) with the mean
// negative log-likelihood over all vertices, and Equation 1 specialised to it:
//   G = (softmax(Z) - onehot(y)) / n.
// L lanes share a row and keep its logits in registers (four per lane, C <= 4 L): one read of Z,
// one write of G, 16 bytes per lane at any alignment, what is left of a ragged row one by one.  Bound by the instructions of the
// reductions where a row is short: with a column per lane a wavefront had one row of 41, now it has four (200 K rows: 44.7 -> 26.8
// us; 300 K rows of 130, three passes before, 232 -> 129 us), and of the exponentials: one per logit, whose share of the row's sum is the
// softmax (a second one, of z - lse, made 200 K rows of 41 25.2 us, now 21.9; 1 M 116 and 94; 120 K of 200 46.5 and 39.4; nearer to 64 bits too,
// G's error 6.5e-8 of its norm and 4.7e-8).  Row maxima and sums are butterfly reductions inside the L lanes.  Workgroups
// stride over the rows; every thread adds its rows' losses in double in a fixed order, then a
// fixed tree joins threads and workgroups, so the loss is reproducible bit for bit.
#include "common.h"
#include "sum_parts.h"

namespace gcn {

template <int L, bool RAGGED, int VEC = 4>
__global__ __launch_bounds__(256) void k_softmax_nll(int64_t n, int32_t C, const float* __restrict__ Z, int64_t ldz,
                                                     const int32_t* __restrict__ labels, float* __restrict__ G,
                                                     int64_t ldg, float inv_n, double* __restrict__ part) {
    static_assert(VEC == 4 || (VEC == 2 && L == 1 && RAGGED), "at most two classes");
    constexpr int ROWS = 256 / L, TAIL = VEC == 4 ? 3 : VEC;
    const int li = threadIdx.x % L;
    const int c0 = li * VEC;
    const bool whole = VEC == 4 && c0 + VEC <= C;
    double mine = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * ROWS + threadIdx.x / L; i < n; i += (int64_t)gridDim.x * ROWS) {
        const float* z = Z + i * ldz;
        float v[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (!RAGGED && whole) {
            const float4 t = *reinterpret_cast<const float4*>(z + c0);
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        } else if (whole) {
            const f4u t = *reinterpret_cast<const f4u*>(z + c0);
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        } else if constexpr (RAGGED) {
#pragma unroll
            for (int e = 0; e < TAIL; ++e)
                if (c0 + e < C) v[e] = z[c0 + e];
        }
        float m = v[0];
#pragma unroll
        for (int e = 1; e < VEC; ++e) m = fmaxf(m, v[e]);
#pragma unroll
        for (int d = L / 2; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
        float p[VEC], ssum = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            p[e] = expf(v[e] - m);                  // exp(-inf) = 0 for padding lanes
            ssum += p[e];
        }
#pragma unroll
        for (int d = L / 2; d >= 1; d >>= 1) ssum += __shfl_xor(ssum, d, 64);
        const float lse = m + logf(ssum);
        int32_t y = labels[i];
        const bool labelled = y >= 0;           // negative label: vertex outside the training split
        y = y < 0 ? 0 : (y >= C ? C - 1 : y);   // labels >= C are the caller's error; stay in bounds
        if (G && c0 < C) {
            float g[4] = {};
            const float inv = 1.f / ssum;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                g[e] = labelled ? (p[e] * inv - (c0 + e == y ? 1.f : 0.f)) * inv_n : 0.f;
            if (!RAGGED && whole) *reinterpret_cast<float4*>(G + i * ldg + c0) = make_float4(g[0], g[1], g[2], g[3]);
            else if (whole) *reinterpret_cast<f4u*>(G + i * ldg + c0) = f4u{g[0], g[1], g[2], g[3]};
            else if constexpr (RAGGED) {
#pragma unroll
                for (int e = 0; e < TAIL; ++e)
                    if (c0 + e < C) G[i * ldg + c0 + e] = g[e];
            }
        }
        // the lane that holds column y contributes lse - z_y
        float zy = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) zy = (c0 + e == y) ? v[e] : zy;
        if (labelled && y >= c0 && y < c0 + VEC) mine += (double)lse - (double)zy;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
    __shared__ double s_w[4];
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
}

// Any C: lanes loop over the columns and re-read the row (three passes, served by the caches), and take a second exponential: they do not hold the first.
__global__ __launch_bounds__(256) void k_softmax_nll_wide(int64_t n, int32_t C, const float* __restrict__ Z,
                                                          int64_t ldz, const int32_t* __restrict__ labels,
                                                          float* __restrict__ G, int64_t ldg, float inv_n,
                                                          double* __restrict__ part) {
    const int li = threadIdx.x & 63;
    double mine = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {
        const float* z = Z + i * ldz;
        float m = -INFINITY;
        for (int j = li; j < C; j += 64) m = fmaxf(m, z[j]);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
        float ssum = 0.f;
        for (int j = li; j < C; j += 64) ssum += expf(z[j] - m);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) ssum += __shfl_xor(ssum, d, 64);
        const float lse = m + logf(ssum);
        int32_t y = labels[i];
        const bool labelled = y >= 0;
        y = y < 0 ? 0 : (y >= C ? C - 1 : y);
        if (G) {
            float* g = G + i * ldg;
            for (int j = li; j < C; j += 64) g[j] = labelled ? (expf(z[j] - lse) - (j == y ? 1.f : 0.f)) * inv_n : 0.f;
        }
        if (li == 0 && labelled) mine += (double)lse - (double)z[y];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
    __shared__ double s_w[4];
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
}

__global__ __launch_bounds__(256) void k_loss_final(int64_t parts, const double* __restrict__ part, double inv_m,
                                                    float* __restrict__ loss) {
    __shared__ double s[256];
    sum_of_losses(part, parts, inv_m, loss, s);
}

template <int L>
static void launch_rows(int64_t blocks, int64_t n, int32_t C, const float* Z, int64_t ldz, const int32_t* labels,
                        float* G, int64_t ldg, double* part, float inv_m, hipStream_t s) {
    const bool aligned = (C % 4 == 0) && (ldz % 4 == 0) && (((uintptr_t)Z & 15u) == 0) &&
                         (!G || ((ldg % 4 == 0) && (((uintptr_t)G & 15u) == 0)));
    if (L == 1 && C <= 2) hipLaunchKernelGGL((k_softmax_nll<1, true, 2>), dim3((unsigned)blocks), dim3(256), 0, s, n, C, Z, ldz, labels, G, ldg, inv_m, part);
    else if (!aligned) hipLaunchKernelGGL((k_softmax_nll<L, true>), dim3((unsigned)blocks), dim3(256), 0, s, n, C, Z, ldz, labels, G, ldg, inv_m, part);
    else hipLaunchKernelGGL((k_softmax_nll<L, false>), dim3((unsigned)blocks), dim3(256), 0, s, n, C, Z, ldz, labels, G, ldg, inv_m, part);
}

static void dispatch_rows(int64_t n, int32_t C, const float* Z, int64_t ldz, const int32_t* labels,
                          float* G, int64_t ldg, double* part, int64_t* blocks_out, float inv_m, hipStream_t s) {
    const int64_t blocks = loss_blocks(n, C);
    *blocks_out = blocks;
    switch (loss_lanes(C)) {
        case 1: launch_rows<1>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        case 2: launch_rows<2>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        case 4: launch_rows<4>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        case 8: launch_rows<8>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        case 16: launch_rows<16>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        case 32: launch_rows<32>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
        default: launch_rows<64>(blocks, n, C, Z, ldz, labels, G, ldg, part, inv_m, s); break;
    }
}

RowsNext loss_next(int32_t C, int64_t parts, const int32_t* labels, int64_t n_labelled, float* G) {
    RowsNext next;
    const EpochEnd* const end = epoch_end();
    if (!end || C > 16 || C % 4 != 0 || parts > LOSS_BLOCKS_MAX) return next;
    next.part = (double*)end->room.loss;
    if (!next.part) return next;
    next.kind = RowsNext::LOSS;
    next.labels = labels;
    next.G = G;
    next.inv_m = 1.0f / (float)n_labelled;
    return next;
}

void loss_made(int64_t parts, int64_t n_labelled, float* loss) {
    EpochEnd* const end = epoch_end();
    end->args.lpart = (double*)end->room.loss;
    end->args.lparts = parts; end->args.inv_m = 1.0 / (double)n_labelled; end->args.loss = loss;
}

}  // namespace gcn

using namespace gcn;

static int softmax_nll_impl(int64_t n, int32_t C, const float* Z, int64_t ldz, const int32_t* labels, int64_t n_labelled,
                            float* loss, float* G, int64_t ldg, hipStream_t s) {
    EpochEnd* const end = epoch_end();
    ScratchLease lease;
    void* scratch = end ? end->room.loss : nullptr;
    const bool later = scratch != nullptr;
    if (!later) GCN_TRY(lease.get(&scratch, loss_scratch_bytes(), s));
    double* part = (double*)scratch;
    int64_t blocks = 0;
    const float inv_m = 1.0f / (float)n_labelled;
    if (C <= 256) {
        dispatch_rows(n, C, Z, ldz, labels, G, ldg, part, &blocks, inv_m, s);
    } else {
        blocks = loss_blocks(n, C);
        hipLaunchKernelGGL(k_softmax_nll_wide, dim3((unsigned)blocks), dim3(256), 0, s, n, C, Z, ldz, labels, G, ldg,
                           inv_m, part);
    }
    GCN_LAUNCH_CHECK();
    if (later) {
        end->args.lpart = part; end->args.lparts = blocks; end->args.inv_m = 1.0 / (double)n_labelled; end->args.loss = loss;
        return GCN_OK;
    }
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, blocks, (const double*)part, 1.0 / (double)n_labelled, loss);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

extern "C" int gcn_softmax_nll(int64_t n, int32_t C, const float* Z, int64_t ldz, const int32_t* labels, float* loss,
                               float* G, int64_t ldg, void* stream) {
    if (!Z || !labels || !loss) return fail(GCN_ERR_BADARG, "gcn_softmax_nll: NULL argument");
    if (n <= 0 || C <= 0 || ldz < C || (G && ldg < C)) return fail(GCN_ERR_BADARG, "gcn_softmax_nll: bad size");
    return softmax_nll_impl(n, C, Z, ldz, labels, n, loss, G, ldg, (hipStream_t)stream);
}

extern "C" int gcn_softmax_nll_masked(int64_t n, int32_t C, const float* Z, int64_t ldz, const int32_t* labels,
                                      int64_t n_labelled, float* loss, float* G, int64_t ldg, void* stream) {
    if (!Z || !labels || !loss) return fail(GCN_ERR_BADARG, "gcn_softmax_nll_masked: NULL argument");
    if (n <= 0 || C <= 0 || ldz < C || (G && ldg < C)) return fail(GCN_ERR_BADARG, "gcn_softmax_nll_masked: bad size");
    if (n_labelled <= 0 || n_labelled > n) return fail(GCN_ERR_BADARG, "gcn_softmax_nll_masked: n_labelled must be in [1, n]");
    return softmax_nll_impl(n, C, Z, ldz, labels, n_labelled, loss, G, ldg, (hipStream_t)stream);
}
