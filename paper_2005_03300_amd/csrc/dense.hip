// Dense products and element-wise kernels around the SpMM: H W of "Forward Propagation", S W^T of
// Equation 2, the weight gradient H^T S of Equation 3, ReLU and its derivative mask, column sums
// for an optional bias gradient, and the gradient step.
#include "common.h"

namespace gcn {

template <int EPI>
__device__ __forceinline__ float apply_epi(float v, const float* zprev_elem) {
    if (EPI == GCN_EPI_RELU) return v > 0.f ? v : 0.f;
    if (EPI == GCN_EPI_MASK) return *zprev_elem > 0.f ? v : 0.f;
    return v;
}

// ---- generic fallback: one thread per output element (any shape, any leading dimension) ----
template <int EPI>
__global__ void k_gemm_naive(int tb, int64_t M, int64_t N, int64_t K, const float* __restrict__ A, int64_t lda,
                             const float* __restrict__ B, int64_t ldb, float* __restrict__ C, int64_t ldc,
                             const float* __restrict__ bias, const float* __restrict__ Zprev, int64_t ldzprev) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / N, j = t % N;
    if (i >= M) return;
    float acc = 0.f;
    if (tb) for (int64_t k = 0; k < K; ++k) acc = fmaf(A[i * lda + k], B[j * ldb + k], acc);
    else for (int64_t k = 0; k < K; ++k) acc = fmaf(A[i * lda + k], B[k * ldb + j], acc);
    if (bias) acc += bias[j];
    C[i * ldc + j] = apply_epi<EPI>(acc, EPI == GCN_EPI_MASK ? Zprev + i * ldzprev + j : nullptr);
}

// ---- element-wise -----------------------------------------------------------------------------
// ReLU, and with M the derivative mask, over rows x cols with leading dimensions.  Dense operands come as one row: 16
// bytes per thread; the others as one thread per element.
__global__ __launch_bounds__(256) void k_relu_dense(int64_t total, const float* X, const float* M, float* out) {
    const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (t + 4 <= total) {
        const float4 x = *reinterpret_cast<const float4*>(X + t);
        const float4 m = *reinterpret_cast<const float4*>(M + t);
        *reinterpret_cast<float4*>(out + t) =
            make_float4(m.x > 0.f ? x.x : 0.f, m.y > 0.f ? x.y : 0.f, m.z > 0.f ? x.z : 0.f, m.w > 0.f ? x.w : 0.f);
    } else {
        for (int64_t e = t; e < total; ++e) out[e] = M[e] > 0.f ? X[e] : 0.f;
    }
}

__global__ void k_relu_mask(int64_t rows, int32_t cols, const float* G, int64_t ldg, const float* Zp, int64_t ldzp, float* out,
                            int64_t ldo) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / cols;
    const int j = (int)(t % cols);
    if (i >= rows) return;
    out[i * ldo + j] = Zp[i * ldzp + j] > 0.f ? G[i * ldg + j] : 0.f;
}

// Column sums: blockDim.x lanes walk the columns (64 or the next power of two above `cols` when that is less),
// blockDim.y row sets split the workgroup's rows, eight loads in flight each; the row sets are added in order in LDS.
__global__ __launch_bounds__(256) void k_colsum_partial(int64_t rows, int32_t cols, int64_t rows_per_block,
                                                        const float* __restrict__ G, int64_t ldg, float* __restrict__ part) {
    __shared__ float s_sum[256];
    const int64_t rb = (int64_t)blockIdx.x * rows_per_block;
    const int64_t re = rb + rows_per_block < rows ? rb + rows_per_block : rows;
    const int j = blockIdx.y * blockDim.x + threadIdx.x;
    const int ty = threadIdx.y, ny = blockDim.y;
    float acc = 0.f;
    if (j < cols) {
        int64_t i = rb + ty;
        for (; i + 7 * ny < re; i += 8 * ny) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = G[(i + e * ny) * ldg + j];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += v[e];
        }
        for (; i < re; i += ny) acc += G[i * ldg + j];
    }
    s_sum[ty * blockDim.x + threadIdx.x] = acc;
    __syncthreads();
    if (ty != 0 || j >= cols) return;
    for (int y = 1; y < ny; ++y) acc += s_sum[y * blockDim.x + threadIdx.x];
    part[(int64_t)blockIdx.x * cols + j] = acc;
}

// Z += 1 bias^T over dense rows, as one run of rows * cols floats, 16 bytes per thread and step.  The stride of a thread is a
// multiple of the row length (the launch picks it so), so its four columns and their biases stay the same: no division
// in the loop.  Bound by memory (200 K x 64 with H: 154 MB; bias and ReLU in two passes took 50 us).
__global__ __launch_bounds__(256) void k_bias_add(int64_t total, int32_t cols, int64_t stride, float* __restrict__ Z,
                                                  const float* __restrict__ bias, int relu, float* __restrict__ H) {
    const int64_t t0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (t0 >= stride) return;
    float b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = bias[(t0 + e) % cols];
    for (int64_t t = t0; t < total; t += stride) {
        if (t + 4 <= total) {
            float4 v = *reinterpret_cast<float4*>(Z + t);
            v.x += b[0]; v.y += b[1]; v.z += b[2]; v.w += b[3];
            const float4 r = make_float4(v.x > 0.f ? v.x : 0.f, v.y > 0.f ? v.y : 0.f, v.z > 0.f ? v.z : 0.f, v.w > 0.f ? v.w : 0.f);
            *reinterpret_cast<float4*>(Z + t) = relu ? r : v;
            if (H) *reinterpret_cast<float4*>(H + t) = r;
        } else {
            for (int e = 0; t + e < total; ++e) {
                const float v = Z[t + e] + b[e], r = v > 0.f ? v : 0.f;
                Z[t + e] = relu ? r : v;
                if (H) H[t + e] = r;
            }
        }
    }
}

// Any alignment.
__global__ void k_bias_add_plain(int64_t total, int32_t cols, float* __restrict__ Z, const float* __restrict__ bias, int relu,
                                 float* __restrict__ H) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const float v = Z[t] + bias[t % cols], r = v > 0.f ? v : 0.f;
    Z[t] = relu ? r : v;
    if (H) H[t] = r;
}

// Y[i,:] = scale[i] * X[i,:]; 16 bytes per thread when the layout allows it.
template <int VEC>
__global__ __launch_bounds__(256) void k_scale_rows(int64_t rows, int32_t lanes, const float* __restrict__ X, int64_t ldx,
                                                    const float* __restrict__ scale, float* __restrict__ Y, int64_t ldy) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / lanes;
    const int j = (int)(t % lanes) * VEC;
    if (i >= rows) return;
    const float sc = scale[i];
    if constexpr (VEC == 4) {
        float4 v = *reinterpret_cast<const float4*>(X + i * ldx + j);
        v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
        *reinterpret_cast<float4*>(Y + i * ldy + j) = v;
    } else {
        Y[i * ldy + j] = sc * X[i * ldx + j];
    }
}

// out[i] = (float)(1 / sqrt((double)deg[i])), 0 for an empty row.
__global__ void k_inv_sqrt_deg(int64_t n, const int32_t* __restrict__ deg, float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = deg[i] > 0 ? (float)__ddiv_rn(1.0, __dsqrt_rn((double)deg[i])) : 0.f;
}

// W = W - lr Y of several layers, a layer per y.  The matrices are a few thousand numbers each, so a launch is what the update
// costs (4.6 us between large kernels): one for all of them.
struct UpdateArgs {
    static constexpr int LAYERS = 16;
    int64_t count[LAYERS];
    float* W[LAYERS];
    const float* Y[LAYERS];
};
__global__ void k_update(UpdateArgs a, float lr) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float* const W = a.W[blockIdx.y];
    if (t < a.count[blockIdx.y]) W[t] = W[t] - lr * a.Y[blockIdx.y][t];
}

static inline unsigned nblocks(int64_t work) { return (unsigned)((work + 255) / 256 > 0 ? (work + 255) / 256 : 1); }

int gemm_mfma_launch(int ta, int tb, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                     int64_t ldb, float* C, int64_t ldc, const float* bias, int epilogue, const float* Zprev,
                     int64_t ldzprev, hipStream_t s, bool* handled, const float* row_scale, bool* scaled, bool few);

int reduce_parts_launch(int32_t M, int32_t N, int parts, bool transposed, const float* part, float* C, int64_t ldc,
                        const float* bias, int epilogue, const float* Zprev, int64_t ldzprev, hipStream_t s);

static void colsum_split(int64_t rows, int64_t* parts_out, int64_t* rpb_out) {
    int64_t parts = (rows + 127) / 128;
    if (parts > 1024) parts = 1024;
    if (parts < 1) parts = 1;
    const int64_t rpb = (rows + parts - 1) / parts;
    *parts_out = (rows + rpb - 1) / rpb;
    *rpb_out = rpb;
}

size_t colsum_scratch_bytes(int64_t rows, int32_t cols) {
    int64_t parts = 0, rpb = 0;
    colsum_split(rows, &parts, &rpb);
    return (size_t)parts * cols * sizeof(float);
}

int gemm_launch(int ta, int tb, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                int64_t ldb, float* C, int64_t ldc, const float* bias, int epilogue, const float* Zprev,
                int64_t ldzprev, hipStream_t s, const float* row_scale, bool few) {
    bool handled = false, scaled = false;
    GCN_TRY(gemm_mfma_launch(ta, tb, M, N, K, A, lda, B, ldb, C, ldc, bias, epilogue, Zprev, ldzprev, s, &handled,
                             row_scale, &scaled, few));
    // kernels without a scaling store path leave the row factors to a pass of their own
    auto finish = [&]() { return (row_scale && !scaled) ? scale_rows_launch(M, (int32_t)N, C, ldc, row_scale, C, ldc, s) : (int)GCN_OK; };
    if (handled) return finish();
    const int64_t work = M * N;
    if ((work + 255) / 256 >= (1ll << 31)) return fail(GCN_ERR_RANGE, "gcn_gemm: output too large");
    switch (epilogue) {
        case GCN_EPI_NONE: hipLaunchKernelGGL(k_gemm_naive<GCN_EPI_NONE>, dim3(nblocks(work)), dim3(256), 0, s, tb, M, N, K, A, lda, B, ldb, C, ldc, bias, Zprev, ldzprev); break;
        case GCN_EPI_RELU: hipLaunchKernelGGL(k_gemm_naive<GCN_EPI_RELU>, dim3(nblocks(work)), dim3(256), 0, s, tb, M, N, K, A, lda, B, ldb, C, ldc, bias, Zprev, ldzprev); break;
        default: hipLaunchKernelGGL(k_gemm_naive<GCN_EPI_MASK>, dim3(nblocks(work)), dim3(256), 0, s, tb, M, N, K, A, lda, B, ldb, C, ldc, bias, Zprev, ldzprev); break;
    }
    GCN_LAUNCH_CHECK();
    return finish();
}

int colsum_launch(int64_t rows, int32_t cols, const float* G, int64_t ldg, float* out, hipStream_t s) {
    int64_t parts = 0, rpb = 0;
    colsum_split(rows, &parts, &rpb);
    EpochEnd* const end = epoch_end();
    ScratchLease lease;
    void* scratch = end ? end->room.bias : nullptr;
    const bool later = scratch != nullptr;
    if (!later) GCN_TRY(lease.get(&scratch, (size_t)parts * cols * sizeof(float), s));
    int tx = 64;
    while (tx > 4 && tx / 2 >= cols) tx /= 2;
    hipLaunchKernelGGL(k_colsum_partial, dim3((unsigned)parts, (unsigned)((cols + tx - 1) / tx)), dim3(tx, 256 / tx), 0, s, rows,
                       cols, rpb, G, ldg, (float*)scratch);
    GCN_LAUNCH_CHECK();
    if (later) {
        end->add((const float*)scratch, out, 1, cols, (int)parts, false);
        return GCN_OK;
    }
    return reduce_parts_launch(1, cols, (int)parts, false, (const float*)scratch, out, cols, nullptr, GCN_EPI_NONE, nullptr, 0, s);
}

static int relu_mask_launch(int64_t rows, int32_t cols, const float* G, int64_t ldg, const float* Zprev, int64_t ldzprev,
                            float* out, int64_t ldo, hipStream_t s) {
    const bool dense = (ldg == cols && ldzprev == cols && ldo == cols) || rows == 1;
    if (dense && (((uintptr_t)G | (uintptr_t)Zprev | (uintptr_t)out) & 15u) == 0)
        hipLaunchKernelGGL(k_relu_dense, dim3(nblocks((rows * cols + 3) / 4)), dim3(256), 0, s, rows * cols, G, Zprev, out);
    else
        hipLaunchKernelGGL(k_relu_mask, dim3(nblocks(rows * cols)), dim3(256), 0, s, rows, cols, G, ldg, Zprev, ldzprev, out, ldo);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// max(Z, 0) is Z where Z is positive, 0 elsewhere
int relu_launch(int64_t rows, int32_t cols, const float* Z, int64_t ldz, float* H, int64_t ldh, hipStream_t s) {
    return relu_mask_launch(rows, cols, Z, ldz, Z, ldz, H, ldh, s);
}

int bias_add_launch(int64_t rows, int32_t cols, float* Z, const float* bias, int relu, float* H, hipStream_t s) {
    const int64_t total = rows * cols;
    if ((((uintptr_t)Z | (uintptr_t)H) & 15u) == 0) {
        // about 2 M floats per step of the grid (8192 wavefronts), rounded up to whole rows in whole 16-byte pieces
        const int64_t unit = cols % 4 == 0 ? cols : (cols % 2 == 0 ? 2 * (int64_t)cols : 4 * (int64_t)cols);
        const int64_t want = total < (2ll << 20) ? total : (2ll << 20);
        const int64_t stride = (want + unit - 1) / unit * unit;
        hipLaunchKernelGGL(k_bias_add, dim3(nblocks((stride + 3) / 4)), dim3(256), 0, s, total, cols, stride, Z, bias, relu, H);
    } else {
        hipLaunchKernelGGL(k_bias_add_plain, dim3(nblocks(total)), dim3(256), 0, s, total, cols, Z, bias, relu, H);
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

int scale_rows_launch(int64_t rows, int32_t cols, const float* X, int64_t ldx, const float* scale, float* Y, int64_t ldy,
                      hipStream_t s) {
    const bool vec4 = (cols % 4 == 0) && (ldx % 4 == 0) && (ldy % 4 == 0) && (((uintptr_t)X & 15u) == 0) &&
                      (((uintptr_t)Y & 15u) == 0);
    if (vec4) {
        const int lanes = cols / 4;
        hipLaunchKernelGGL(k_scale_rows<4>, dim3(nblocks(rows * lanes)), dim3(256), 0, s, rows, lanes, X, ldx, scale, Y, ldy);
    } else {
        hipLaunchKernelGGL(k_scale_rows<1>, dim3(nblocks(rows * cols)), dim3(256), 0, s, rows, cols, X, ldx, scale, Y, ldy);
    }
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

int inv_sqrt_deg_launch(int64_t n, const int32_t* deg, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_inv_sqrt_deg, dim3(nblocks(n)), dim3(256), 0, s, n, deg, out);
    GCN_LAUNCH_CHECK();
    return GCN_OK;
}

// The layers in turn, those of a launch side by side: a layer whose W is also the W or the Y of another one in the launch (tied
// weights) starts the next launch.
int update_launch(int32_t L, const int32_t* dims, float* const* W, float* const* Y, float lr, hipStream_t s) {
    auto meet = [](const float* p, int64_t np, const float* q, int64_t nq) { return p < q + nq && q < p + np; };
    for (int l = 0; l < L;) {
        UpdateArgs a;
        int k = 0;
        int64_t most = 0;
        for (; l < L && k < UpdateArgs::LAYERS; ++l, ++k) {
            const int64_t count = (int64_t)dims[l] * dims[l + 1];
            bool apart = true;
            for (int j = 0; j < k; ++j)
                apart = apart && !meet(W[l], count, a.W[j], a.count[j]) && !meet(W[l], count, a.Y[j], a.count[j]) &&
                        !meet(Y[l], count, a.W[j], a.count[j]);
            if (!apart) break;
            a.count[k] = count; a.W[k] = W[l]; a.Y[k] = Y[l];
            most = count > most ? count : most;
        }
        hipLaunchKernelGGL(k_update, dim3(nblocks(most), (unsigned)k), dim3(256), 0, s, a, lr);
        GCN_LAUNCH_CHECK();
    }
    return GCN_OK;
}

}  // namespace gcn

using namespace gcn;

extern "C" {

int gcn_gemm(int ta, int tb, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
             int64_t ldb, float* C, int64_t ldc, const float* bias, int epilogue, const float* Zprev,
             int64_t ldzprev, void* stream) {
    if (!A || !B || !C) return fail(GCN_ERR_BADARG, "gcn_gemm: NULL matrix");
    if (M <= 0 || N <= 0 || K <= 0) return fail(GCN_ERR_BADARG, "gcn_gemm: sizes must be positive");
    if (ta && tb) return fail(GCN_ERR_BADARG, "gcn_gemm: ta and tb together are not supported");
    if (lda < (ta ? M : K) || ldb < (tb ? K : N) || ldc < N) return fail(GCN_ERR_BADARG, "gcn_gemm: leading dimension too small");
    if (epilogue < GCN_EPI_NONE || epilogue > GCN_EPI_MASK) return fail(GCN_ERR_BADARG, "gcn_gemm: unknown epilogue");
    if (epilogue == GCN_EPI_MASK && (!Zprev || ldzprev < N)) return fail(GCN_ERR_BADARG, "gcn_gemm: mask epilogue needs Zprev with ld >= N");
    return gemm_launch(ta, tb, M, N, K, A, lda, B, ldb, C, ldc, bias, epilogue, Zprev, ldzprev, (hipStream_t)stream, nullptr, ta && few_rows_alone(M, N, K));
}

int gcn_relu(int64_t rows, int32_t cols, const float* Z, int64_t ldz, float* H, int64_t ldh, void* stream) {
    if (!Z || !H || rows <= 0 || cols <= 0 || ldz < cols || ldh < cols) return fail(GCN_ERR_BADARG, "gcn_relu: bad argument");
    return relu_launch(rows, cols, Z, ldz, H, ldh, (hipStream_t)stream);
}

int gcn_relu_mask(int64_t rows, int32_t cols, const float* G, int64_t ldg, const float* Zprev, int64_t ldzprev,
                  float* out, int64_t ldo, void* stream) {
    if (!G || !Zprev || !out || rows <= 0 || cols <= 0 || ldg < cols || ldzprev < cols || ldo < cols)
        return fail(GCN_ERR_BADARG, "gcn_relu_mask: bad argument");
    return relu_mask_launch(rows, cols, G, ldg, Zprev, ldzprev, out, ldo, (hipStream_t)stream);
}

int gcn_scale_rows(int64_t rows, int32_t cols, const float* X, int64_t ldx, const float* scale, float* Y, int64_t ldy,
                   void* stream) {
    if (!X || !scale || !Y || rows <= 0 || cols <= 0 || ldx < cols || ldy < cols)
        return fail(GCN_ERR_BADARG, "gcn_scale_rows: bad argument");
    return scale_rows_launch(rows, cols, X, ldx, scale, Y, ldy, (hipStream_t)stream);
}

int gcn_csr_inv_sqrt_degrees(const gcn_csr* a, float* out, void* stream) {
    if (!a || !out) return fail(GCN_ERR_BADARG, "gcn_csr_inv_sqrt_degrees: NULL argument");
    if (a->n != a->ncols) return fail(GCN_ERR_BADARG, "gcn_csr_inv_sqrt_degrees: the matrix must be square");
    return inv_sqrt_deg_launch(a->n, a->deg, out, (hipStream_t)stream);
}

}  // extern "C"
