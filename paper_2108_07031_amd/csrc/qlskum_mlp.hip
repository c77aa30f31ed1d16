// Warm-start network kernels for gfx950: a multilayer perceptron
//   a_0 = x,  z_l = a_{l-1} W_l + b_l,  a_l = tanh(z_l) (hidden),  y = z_L
// evaluated and trained with bfloat16 operands on the matrix cores
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation); bias, tanh, loss, the
// gradient sums and Adam in FP32.
//
// Product kernel: one wavefront computes one 16 x 16 block of
// C = op(A) op(B) (M x N, inner dimension K) in steps of 32 along K.  With
// the gfx950 16x16x32 layout, lane l holds
//   A[row l%16][k 8(l/16) .. 8(l/16)+7],  B[k 8(l/16) .. +7][col l%16],
//   C[rows 4(l/16) .. 4(l/16)+3][col l%16].
// Operands are addressed through (pointer, leading dimension, transposed):
// element (r, k) of op(P) is P[r*ld + k] (k contiguous) or P[k*ld + r].
#include "qlskum_mlp_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace ql {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;  // wavefronts (output blocks) per workgroup

// 8 consecutive-k elements of row r of op(P), zero outside r < R, k < K
template <bool KCONTIG>
__device__ __forceinline__ bf16x8 load_frag(const bf16 *__restrict__ P, int ld, int r, int k0,
                                            int R, int K) {
    bf16x8 v;
    if (KCONTIG && r < R && k0 + 8 <= K && (ld & 7) == 0) {
        v = *reinterpret_cast<const bf16x8 *>(P + (size_t)r * ld + k0);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k0 + i;
            v[i] = (r < R && k < K) ? P[KCONTIG ? (size_t)r * ld + k : (size_t)k * ld + r]
                                    : (bf16)0.0f;
        }
    }
    return v;
}

}  // namespace

// C = op(A) op(B) with an epilogue:
//   kEpiStore     C32[m, n] = acc
//   kEpiBias      C32[m, n] = acc + bias[n]
//   kEpiBiasTanh  C16[m, n] = bf16(tanh(acc + bias[n]))
//   kEpiTanhGrad  C16[m, n] = bf16(acc * (1 - a^2)),  a = act[m, n] (bf16)
// A_KC: element (m, k) of op(A) is A[m*lda + k] (else A[k*lda + m]);
// B_NC: element (k, n) of op(B) is B[n*ldb + k] (else B[k*ldb + n]).
template <bool A_KC, bool B_NC, int EPI>
__global__ void __launch_bounds__(64 * kWaves)
    k_mfma_gemm(int M, int N, int K, const bf16 *__restrict__ A, int lda,
                const bf16 *__restrict__ B, int ldb, const float *__restrict__ bias,
                const bf16 *__restrict__ act, float *__restrict__ C32, bf16 *__restrict__ C16,
                int ldc) {
    const int lane = threadIdx.x & 63;
    const int tile = blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int ntn = (N + 15) / 16;
    const int ntiles = ((M + 15) / 16) * ntn;
    if (tile >= ntiles) return;  // whole wavefront leaves together
    const int tm = tile / ntn, tn = tile % ntn;
    const int r = tm * 16 + (lane & 15);  // row of op(A) this lane loads
    const int c = tn * 16 + (lane & 15);  // column of op(B) this lane loads
    const int kq = 8 * (lane >> 4);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        const bf16x8 a = load_frag<A_KC>(A, lda, r, k0 + kq, M, K);
        const bf16x8 b = load_frag<B_NC>(B, ldb, c, k0 + kq, N, K);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    const int n = tn * 16 + (lane & 15);
    if (n >= N) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = tm * 16 + 4 * (lane >> 4) + i;
        if (m >= M) continue;
        const size_t o = (size_t)m * ldc + n;
        const float v = acc[i];
        if (EPI == kEpiStore) {
            C32[o] = v;
        } else if (EPI == kEpiBias) {
            C32[o] = v + bias[n];
        } else if (EPI == kEpiBiasTanh) {
            C16[o] = (bf16)tanhf(v + bias[n]);
        } else {
            const float a = (float)act[o];
            C16[o] = (bf16)(v * (1.0f - a * a));
        }
    }
}

hipError_t launch_mfma_gemm(hipStream_t st, int epi, bool a_kc, bool b_nc, int M, int N, int K,
                            const bf16 *A, int lda, const bf16 *B, int ldb, const float *bias,
                            const bf16 *act, float *C32, bf16 *C16, int ldc) {
    const int tiles = ((M + 15) / 16) * ((N + 15) / 16);
    if (tiles == 0) return hipSuccess;
    const dim3 grid((tiles + kWaves - 1) / kWaves), block(64 * kWaves);
#define QL_GEMM(AK, BN, E)                                                                 \
    hipLaunchKernelGGL((k_mfma_gemm<AK, BN, E>), grid, block, 0, st, M, N, K, A, lda, B, ldb, \
                       bias, act, C32, C16, ldc)
#define QL_GEMM_EPI(AK, BN)                                    \
    switch (epi) {                                             \
    case kEpiStore: QL_GEMM(AK, BN, kEpiStore); break;         \
    case kEpiBias: QL_GEMM(AK, BN, kEpiBias); break;           \
    case kEpiBiasTanh: QL_GEMM(AK, BN, kEpiBiasTanh); break;   \
    default: QL_GEMM(AK, BN, kEpiTanhGrad); break;             \
    }
    if (a_kc && b_nc) { QL_GEMM_EPI(true, true) }
    else if (a_kc) { QL_GEMM_EPI(true, false) }
    else if (b_nc) { QL_GEMM_EPI(false, true) }
    else { QL_GEMM_EPI(false, false) }
#undef QL_GEMM_EPI
#undef QL_GEMM
    return hipGetLastError();
}

// Split-K form of the plain product (kEpiStore) for few output blocks and a
// long inner dimension -- the weight gradients a^T d, whose inner dimension
// is the batch: wavefront (slice, block) sums one 16 x 16 block over the
// kslice-long slice of K into part[slice][M][N], and k_gemm_reduce adds the
// slices in slice order (a fixed order: results do not depend on timing).
template <bool A_KC, bool B_NC>
__global__ void __launch_bounds__(64 * kWaves)
    k_mfma_gemm_splitk(int M, int N, int K, int kslice, const bf16 *__restrict__ A, int lda,
                       const bf16 *__restrict__ B, int ldb, float *__restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int item = blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int ntn = (N + 15) / 16;
    const int ntiles = ((M + 15) / 16) * ntn;
    const int nsl = (K + kslice - 1) / kslice;
    if (item >= ntiles * nsl) return;  // whole wavefront leaves together
    const int sl = item / ntiles, tile = item % ntiles;
    const int tm = tile / ntn, tn = tile % ntn;
    const int r = tm * 16 + (lane & 15);
    const int c = tn * 16 + (lane & 15);
    const int kq = 8 * (lane >> 4);
    const int kb = sl * kslice, ke = min(K, kb + kslice);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = kb; k0 < ke; k0 += 32) {
        const bf16x8 a = load_frag<A_KC>(A, lda, r, k0 + kq, M, ke);
        const bf16x8 b = load_frag<B_NC>(B, ldb, c, k0 + kq, N, ke);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    const int n = tn * 16 + (lane & 15);
    if (n >= N) return;
    float *P = part + (size_t)sl * M * N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = tm * 16 + 4 * (lane >> 4) + i;
        if (m < M) P[(size_t)m * N + n] = acc[i];
    }
}

__global__ void __launch_bounds__(256) k_gemm_reduce(int M, int N, int nsl,
                                                     const float *__restrict__ part,
                                                     float *__restrict__ C, int ldc) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= M * N) return;
    float s = 0.0f;
    for (int sl = 0; sl < nsl; ++sl) s += part[(size_t)sl * M * N + idx];
    C[(size_t)(idx / N) * ldc + idx % N] = s;
}

int gemm_splitk_slices(int M, int N, int K) {
    const int tiles = ((M + 15) / 16) * ((N + 15) / 16);
    if (tiles == 0 || tiles > kSplitKMaxTiles || K < 2 * kSplitKSlice) return 1;
    return std::min(kSplitKMaxSlices, (K + kSplitKSlice - 1) / kSplitKSlice);
}

hipError_t launch_mfma_gemm_splitk(hipStream_t st, bool a_kc, bool b_nc, int M, int N, int K,
                                   const bf16 *A, int lda, const bf16 *B, int ldb, float *part,
                                   float *C32, int ldc) {
    const int nsl = gemm_splitk_slices(M, N, K);
    if (nsl <= 1)
        return launch_mfma_gemm(st, kEpiStore, a_kc, b_nc, M, N, K, A, lda, B, ldb, nullptr,
                                nullptr, C32, nullptr, ldc);
    // slices of a whole number of 32-deep steps, nsl of them covering K
    const int kslice = ((K + nsl - 1) / nsl + 31) / 32 * 32;
    const int nsl_used = (K + kslice - 1) / kslice;
    const int items = ((M + 15) / 16) * ((N + 15) / 16) * nsl_used;
    const dim3 grid((items + kWaves - 1) / kWaves), block(64 * kWaves);
    if (a_kc && b_nc)
        hipLaunchKernelGGL((k_mfma_gemm_splitk<true, true>), grid, block, 0, st, M, N, K, kslice,
                           A, lda, B, ldb, part);
    else if (a_kc)
        hipLaunchKernelGGL((k_mfma_gemm_splitk<true, false>), grid, block, 0, st, M, N, K, kslice,
                           A, lda, B, ldb, part);
    else if (b_nc)
        hipLaunchKernelGGL((k_mfma_gemm_splitk<false, true>), grid, block, 0, st, M, N, K, kslice,
                           A, lda, B, ldb, part);
    else
        hipLaunchKernelGGL((k_mfma_gemm_splitk<false, false>), grid, block, 0, st, M, N, K,
                           kslice, A, lda, B, ldb, part);
    hipLaunchKernelGGL(k_gemm_reduce, dim3((M * N + 255) / 256), dim3(256), 0, st, M, N, nsl_used,
                       part, C32, ldc);
    return hipGetLastError();
}

// FP32 -> bf16, row-major [n][w] with leading dimension ld (columns w..ld-1
// of the destination are set to zero).
__global__ void __launch_bounds__(256) k_to_bf16(int64_t n, int w, int ld,
                                                 const float *__restrict__ x,
                                                 bf16 *__restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * ld) return;
    const int64_t r = i / ld;
    const int c = (int)(i - r * ld);
    y[i] = (c < w) ? (bf16)x[r * w + c] : (bf16)0.0f;
}

hipError_t launch_to_bf16(hipStream_t st, int64_t n, int w, int ld, const float *x, bf16 *y) {
    const int64_t tot = n * ld;
    if (tot == 0) return hipSuccess;
    if (tot >= (int64_t)1 << 32) {  // more threads than one launch holds
        const hipError_t e = launch_to_bf16(st, n / 2, w, ld, x, y);
        return e != hipSuccess ? e
                               : launch_to_bf16(st, n - n / 2, w, ld, x + n / 2 * w, y + n / 2 * ld);
    }
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, w, ld,
                       x, y);
    return hipGetLastError();
}

// Output error of the mean squared loss: dy = bf16(scale (y - t)) with
// scale = 2 / (n nout), and one partial sum of (y - t)^2 per workgroup
// (fixed-order tree).
__global__ void __launch_bounds__(256) k_loss(int64_t cnt, float scale,
                                              const float *__restrict__ y,
                                              const float *__restrict__ t,
                                              bf16 *__restrict__ dy, float *__restrict__ part) {
    __shared__ float red[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float e2 = 0.0f;
    if (i < cnt) {
        const float d = y[i] - t[i];
        dy[i] = (bf16)(scale * d);
        e2 = d * d;
    }
    red[threadIdx.x] = e2;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// out[0] = sum of part[0..np) in a fixed order (one workgroup)
__global__ void __launch_bounds__(256) k_sum(int np, const float *__restrict__ part,
                                             float *__restrict__ out) {
    __shared__ float red[256];
    float s = 0.0f;
    for (int i = threadIdx.x; i < np; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

hipError_t launch_loss(hipStream_t st, int64_t cnt, float scale, const float *y, const float *t,
                       bf16 *dy, float *part, float *out) {
    const unsigned nb = (unsigned)((cnt + 255) / 256);
    if (nb == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_loss, dim3(nb), dim3(256), 0, st, cnt, scale, y, t, dy, part);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, st, (int)nb, part, out);
    return hipGetLastError();
}

// Column sums of a bf16 matrix [n][w] into FP32 out[w]: one workgroup per
// column, fixed-order tree.
__global__ void __launch_bounds__(256) k_colsum(int64_t n, int w, const bf16 *__restrict__ d,
                                                float *__restrict__ out) {
    __shared__ float red[256];
    const int c = blockIdx.x;
    float s = 0.0f;
    for (int64_t r = threadIdx.x; r < n; r += 256) s += (float)d[r * w + c];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[c] = red[0];
}

hipError_t launch_colsum(hipStream_t st, int64_t n, int w, const bf16 *d, float *out) {
    hipLaunchKernelGGL(k_colsum, dim3(w), dim3(256), 0, st, n, w, d, out);
    return hipGetLastError();
}

// Adam (Kingma and Ba, 2015) on one FP32 master weight with bias-corrected
// moments: c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t).  Returns the new weight.
__device__ __forceinline__ float adam_step(float gi, float lr, float b1, float b2, float eps,
                                           float c1, float c2, float *w, float *m, float *v) {
    const float mi = b1 * *m + (1.0f - b1) * gi;
    const float vi = b2 * *v + (1.0f - b2) * gi * gi;
    *m = mi;
    *v = vi;
    return *w = *w - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

__global__ void __launch_bounds__(256) k_adam(int np, float lr, float b1, float b2, float eps,
                                              float c1, float c2, const float *__restrict__ g,
                                              float *__restrict__ w, float *__restrict__ m,
                                              float *__restrict__ v) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= np) return;
    adam_step(g[i], lr, b1, b2, eps, c1, c2, w + i, m + i, v + i);
}

hipError_t launch_adam(hipStream_t st, int np, float lr, float b1, float b2, float eps, float c1,
                       float c2, const float *g, float *w, float *m, float *v) {
    hipLaunchKernelGGL(k_adam, dim3((np + 255) / 256), dim3(256), 0, st, np, lr, b1, b2, eps, c1,
                       c2, g, w, m, v);
    return hipGetLastError();
}

// bf16 operand copies of one layer's FP32 weights W [fi][fo] (row-major):
// Wb = W (row-major) and WbT = W^T (row-major [fo][fi]).
__global__ void __launch_bounds__(256) k_weights_bf16(int fi, int fo, const float *__restrict__ W,
                                                      bf16 *__restrict__ Wb,
                                                      bf16 *__restrict__ WbT) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= fi * fo) return;
    const int r = i / fo, c = i - r * fo;
    const bf16 v = (bf16)W[i];
    Wb[i] = v;
    WbT[(size_t)c * fi + r] = v;
}

hipError_t launch_weights_bf16(hipStream_t st, int fi, int fo, const float *W, bf16 *Wb,
                               bf16 *WbT) {
    hipLaunchKernelGGL(k_weights_bf16, dim3((fi * fo + 255) / 256), dim3(256), 0, st, fi, fo, W,
                       Wb, WbT);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused path.  The products, their order along the inner dimension and every
// rounding are those of the kernels above, so a network's outputs and gradients
// do not depend on the path.
// ---------------------------------------------------------------------------
namespace {

// LDS row of a network of widths up to W: 16 bytes more than a power of two, 16
// rows on distinct banks
constexpr int lds_row(int W) { return W + 8; }
constexpr int kFrag = 16 * 32;       // elements of a fragment

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Place of element (column c, inner index k) among fragments of `steps` steps
// per 16 columns: lane 16 (k % 32 / 8) + c % 16 holds eight consecutive k.
__device__ __forceinline__ size_t frag_index(int c, int k, int steps) {
    return ((size_t)(c >> 4) * steps + (k >> 5)) * kFrag + (((k >> 3) & 3) * 16 + (c & 15)) * 8 +
           (k & 7);
}

// Element (column c, row k) of a batch array of w columns: fragments along the
// rows, the columns past the last whole 16 in fragments of their own number of
// columns (a narrow layer then takes its own size, where whole fragments took up to
// 16 times that).
__device__ __forceinline__ size_t batch_index(int c, int k, int w, int steps) {
    return (size_t)(c >> 4) * steps * kFrag + (size_t)(k >> 3) * (8 * min(16, w - (c & ~15))) +
           8 * (c & 15) + (k & 7);
}
// A lane's eight rows of step 0 in 16-column block j of such an array, and the
// distance between steps.  Lanes past the block's columns read its last one; what
// they make of it is not stored.
struct BatchLane {
    const bf16 *p;
    int step;
    __device__ __forceinline__ BatchLane(const bf16 *P, int j, int w, int steps, int c, int quarter) {
        const int wb = min(16, w - 16 * j);
        p = P + (size_t)j * steps * kFrag + 8 * (quarter * wb + min(c, wb - 1));
        step = 32 * wb;
    }
};

// 16 x 16 block: rows of A in LDS (leading dimension lds_row(W), zero past K),
// columns b of B, K in ks steps of 32
template <int W>
__device__ __forceinline__ f32x4 block_product(const bf16 *A, const bf16x8 b[W / 32], int ks,
                                               int lane) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const bf16 *r = A + (lane & 15) * lds_row(W) + 8 * (lane >> 4);
#pragma unroll
    for (int s = 0; s < W / 32; ++s)
        if (s < ks)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                *reinterpret_cast<const bf16x8 *>(r + 32 * s), b[s], acc, 0, 0, 0);
    return acc;
}

}  // namespace

// MB blocks of 16 rows through all layers: bf16 activations in LDS, NW
// wavefronts sharing a layer's 16-column blocks, the weights' fragments read
// from L2 once per row tile, a layer's first ones while the layer before ends.
// Bound by tanh: 6-128x4-4 inference needs 512 of them a row against 51k
// multiply-adds on the matrix cores.  640,000 rows 279 us; layer by layer it took
// six kernels per max_batch rows, with every activation through memory twice
// (2033 us).
// W: the widths' limit, 128 or 256 (a narrow network would hold the wider form's
// operand registers and LDS rows without using them).
// TRAIN: the same, then the output error and the errors of every layer back to
// the first (each row's own).  a_l and d_l are left in memory as batch arrays
// (batch_index), zero past row n: a lane's four results are consecutive rows of one
// column, and the wavefront's 8-byte stores fill 512 bytes in a row.
// XT: float, or bf16 for rows that were converted before (outputs over X).
template <int W, int MB, int NW, bool TRAIN, class XT = float>
__global__ void __launch_bounds__(64 * NW)
    k_mlp_rows(MlpNet net, int64_t n, const XT *__restrict__ X, const float *__restrict__ T,
               float *__restrict__ Y, float scale, float *__restrict__ losspart) {
    constexpr int MT = 16 * MB, kLd = lds_row(W), KS = W / 32;
    extern __shared__ __align__(16) bf16 sm[];
    auto buf = [&](int i) { return sm + i * MT * kLd; };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, mq = 4 * (lane >> 4);
    const int64_t r0 = (int64_t)blockIdx.x * MT;
    const int rows = (int)max((int64_t)0, min((int64_t)MT, n - r0));
    // this wavefront's block t of step s: the forward layers 0 .. L-1, then the
    // layers L-1 .. 1 backward
    auto fetch = [&](int s, int t, bf16x8 b[KS], float &bias) {
        const bool fwd = s < net.L;
        const int l = fwd ? s : 2 * net.L - 1 - s;
        const int K = net.w[fwd ? l : l + 1], N = net.w[fwd ? l + 1 : l], c = 16 * t + col;
        const int ks = (K + 31) / 32;
        const bf16 *P = (fwd ? net.Wf[l] : net.Wr[l]) + (size_t)t * ks * kFrag + 8 * lane;
        if (16 * t < mlp_pad(N)) {
#pragma unroll
            for (int k = 0; k < KS; ++k)
                if (k < ks) b[k] = *reinterpret_cast<const bf16x8 *>(P + k * kFrag);
        }
        bias = (fwd && c < N) ? net.wt[net.woff[l] + K * N + c] : 0.0f;
    };
    // rows m .. m + 3 of column c into a batch array of w columns, zero past row n
    auto put = [&](bf16 *P, int m, int c, int w, bf16x4 v) {
        if (c >= w) return;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (m + i >= rows) v[i] = (bf16)0.0f;
        *reinterpret_cast<bf16x4 *>(P + batch_index(c, (int)(r0 + m), w, net.steps)) = v;
    };
    bf16x8 b[KS];
    float bias;
    fetch(0, wave, b, bias);
    const int w0 = net.w[0], w0p = mlp_pad(w0);
    for (int e = threadIdx.x; e < MT * w0p; e += 64 * NW) {
        const int m = e / w0p, c = e - m * w0p;
        buf(0)[m * kLd + c] = (m < rows && c < w0) ? (bf16)X[(r0 + m) * w0 + c] : (bf16)0.0f;
    }
    __syncthreads();
    if (TRAIN) {
        for (int e = threadIdx.x; e < MT / 4 * w0p; e += 64 * NW) {
            const int m = e / w0p * 4, c = e % w0p;
            bf16x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = buf(0)[(m + i) * kLd + c];
            put(net.aT[0], m, c, w0, v);
        }
    }
    float e2 = 0.0f;
    for (int l = 0; l < net.L; ++l) {
        const int fi = net.w[l], fo = net.w[l + 1], ks = (fi + 31) / 32;
        const bool last = l + 1 == net.L;
        const bf16 *in = buf(TRAIN ? l : l & 1);
        bf16 *out = buf(TRAIN ? l + 1 : (l + 1) & 1);
        const int nt = last && !TRAIN ? (fo + 15) / 16 : mlp_pad(fo) / 16;
        for (int t = wave; t < nt; t += NW) {
            const int c = 16 * t + col;
            if (t != wave) fetch(l, t, b, bias);
#pragma unroll 1
            for (int mb = 0; mb < MB; ++mb) {
                const f32x4 acc = block_product<W>(in + 16 * mb * kLd, b, ks, lane);
                const int m = 16 * mb + mq;
                bf16x4 h;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = acc[i] + bias;
                    if (!last) {
                        h[i] = c < fo ? (bf16)tanhf(v) : (bf16)0.0f;
                    } else if (TRAIN) {
                        const float d = (c < fo && m + i < rows) ? v - T[(r0 + m + i) * fo + c]
                                                                 : 0.0f;
                        h[i] = (bf16)(scale * d);
                        e2 += d * d;
                    } else if (c < fo && m + i < rows) {
                        Y[(r0 + m + i) * fo + c] = v;
                    }
                }
                if (last && !TRAIN) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) out[(m + i) * kLd + c] = h[i];
                if (TRAIN) put(last ? net.dT[l] : net.aT[l + 1], m, c, fo, h);
            }
        }
        if (!last || (TRAIN && net.L > 1)) fetch(l + 1, wave, b, bias);
        __syncthreads();
    }
    if (!TRAIN) return;
    // d_{l-1} = (d_l W_l^T) (1 - a_l^2), between the buffers past the activations
    int cur = net.L;
    for (int l = net.L - 1; l > 0; --l) {
        const int fi = net.w[l], fo = net.w[l + 1], ks = (fo + 31) / 32;
        const int step = 2 * net.L - 1 - l;
        const bf16 *in = buf(cur), *a = buf(l);
        cur = 2 * net.L + 1 - cur;
        bf16 *out = buf(cur);
        for (int t = wave; t < mlp_pad(fi) / 16; t += NW) {
            const int c = 16 * t + col;
            if (t != wave) fetch(step, t, b, bias);
#pragma unroll 1
            for (int mb = 0; mb < MB; ++mb) {
                const f32x4 acc = block_product<W>(in + 16 * mb * kLd, b, ks, lane);
                const int m = 16 * mb + mq;
                bf16x4 h;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float av = (float)a[(m + i) * kLd + c];
                    h[i] = c < fi ? (bf16)(acc[i] * (1.0f - av * av)) : (bf16)0.0f;
                    out[(m + i) * kLd + c] = h[i];
                }
                put(net.dT[l - 1], m, c, fi, h);
            }
        }
        if (l > 1) fetch(step + 1, wave, b, bias);
        __syncthreads();
    }
    // the tile's sum of squared errors, in a fixed order
    float *red = reinterpret_cast<float *>(sm);
    red[threadIdx.x] = e2;
    __syncthreads();
    for (int s = 32 * NW; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) losspart[blockIdx.x] = red[0];
}

// All layers' weight gradients a_{l-1}^T d_l in one launch: wavefront (slice,
// block) sums one 16 x 32 block over its slice of the rows into
// part[slice][flat weight].  The first workgroups sum the bias gradients of 16
// columns of d_l each, in k_colsum's order: row r belongs to partial sum r % 256, a
// thread holds eight consecutive ones of a column (one 16-byte load a round) for two
// row groups, and the 256 are added as a tree.  They are the longest chains, so they
// start first (last in the grid: 15.1 us where this is 12.8).  Bound by load latency:
// a chain's loads are issued in batches, held in that order by scheduling barriers
// (without them 19.3 us), with four waves per SIMD as the registers' target.
// 8,192 rows of the 6-128x4-4 network 12.8 us; one launch per layer and sum,
// gathering both operands two bytes at a time, took 105.
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(4, 4)))
    k_mlp_wgrad(MlpNet net, int n, int kslice, int nblock, int items, float *__restrict__ part) {
    const int bias_wgs = gridDim.x - (items + kWaves - 1) / kWaves;
    const int lane = threadIdx.x & 63;
    if ((int)blockIdx.x < bias_wgs) {
        __shared__ float red[256][17];
        int j = blockIdx.x, l = 0;
        while (j >= (net.w[l + 1] + 15) / 16) j -= (net.w[++l] + 15) / 16;
        const int steps = (n + 31) / 32;
        // rows 8 g .. 8 g + 7 (mod 256) of column c; g and g + 16
        const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
        const BatchLane d(net.dT[l], j, net.w[l + 1], net.steps, c, g & 3);
        float s[2][8] = {};
        auto add = [](bf16x8 v, float t[8]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] += (float)v[i];
        };
        // whole rounds of 256 rows, kBatch at a time with all their loads in flight
        constexpr int kBatch = 8;
        auto sum = [&](int step) {
            const bf16 *q = d.p + (size_t)(g >> 2) * step;
            auto load = [&](int at) {
                return *reinterpret_cast<const bf16x8 *>(q + (size_t)at * step);
            };
            const int left = steps % 8 - (g >> 2);
            int r = steps / 8;
            for (; r >= kBatch; r -= kBatch, q += 8 * kBatch * (size_t)step) {
                bf16x8 v[2 * kBatch];
#pragma unroll
                for (int u = 0; u < 2 * kBatch; ++u) {
                    v[u] = load(4 * u);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int u = 0; u < 2 * kBatch; ++u) {
                    add(v[u], s[u & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            for (; r > 0; --r, q += 8 * (size_t)step) {
                add(load(0), s[0]);
                add(load(4), s[1]);
            }
            if (left > 0) add(load(0), s[0]);
            if (left > 4) add(load(4), s[1]);
        };
        // whole blocks lie at constant distances, which take no address registers
        if (d.step == kFrag) sum(kFrag);
        else sum(d.step);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 8; ++i) red[128 * h + 8 * g + i][c] = s[h][i];
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            for (int r = g; r < h; r += 16) red[r][c] += red[r + h][c];
            __syncthreads();
        }
        if (g == 0 && 16 * j + c < net.w[l + 1])
            net.g[net.woff[l] + net.w[l] * net.w[l + 1] + 16 * j + c] = red[0][c];
        return;
    }
    const int item = (blockIdx.x - bias_wgs) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= items) return;  // whole wavefront leaves together
    const int sl = item / nblock;
    int blk = item - sl * nblock, l = 0, ntn;
    for (;; ++l) {
        const int ntm = (net.w[l] + 15) / 16;
        ntn = (net.w[l + 1] + 31) / 32;
        if (blk < ntm * ntn) break;
        blk -= ntm * ntn;
    }
    const int fi = net.w[l], fo = net.w[l + 1];
    const int i0 = blk / ntn, j0 = blk % ntn * 2;  // blocks of 16
    const int kb = sl * kslice, ke = min(n, kb + kslice);
    // an odd last block of d_l stands in for the one past it
    const int c = lane & 15, quarter = lane >> 4, j1 = 16 * (j0 + 1) < fo ? j0 + 1 : j0;
    const BatchLane A(net.aT[l], i0, fi, net.steps, c, quarter);
    const BatchLane B0(net.dT[l], j0, fo, net.steps, c, quarter);
    const BatchLane B1(net.dT[l], j1, fo, net.steps, c, quarter);
    f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
    auto product = [&](int sa, int s0, int s1) {
        const bf16 *pa = A.p + (size_t)(kb / 32) * sa, *p0 = B0.p + (size_t)(kb / 32) * s0,
                   *p1 = B1.p + (size_t)(kb / 32) * s1;
        auto load = [](const bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); };
        auto mac = [&](bf16x8 a, bf16x8 b0, bf16x8 b1) {
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b1, acc[1], 0, 0, 0);
        };
        int k = (ke - kb + 31) / 32;
        for (; k >= 4; k -= 4, pa += 4 * sa, p0 += 4 * s0, p1 += 4 * s1) {
            bf16x8 a[4], b0[4], b1[4];  // four steps' loads in flight
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = load(pa + u * sa);
                b0[u] = load(p0 + u * s0);
                b1[u] = load(p1 + u * s1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) mac(a[u], b0[u], b1[u]);
        }
        for (; k > 0; --k, pa += sa, p0 += s0, p1 += s1) mac(load(pa), load(p0), load(p1));
    };
    if (A.step == kFrag && B0.step == kFrag && B1.step == kFrag) product(kFrag, kFrag, kFrag);
    else product(A.step, B0.step, B1.step);
    float *P = part + (size_t)sl * net.np + net.woff[l];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int j = 16 * (j0 + h) + (lane & 15);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * i0 + 4 * (lane >> 4) + i;
            if (r < fi && j < fo) P[(size_t)r * fo + j] = acc[h][i];
        }
    }
}

namespace {

// bf16 copies of element (r, c) of W_l
__device__ __forceinline__ void pack_weight(const MlpNet &net, int l, int r, int c, float w) {
    const bf16 v = (bf16)w;
    net.Wf[l][frag_index(c, r, (net.w[l] + 31) / 32)] = v;
    net.Wr[l][frag_index(r, c, (net.w[l + 1] + 31) / 32)] = v;
}

__device__ __forceinline__ int layer_of(const MlpNet &net, int i) {
    int l = 0;
    while (l + 1 < net.L && i >= net.woff[l + 1]) ++l;
    return l;
}

}  // namespace

// every fragment element of layer blockIdx.y, the padding as zero
__global__ void __launch_bounds__(256) k_mlp_pack(MlpNet net) {
    const int l = blockIdx.y, fi = net.w[l], fo = net.w[l + 1];
    const int i = blockIdx.x * 256 + threadIdx.x, r = i / mlp_pad(fo), c = i % mlp_pad(fo);
    if (r >= mlp_pad(fi)) return;
    pack_weight(net, l, r, c, (r < fi && c < fo) ? net.wt[net.woff[l] + r * fo + c] : 0.0f);
}

// Slices added in slice order into the gradient, one thread per parameter, and
// with ADAM the step and the bf16 copies; the last workgroup adds the loss.
template <bool ADAM>
__global__ void __launch_bounds__(256)
    k_mlp_update(MlpNet net, int nsl, const float *__restrict__ part, MlpAdam ad, int nloss,
                 const float *__restrict__ losspart, float *__restrict__ loss) {
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ float red[256];
        float s = 0.0f;
        for (int i = threadIdx.x; i < nloss; i += 256) s += losspart[i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) loss[0] = red[0];
        return;
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= net.np) return;
    const int l = layer_of(net, i), o = i - net.woff[l];
    const bool weight = o < net.w[l] * net.w[l + 1];
    float gi;
    if (weight) {
        gi = 0.0f;
#pragma unroll 8
        for (int sl = 0; sl < nsl; ++sl) gi += part[(size_t)sl * net.np + i];
        net.g[i] = gi;
    } else {
        gi = net.g[i];
    }
    if (!ADAM) return;
    const float w = adam_step(gi, ad.lr, ad.b1, ad.b2, ad.eps, ad.c1, ad.c2, net.wt + i, ad.m + i,
                              ad.v + i);
    if (weight) pack_weight(net, l, o / net.w[l + 1], o % net.w[l + 1], w);
}

bool mlp_fusable(const int *widths, int nwidth) {
    if (nwidth - 1 > kFuseLayers) return false;
    return std::all_of(widths, widths + nwidth, [](int w) { return w <= kFuseWidth; });
}

namespace {

// slices of the weight gradients' inner dimension, as launch_mfma_gemm_splitk
// takes them (no layer of a fusable network has more than kSplitKMaxTiles blocks)
void batch_slices(int64_t n, int &nsl, int &kslice) {
    nsl = gemm_splitk_slices(16, 16, (int)n);
    kslice = nsl > 1 ? ((int)((n + nsl - 1) / nsl) + 31) / 32 * 32 : (int)n;
    nsl = (int)((n + kslice - 1) / kslice);
}

size_t rows_lds(int W, int mb, int bufs) {
    return (size_t)bufs * 16 * mb * lds_row(W) * sizeof(bf16);
}

bool wide(const MlpNet &net) {
    return std::any_of(net.w, net.w + net.L + 1, [](int w) { return w > 128; });
}

}  // namespace

// the slices asked for, which grow with n (those used need not: their length
// is rounded to whole steps)
size_t mlp_part_floats(int np, int64_t n) {
    return (size_t)gemm_splitk_slices(16, 16, (int)n) * np;
}

// row tiles of a gradient of n rows: whole steps of 32 rows
int64_t mlp_loss_parts(int64_t n) { return (n + 31) / 32 * 2; }

// Tile and wavefronts by rows: tiles of 32 with four wavefronts read the weights
// less often and keep more workgroups per CU than any other once the chip is
// full (640,000 rows: 279 us; 16 rows 416, 32 rows with eight wavefronts 346, 64
// rows 361 and 382); up to 32,768 rows tiles of 16 spread wider (20,000: 18.8
// against 22.1 us), and up to 8,192, where a call is one chain of layers, a
// wavefront per 16-column block shortens each (4,000: 8.0, with four
// wavefronts 11.6, tiles of 32 18.2).  Wider than 128 a layer has twice the
// blocks and eight wavefronts are better throughout (6-256x3-4, the call: 400,000
// rows 378 us with tiles of 32, 601 with 16, 417 with four wavefronts; 2,000 rows
// 32.4 with tiles of 32, 26.1 with 16; layer by layer 2155 and 43.1).
//
// A launch holds fewer than 2^32 threads and a grid past that is cut without an
// error, so more rows (16 threads each in the wide form) go in several launches.
hipError_t launch_mlp_forward(hipStream_t st, const MlpNet &net, const float *X, float *Y,
                              int64_t n) {
    constexpr int64_t kMaxRows = (int64_t)1 << 27;
    for (; n > kMaxRows; n -= kMaxRows) {
        const hipError_t e = launch_mlp_forward(st, net, X, Y, kMaxRows);
        if (e != hipSuccess) return e;
        X += kMaxRows * net.w[0];
        Y += kMaxRows * net.w[net.L];
    }
    if (n <= 0) return hipSuccess;
    const int W = wide(net) ? 256 : 128;
    auto go = [&](auto kern, int mb, int nw) {
        const int64_t wgs = (n + 16 * mb - 1) / (16 * mb);
        hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(64 * nw), rows_lds(W, mb, 2), st, net, n,
                           X, (const float *)nullptr, Y, 0.0f, (float *)nullptr);
        return hipGetLastError();
    };
    if (W == 256) {
        if (n <= 8192) return go(k_mlp_rows<256, 1, 8, false>, 1, 8);
        return go(k_mlp_rows<256, 2, 8, false>, 2, 8);
    }
    if (n <= 8192) return go(k_mlp_rows<128, 1, 8, false>, 1, 8);
    if (n <= 32768) return go(k_mlp_rows<128, 1, 4, false>, 1, 4);
    return go(k_mlp_rows<128, 2, 4, false>, 2, 4);
}

// One tile form for every width and row count: a rare call, which has paid a pass
// over X for its copy.
hipError_t launch_mlp_forward_bf16(hipStream_t st, const MlpNet &net, const bf16 *X, float *Y,
                                   int64_t n) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_mlp_rows<256, 2, 8, false, bf16>), dim3((unsigned)((n + 31) / 32)),
                       dim3(64 * 8), rows_lds(256, 2, 2), st, net, n, X, (const float *)nullptr, Y,
                       0.0f, (float *)nullptr);
    return hipGetLastError();
}

// 16 rows per workgroup and a wavefront per 16-column block: the row kernel is
// a chain of layers, and 8,192 rows then put two workgroups on each CU (23 us;
// 32 rows and eight wavefronts 31, four 44).  Wider than 128 a wavefront takes two
// blocks (6-256x3-4, 8,192 rows, the call: 122 us, with sixteen wavefronts 130,
// layer by layer 318).
hipError_t launch_mlp_gradient(hipStream_t st, const MlpNet &net, const float *X, const float *T,
                               int64_t n, float *part, float *losspart, float *loss,
                               const MlpAdam *adam) {
    const int nloss = (int)mlp_loss_parts(n);
    const float scale = (float)(2.0 / (double)(n * net.w[net.L]));
    const int W = wide(net) ? 256 : 128;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nloss), dim3(64 * 8), rows_lds(W, 1, net.L + 2), st, net, n,
                           X, T, (float *)nullptr, scale, losspart);
    };
    if (W == 256) go(k_mlp_rows<256, 1, 8, true>);
    else go(k_mlp_rows<128, 1, 8, true>);
    int nsl, kslice, nblock = 0, cols = 0;
    batch_slices(n, nsl, kslice);
    for (int l = 0; l < net.L; ++l) {
        nblock += ((net.w[l] + 15) / 16) * ((net.w[l + 1] + 31) / 32);
        cols += (net.w[l + 1] + 15) / 16;
    }
    const int items = nblock * nsl;
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((items + kWaves - 1) / kWaves + cols), dim3(64 * kWaves), 0,
                       st, net, (int)n, kslice, nblock, items, part);
    const dim3 grid((net.np + 255) / 256 + 1), block(256);
    if (adam)
        hipLaunchKernelGGL(k_mlp_update<true>, grid, block, 0, st, net, nsl, part, *adam, nloss,
                           losspart, loss);
    else
        hipLaunchKernelGGL(k_mlp_update<false>, grid, block, 0, st, net, nsl, part, MlpAdam{}, nloss,
                           losspart, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_pack(hipStream_t st, const MlpNet &net) {
    hipLaunchKernelGGL(k_mlp_pack, dim3(kFuseWidth * kFuseWidth / 256, net.L), dim3(256), 0, st, net);
    return hipGetLastError();
}

}  // namespace ql
