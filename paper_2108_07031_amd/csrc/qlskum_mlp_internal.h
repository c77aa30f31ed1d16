// Internal interface between the warm-start network's host runtime and its
// HIP kernels.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ql {

typedef __bf16 bf16;

enum MlpEpilogue : int { kEpiStore = 0, kEpiBias = 1, kEpiBiasTanh = 2, kEpiTanhGrad = 3 };

// C (M x N, leading dimension ldc) = op(A) op(B) with inner dimension K on
// the bf16 matrix cores, FP32 accumulation, then the epilogue (see the
// kernel).  a_kc: element (m, k) of op(A) is A[m*lda + k], else A[k*lda + m];
// b_nc: element (k, n) of op(B) is B[n*ldb + k], else B[k*ldb + n].
hipError_t launch_mfma_gemm(hipStream_t st, int epi, bool a_kc, bool b_nc, int M, int N, int K,
                            const bf16 *A, int lda, const bf16 *B, int ldb, const float *bias,
                            const bf16 *act, float *C32, bf16 *C16, int ldc);
// The plain product (kEpiStore) split along K when it has at most
// kSplitKMaxTiles output blocks and K is long: up to kSplitKMaxSlices
// slices of at least kSplitKSlice, partial products in part (at least
// gemm_splitk_slices(M, N, K) * M * N floats), then added in slice order.
constexpr int kSplitKMaxTiles = 256, kSplitKMaxSlices = 64, kSplitKSlice = 256;
int gemm_splitk_slices(int M, int N, int K);
hipError_t launch_mfma_gemm_splitk(hipStream_t st, bool a_kc, bool b_nc, int M, int N, int K,
                                   const bf16 *A, int lda, const bf16 *B, int ldb, float *part,
                                   float *C32, int ldc);
hipError_t launch_to_bf16(hipStream_t st, int64_t n, int w, int ld, const float *x, bf16 *y);
// dy = bf16(scale (y - t)); *out = sum (y - t)^2 (part: >= ceil(cnt/256) floats)
hipError_t launch_loss(hipStream_t st, int64_t cnt, float scale, const float *y, const float *t,
                       bf16 *dy, float *part, float *out);
hipError_t launch_colsum(hipStream_t st, int64_t n, int w, const bf16 *d, float *out);
hipError_t launch_adam(hipStream_t st, int np, float lr, float b1, float b2, float eps, float c1,
                       float c2, const float *g, float *w, float *m, float *v);
hipError_t launch_weights_bf16(hipStream_t st, int fi, int fo, const float *W, bf16 *Wb,
                               bf16 *WbT);

// --- networks that fit the fused path ---------------------------------------
// Every width at most kFuseWidth and at most kFuseLayers layers: a workgroup
// then holds the activations of its rows in LDS through all layers (68 KB to
// train the widest, two workgroups per CU).  Wider layers would leave one
// workgroup per CU and are served by the products above.
constexpr int kFuseWidth = 256, kFuseLayers = 6;

// One network and its training workspace as the fused kernels see it.  The
// matrix-core operands lie in memory as the instruction takes them, in
// fragments of 16 columns by 32 steps of the inner dimension: a wavefront reads a
// fragment as 1 KB in a row.  The weights' (frag_index) are padded with zeros; the
// batch arrays hold w_l columns (batch_index).
struct MlpNet {
    int L;                      // layers
    int w[kFuseLayers + 1];     // widths
    int woff[kFuseLayers];      // offset of W_l in the flat vectors (b_l follows)
    int np;
    bf16 *Wf[kFuseLayers], *Wr[kFuseLayers];  // W_l for a_{l-1} W_l and for d_l W_l^T
    bf16 *aT[kFuseLayers], *dT[kFuseLayers];  // a_l and the error of layer l's output,
    int steps;                  // whose inner dimension is the batch: room for 32 steps rows
    float *wt, *g;              // FP32 weights and gradient (flat)
};
constexpr int mlp_pad(int w) { return (w + 31) & ~31; }
bool mlp_fusable(const int *widths, int nwidth);
// floats of workspace for the slices of a gradient of n rows or fewer
size_t mlp_part_floats(int np, int64_t n);
// loss partials of a gradient of n rows
int64_t mlp_loss_parts(int64_t n);
// Y = network(X), n rows; Y may not overlap X (row tiles run in any order)
hipError_t launch_mlp_forward(hipStream_t st, const MlpNet &net, const float *X, float *Y,
                              int64_t n);
// the same for at most 2^26 rows already rounded to bf16 (row-major [n][w_in])
hipError_t launch_mlp_forward_bf16(hipStream_t st, const MlpNet &net, const bf16 *X, float *Y,
                                   int64_t n);
// gradient of the mean squared error over n rows into net.g and the sum of
// squared errors into *loss; with adam, one Adam step on net.wt, m and v and the
// bf16 copies of the new weights
struct MlpAdam {
    float lr, b1, b2, eps, c1, c2;
    float *m, *v;
};
hipError_t launch_mlp_gradient(hipStream_t st, const MlpNet &net, const float *X, const float *T,
                               int64_t n, float *part, float *losspart, float *loss,
                               const MlpAdam *adam);
// the fragments of the FP32 weights net.wt
hipError_t launch_mlp_pack(hipStream_t st, const MlpNet &net);

}  // namespace ql
