// Host entry points of the warm-start network kernels (mlp.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <stddef.h>

namespace pdhcg {

// GEMM epilogues
enum : int {
  EPI_BIAS_F32 = 0,     // out = acc + bias[n]             (FP32)
  EPI_BIAS_RELU_BF16,   // out = bf16(max(acc + bias, 0))
  EPI_MASK_BF16,        // out = bf16(mask > 0 ? acc : 0)
  EPI_GRAD              // out = acc (FP32), and the rest of GradStep
};

struct AdamStep {
  float lr, b1, b2, eps;
  float omb1, omb2;     // 1 - b1, 1 - b2 (formed in FP64: 1 - 0.999f loses digits)
  float c1, c2;         // bias corrections 1 - b1^t, 1 - b2^t
};

// what a layer's weight gradient is used for: the bias gradient db, and with
// `on` the Adam step of W (and its BF16 copy Wb) and b
struct GradStep {
  int on;
  AdamStep a;
  float *W, *mW, *vW;
  __bf16* Wb;
  float *b, *mb, *vb, *db;
};

// C = A op(B) with the epilogue `epi`; `work` holds the sums of K's chunks
hipError_t mlp_gemm(const __bf16* A, long lda, const __bf16* B, bool tb, long ldb, int M, int N, int K, int epi,
                    const float* bias, const __bf16* mask, float* outf, __bf16* outb, float* work,
                    size_t work_floats, hipStream_t st);
// dW = in^T dz (K x N), db = the column sums of dz (FP32, rows in order), and
// the Adam step
hipError_t mlp_grad(const __bf16* in, const __bf16* dz, int rows, int K, int N, float* dW, const GradStep& s,
                    size_t work_floats, hipStream_t st);
hipError_t mlp_to_bf16(const float* x, __bf16* y, long n, hipStream_t st);
// dz = bf16(scale (yhat - y)); *loss = sum (yhat - y)^2 (device scalar)
hipError_t mlp_mse_grad(const float* yhat, const float* y, __bf16* dz, long n, float scale, double* part,
                        double* loss, hipStream_t st);

}  // namespace pdhcg
