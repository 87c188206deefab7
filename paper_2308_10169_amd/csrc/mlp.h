// Learned initializer: launchers of the device kernels (mlp.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace sepso {

enum : int { EPI_BIAS_RELU_BF16 = 0, EPI_BIAS_F32 = 1, EPI_BIAS_LOSS = 2, EPI_MASK = 3 };

// GEMM epilogue: what happens to each FP32 accumulator C(row, col).
struct Epi {
  int mode;              // EPI_*
  const float* bias;     // per column (EPI_BIAS_*)
  float* out_f32;        // row stride ldo
  uint16_t* out_bf16;    // row stride ldo
  const uint16_t* mask;  // ReLU mask source (BF16 activations), row stride ldo
  int ldo;
  const float* target;   // EPI_BIAS_LOSS: row stride ldo; out_bf16 = scale * (C + bias - target)
  float scale;
};

void launch_raster(const Pools& pl, int n_inst, uint16_t* X, int ldx, int32_t* eligible,
                   hipStream_t s);
// C[M x N] = A[M x K] B[N x K]^T (k contiguous in both, K % 32 == 0, N % 32 == 0, 16-byte aligned rows).
void launch_gemm(const uint16_t* A, int lda, const uint16_t* B, int ldb, int M, int N, int K, const Epi& ep,
                 hipStream_t s);
void launch_targets(const Pools& pl, int n_inst, float* T, int ldt, hipStream_t s);

struct AdamStep {
  int on;  // 0: gradients are stored, parameters stay
  float lr, b1, b2, eps, c1, c2;
};
// One layer's weights: dW[M x N] = A^T B over the batch's K rows (A: K x M, B: K x N,
// its rows and those of p16 ldb apart).
struct DwSet {
  const uint16_t *A, *B;
  int M, N, ldb;
  float *g, *p, *m, *v;  // gradient; parameters and moments (M x N)
  uint16_t *p16, *pT;    // BF16 parameters, and transposed (N x M) or NULL
  int kper, first;       // filled by launch_weight_grads
};
// The same layer's biases: column sums of its FP32 dZ (K x n; NULL: the last
// layer's, from y and target).
struct ColSet {
  const float* dz;
  int n;
  float* part;  // scratch, col_part_floats of the largest K
  float *g, *p, *m, *v;
  int cr, first;  // filled by launch_weight_grads
};
struct DwArgs {
  DwSet w[4];
  ColSet c[4];
  int K, tiles, col_blocks;
  AdamStep adam;
  const float *y, *target;  // K x kLinOut
  float scale;              // dY = scale (y - target)
  float* row_sq;            // K: squared errors per row
};
// Weight and bias gradients of all layers, the Adam step where a.adam.on, and
// the loss (loss_scale times the sum of squared errors): two launches.
void launch_weight_grads(DwArgs a, float loss_scale, float* loss, hipStream_t s);
constexpr int64_t col_part_floats(int64_t max_rows) { return (max_rows / 256 + 256) * kLinHidden; }
// BF16 copies of M x N weights: p16 (rows ld apart) and, transposed, pT (or NULL).
void launch_cvt_bf16(const float* p, uint16_t* p16, int ld, uint16_t* pT, int M, int N, hipStream_t s);
void launch_proposal(const Pools& pl, int n_inst, const float* Y, int ldy, const int32_t* eligible,
                     hipStream_t s);

}  // namespace sepso
