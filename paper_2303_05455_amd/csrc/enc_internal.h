// Internal declarations of the encoder kernels (enc.hip) and host code
// (enc_api.hip).  Not part of the public ABI.
#pragma once

#include "ivhd_internal.h"

namespace ivhd {

enum { GEMM_EPI_F32 = 0, GEMM_EPI_BIAS_RELU_BF16 = 1, GEMM_EPI_RELU_MASK_BF16 = 2 };

struct GemmArgs {
  const uint16_t *A;
  const uint16_t *B;
  int64_t M, N, K;
  int64_t lda, ldb;
  int64_t kchunk;          // K range per blockIdx.z (set by launch_gemm_bf16)
  const float *bias;       // [N] or NULL (GEMM_EPI_BIAS_RELU_BF16)
  const uint16_t *mask;    // [M][ldm] forward activation (GEMM_EPI_RELU_MASK_BF16)
  int64_t ldm;
  void *C;                 // FP32 slabs [splits][M][ldc] or BF16 [M][ldc]
  int64_t ldc;
  bool vec_a, vec_b;       // 16-byte vector loads allowed (ld % 8 == 0, aligned base)
  bool whole_b;            // B K-major: every row of B holds whole 16-byte chunks up to N
};

hipError_t launch_gemm_bf16(const GemmArgs &g, int ta, int tb, int epi, int splits, hipStream_t s);
int gemm_splits_used(int64_t K, int splits);
hipError_t launch_splitk_reduce(const float *part, int splits, int64_t M, int64_t N, int64_t ldp, float *out,
                                int64_t ldo, hipStream_t s);
hipError_t launch_f32_to_bf16(const float *x, int64_t n, uint16_t *y, hipStream_t s);
// out [R][ldo] = X[rows[r]][0..N) (rows NULL: X[r]), zeros up to ldo (a multiple of 8); 16-byte aligned out
hipError_t launch_gather_rows(const uint16_t *X, int64_t N, const int32_t *rows, int64_t R, uint16_t *out,
                              int64_t ldo, hipStream_t s);
hipError_t launch_head_forward(const uint16_t *H, int64_t R, int K, const uint16_t *W3, const float *b3, float *Z,
                               hipStream_t s);
// backward of the head: dH = (dZ W3) * [H > 0], and over the rows the sums of
// dZ x H: out [2][K]; ws as for launch_colsum with J = 2 K
hipError_t launch_head_backward(const float *dZ, const uint16_t *W3, const uint16_t *H, int64_t R, int K,
                                uint16_t *dH, float *ws, float *out, hipStream_t s);
// column sums of the BF16 matrix X [R][J] (fixed order); ws: [bias_workspace(J)]
int64_t bias_workspace(int64_t J);
hipError_t launch_bias_sum(const uint16_t *X, int64_t R, int64_t J, float *ws, float *out, hipStream_t s);
// column sums of the FP32 matrix X [R][J] as a fixed-order tree of kColsumRows-row
// partial sums (deterministic).  ws must hold colsum_workspace(R, J) floats.
constexpr int kColsumRows = 256;
int64_t colsum_workspace(int64_t R, int64_t J);
hipError_t launch_colsum(const float *X, int64_t R, int64_t J, float *ws, float *out, hipStream_t s);
// out [C][ldo] = transpose of the BF16 matrix in [R][C], entries r >= R of
// each out row zero (ldo >= R)
hipError_t launch_transpose_bf16(const uint16_t *in, int64_t R, int64_t C, uint16_t *out, int64_t ldo,
                                 hipStream_t s);
hipError_t launch_adam(float *w, const float *g, float *m, float *v, uint16_t *w16, int64_t n, float lr, float b1,
                       float b2, float eps, int64_t t, float gscale, hipStream_t s);
hipError_t launch_glorot(float *w, int64_t n, int fan_in, int fan_out, uint64_t seed, uint64_t offset,
                         hipStream_t s);

// ---- enc_mlp.hip ----
// the whole forward pass of R rows X [R][ldx] into Z [R][2]; ldx is n_in, or a
// multiple of 8 above it with zeros in between; A1 and A2, the hidden
// activations, are stored when A1 is given (both then)
struct MlpArgs {
  const uint16_t *X;
  int ldx;
  const uint16_t *W1p, *W2p;   // packed weights (set by launch_mlp_forward)
  const float *b1, *b2, *b3;
  const uint16_t *W3;          // [2][h2]
  uint16_t *A1, *A2;
  float *Z;
  int64_t R;
  int n_in, h1, h2;
};
// at least one 16-byte chunk to a row, and hidden widths that leave none of the
// eight wavefronts of 64 columns idle
bool mlp_ok(int n_in, int h1, int h2);
int64_t mlp_pack_elems(int n_in, int h1);
// pack: [mlp_pack_elems] scratch, 16-byte aligned
hipError_t launch_mlp_forward(MlpArgs a, const uint16_t *W1, const uint16_t *W2, uint16_t *pack, hipStream_t s);

hipError_t launch_batch_rows(const int32_t *nn_idx, int nn, const int32_t *rn_idx, int rn, int64_t M, int64_t B,
                             uint64_t a, uint64_t c0, int64_t off, int32_t *rows, hipStream_t s);
hipError_t launch_batch_plan(int64_t B, int nn, int rn, int32_t *lnn, int32_t *lrn, hipStream_t s);

}  // namespace ivhd
