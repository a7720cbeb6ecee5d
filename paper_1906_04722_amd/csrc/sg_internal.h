// sg_internal.h -- kernels of the learned entry-pressure surrogate (internal;
// the public interface is lbm_surrogate.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sg {

typedef uint16_t bf16;  // bfloat16 bit pattern (round to nearest even from FP32)

constexpr int kFeat = 80;
constexpr int kHidden = 256;
constexpr int kOut = 17;
constexpr int kLayers = 4;
// widths of the layer inputs/outputs: 80 -> 256 -> 256 -> 256 -> 17
constexpr int kWidth[kLayers + 1] = {kFeat, kHidden, kHidden, kHidden, kOut};
// offsets of W_l ([out][in]) and b_l inside one member's flat parameters
constexpr long long w_off(int l) {
  long long o = 0;
  for (int i = 0; i < l; ++i) o += (long long)kWidth[i + 1] * kWidth[i] + kWidth[i + 1];
  return o;
}
constexpr long long b_off(int l) { return w_off(l) + (long long)kWidth[l + 1] * kWidth[l]; }
constexpr long long kParams = w_off(kLayers);
static_assert(kParams == 156689, "parameter count");

constexpr int kOcc = 32;   // occupancy samples per axis
constexpr int kPool = 8;   // samples per pooled cell and axis

// BF16 weights packed in the operand order of the 16x16x32 matrix instruction:
// per member and layer, output tiles of 16 by chunks of 32 inputs, each a
// fragment of 64 lanes x 8 values, W[16 t + l % 16][32 c + 8 (l / 16) + i] for
// lane l, zero beyond the layer's widths
constexpr int kTilesN[kLayers] = {16, 16, 16, 2};
constexpr int kChunksK[kLayers] = {3, 8, 8, 8};
constexpr int kFrag = 512;  // values of one fragment
constexpr int pack_off(int l) {
  int o = 0;
  for (int i = 0; i < l; ++i) o += kTilesN[i] * kChunksK[i];
  return o;
}
constexpr long long kPackF = (long long)pack_off(kLayers) * kFrag;
// then, for layers 1..3, the transposed weights of the backward products:
// tiles of 16 inputs by chunks of 32 outputs, W[32 c + 8 (l / 16) + i][16 t + l % 16]
constexpr int kChunksN[kLayers] = {8, 8, 8, 1};
constexpr int packt_off(int l) {
  int o = pack_off(kLayers);
  for (int i = 1; i < l; ++i) o += 16 * kChunksN[i];
  return o;
}
constexpr long long kPack = (long long)packt_off(kLayers) * kFrag;
hipError_t launch_pack(const float *w, bf16 *wp, int members, hipStream_t st);

// y[z*ycap + b][17] (f32, standardised outputs) of every member for n rows of
// X [n][80] (FP64), standardised with mu, sd; bad[0] = 1 when X is not finite
hipError_t launch_mlp(const double *X, const double *mu, const double *sd, int n, int members,
                      const bf16 *wp, const float *w, float *y, long long ycap, int *bad,
                      hipStream_t st);

// per-column mean and population std (FP64) of X [n][cols], std < 1e-12 -> 1
hipError_t launch_col_stats(const double *X, int n, int cols, double *mu, double *sd,
                            hipStream_t st);
// Y[i][j] = (float)((X[i][j] - mu[j]) / sd[j])
hipError_t launch_standardise(const double *X, int n, int cols, const double *mu,
                              const double *sd, float *Y, hipStream_t st);
// ---- one training batch: forward, loss gradient and backward in one kernel,
// the weight gradients and Adam in a second ------------------------------------
// Operands of the weight gradients, per member and layer in fragments over
// chunks of 32 batch rows: inputs act[b][k] as tiles of 16 k, gradients D[b][n]
// as tiles of 16 n, lane l holding row 32 c + 8 (l / 16) + i of column
// 16 t + l % 16; rows beyond the batch are zero.  cb = chunks of the batch.
constexpr int kTilesK[kLayers] = {5, 16, 16, 16};
constexpr int kActTiles = 5 + 3 * 16, kGradTiles = 3 * 16 + 2;
constexpr int act_tile(int l) { return l == 0 ? 0 : 5 + 16 * (l - 1); }
constexpr int grad_tile(int l) { return 16 * l; }
// FP32 gradients of the biases' sums: D[b][n] of all layers, 785 columns
constexpr int kGradCols = 3 * kHidden + kOut;
constexpr int grad_col(int l) { return l * kHidden; }
inline int batch_chunks(int bsz) { return (bsz + 31) / 32; }

struct Batch {
  const float *X, *T;      // standardised rows [n][80], targets [n][17]
  const int *idx;          // row of batch entry b of member z: idx[z idx_stride + b]
  long long idx_stride;    //   (null: row b)
  int bsz, members;
  const bf16 *wp;
  bf16 *actp;              // [members][kActTiles][cb][512]
  bf16 *gradp;             // [members][kGradTiles][cb][512]
  float *gradf;            // [members][bsz][kGradCols]
  double *lossp;           // [members][2 cb] squared errors of 16 rows
};
struct AdamStep {
  float lr, b1, b2, eps, bc1, bc2;
};
hipError_t launch_fb(const Batch &q, const float *w, hipStream_t st);
// gradients into g (adam null), or Adam on w, m, v and the packed weights
// wp; loss[z] = mean squared error of the batch (FP64)
hipError_t launch_update(const Batch &q, float *g, float *w, float *m, float *v, bf16 *wp,
                         const AdamStep *adam, double *loss, hipStream_t st);
// ensemble mean / population std of the de-standardised outputs
hipError_t launch_ensemble(const float *Y, int members, int n, long long cap, const double *mu,
                           const double *sd, double *mean, double *std, hipStream_t st);
// descriptor of n four-sphere throats: geo[n][19] = 4 spheres (cx, cy, cz, r;
// throat spheres first) and nx, ny, nz; feat [n][80]
hipError_t launch_describe(const double *geo, int n, double *feat, hipStream_t st);

}  // namespace sg
