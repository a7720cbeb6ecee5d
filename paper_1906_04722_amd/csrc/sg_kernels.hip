// sg_kernels.hip -- kernels of the learned entry-pressure surrogate on gfx950:
// the ensemble's forward in one kernel, a training batch in two (forward, loss
// gradient and backward; weight gradients and Adam on FP32 master weights), all
// on BF16 matrix-core products with FP32 accumulation, standardisation,
// ensemble statistics and the geometry + occupancy descriptor of a throat.
#include <hip/hip_runtime.h>

#include "geom.h"
#include "sg_internal.h"

namespace sg {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16 to_bf16(float f) {
  // round to nearest, ties to even (inputs are finite)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16)(u >> 16);
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// Products are v_mfma_f32_16x16x32_bf16 (gfx950).  Operand layout of that
// instruction (64 lanes, 8 values each): lane l holds A[l % 16][8 (l / 16) + i]
// and B[8 (l / 16) + i][l % 16]; the result C[4 (l / 16) + i][l % 16].
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// ---- ensemble forward in one kernel --------------------------------------------
__global__ void k_pack(const float *w, bf16 *wp, int members) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= members * kPack) return;
  const int z = (int)(i / kPack), r = (int)(i % kPack);
  int f = r / kFrag, l = 0, n, k;
  const int lane = (r % kFrag) / 8, j = r % 8;
  if (f < pack_off(kLayers)) {
    while (l + 1 < kLayers && f >= pack_off(l + 1)) ++l;
    f -= pack_off(l);
    n = 16 * (f / kChunksK[l]) + lane % 16;
    k = 32 * (f % kChunksK[l]) + 8 * (lane / 16) + j;
  } else {
    l = 1;
    while (l + 1 < kLayers && f >= packt_off(l + 1)) ++l;
    f -= packt_off(l);
    k = 16 * (f / kChunksN[l]) + lane % 16;
    n = 32 * (f % kChunksN[l]) + 8 * (lane / 16) + j;
  }
  const bool in = n < kWidth[l + 1] && k < kWidth[l];
  wp[i] = in ? to_bf16(w[(long long)z * kParams + w_off(l) + (long long)n * kWidth[l] + k])
             : (bf16)0;
}

hipError_t launch_pack(const float *w, bf16 *wp, int members, hipStream_t st) {
  const long long total = members * kPack;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, w, wp,
                     members);
  return hipGetLastError();
}

// Rows of activations in LDS, k-contiguous; 264 (104) values apart, so that
// the 16 rows of an operand start in different banks.
constexpr int LDA = kHidden + 8, LDX = 32 * kChunksK[0] + 8;

// acc[t][j] = W tiles (rows) times activation tiles (columns): TPW output
// tiles from `tile0`, MT tiles of 16 rows of the batch in `in`
template <int L, int MT, int TPW, int LD>
__device__ __forceinline__ void layer_acc(const bf16 *wp, const bf16 *in, int tile0, int lane,
                                          v4f (&acc)[TPW][MT]) {
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[t][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kChunksK[L]; ++c) {
    v8bf a[TPW], b[MT];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
      a[t] = *(const v8bf *)(wp + ((long long)(pack_off(L) + (tile0 + t) * kChunksK[L] + c) * 64 +
                                   lane) * 8);
#pragma unroll
    for (int j = 0; j < MT; ++j)
      b[j] = *(const v8bf *)(in + (16 * j + (lane & 15)) * LD + 32 * c + 8 * (lane >> 4));
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int j = 0; j < MT; ++j)
        acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[j], acc[t][j], 0, 0, 0);
  }
}

// The same in two halves for workgroups of one row tile: the weights of a
// layer go to registers while the layer before it is still in its barriers,
// which hides their trip from the L2.
template <int OFF, int TPW, int C>
__device__ __forceinline__ void frag_load(const bf16 *wp, int tile0, int lane, v8bf (&a)[TPW][C]) {
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int c = 0; c < C; ++c)
      a[t][c] = *(const v8bf *)(wp + ((long long)(OFF + (tile0 + t) * C + c) * 64 + lane) * 8);
}
template <int TPW, int C, int LD>
__device__ __forceinline__ void frag_mul(const v8bf (&a)[TPW][C], const bf16 *in, int lane,
                                         v4f (&acc)[TPW][1]) {
#pragma unroll
  for (int t = 0; t < TPW; ++t) acc[t][0] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const v8bf b = *(const v8bf *)(in + (lane & 15) * LD + 32 * c + 8 * (lane >> 4));
#pragma unroll
    for (int t = 0; t < TPW; ++t)
      acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][c], b, acc[t][0], 0, 0, 0);
  }
}

// a hidden layer's bias and SiLU; the result goes to act once every wavefront
// has read the layer's input
template <int L, int MT, int TPW>
__device__ __forceinline__ void layer_silu(const float *w, int tile0, int lane,
                                           const v4f (&acc)[TPW][MT], bf16 *act) {
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int n = 16 * (tile0 + t) + 4 * (lane >> 4);
    float bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i] = w[b_off(L) + n + i];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      uint2 q;
      bf16 *e = (bf16 *)&q;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float zz = acc[t][j][i] + bias[i];
        e[i] = to_bf16(silu(zz));
      }
      *(uint2 *)(act + (16 * j + (lane & 15)) * LDA + n) = q;
    }
  }
  __syncthreads();
}

// One workgroup carries 16 MT rows through all four layers of `per` members:
// the activations stay in LDS, the weights come as whole packed fragments
// straight into the operand registers.  Each wavefront owns 16 / NW output
// tiles of a hidden layer.
//
// Bound: a workgroup reads a member's 320 KB of weights from the L2 for every
// 16 MT rows; at MT = 4 that is as many bytes per clock as a CU can take while
// its matrix cores run at full rate.  One row tile per workgroup (MT = 1) and
// one member per workgroup spread a small call over the chip.
template <int MT, int NW>
__global__ __launch_bounds__(64 * NW) void k_mlp(const double *X, const double *mu,
                                                 const double *sd, int n, int per,
                                                 const bf16 *wp, const float *w, float *y,
                                                 long long ycap, int *bad) {
  constexpr int TPW = 16 / NW;
  __shared__ __attribute__((aligned(16))) bf16 x0[16 * MT * LDX];
  __shared__ __attribute__((aligned(16))) bf16 act[16 * MT * LDA];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row0 = blockIdx.x * 16 * MT;
  bool finite = true;
  for (int e = tid; e < 16 * MT * 32 * kChunksK[0]; e += 64 * NW) {
    const int r = e / (32 * kChunksK[0]), c = e % (32 * kChunksK[0]);
    bf16 v = 0;
    if (c < kFeat && row0 + r < n) {
      const double x = X[(long long)(row0 + r) * kFeat + c];
      finite = finite && isfinite(x);
      v = to_bf16((float)((x - mu[c]) / sd[c]));
    }
    x0[r * LDX + c] = v;
  }
  if (!finite) *bad = 1;
  __syncthreads();
  for (int z = blockIdx.y * per; z < (int)(blockIdx.y + 1) * per; ++z) {
    const bf16 *wz = wp + z * kPack;
    const float *pz = w + z * kParams;
    v4f acc[TPW][MT], out[1][MT];
    if constexpr (MT == 1) {
      v8bf a0[TPW][kChunksK[0]], a1[TPW][kChunksK[1]], a2[TPW][kChunksK[2]], a3[1][kChunksK[3]];
      frag_load<pack_off(0)>(wz, wv * TPW, lane, a0);
      frag_load<pack_off(1)>(wz, wv * TPW, lane, a1);
      frag_mul<TPW, kChunksK[0], LDX>(a0, x0, lane, acc);
      layer_silu<0, MT, TPW>(pz, wv * TPW, lane, acc, act);
      frag_load<pack_off(2)>(wz, wv * TPW, lane, a2);
      frag_mul<TPW, kChunksK[1], LDA>(a1, act, lane, acc);
      layer_silu<1, MT, TPW>(pz, wv * TPW, lane, acc, act);
      if (wv < kTilesN[3]) frag_load<pack_off(3)>(wz, wv, lane, a3);
      frag_mul<TPW, kChunksK[2], LDA>(a2, act, lane, acc);
      layer_silu<2, MT, TPW>(pz, wv * TPW, lane, acc, act);
      if (wv < kTilesN[3]) frag_mul<1, kChunksK[3], LDA>(a3, act, lane, out);
    } else {
      layer_acc<0, MT, TPW, LDX>(wz, x0, wv * TPW, lane, acc);
      layer_silu<0, MT, TPW>(pz, wv * TPW, lane, acc, act);
      layer_acc<1, MT, TPW, LDA>(wz, act, wv * TPW, lane, acc);
      layer_silu<1, MT, TPW>(pz, wv * TPW, lane, acc, act);
      layer_acc<2, MT, TPW, LDA>(wz, act, wv * TPW, lane, acc);
      layer_silu<2, MT, TPW>(pz, wv * TPW, lane, acc, act);
      if (wv < kTilesN[3]) layer_acc<3, MT, 1, LDA>(wz, act, wv, lane, out);
    }
    if (wv < kTilesN[3]) {
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int o = 16 * wv + 4 * (lane >> 4) + i, row = row0 + 16 * j + (lane & 15);
          if (o < kOut && row < n)
            y[(z * ycap + row) * kOut + o] = out[0][j][i] + pz[b_off(3) + o];
        }
    }
  }
}

hipError_t launch_mlp(const double *X, const double *mu, const double *sd, int n, int members,
                      const bf16 *wp, const float *w, float *y, long long ycap, int *bad,
                      hipStream_t st) {
  if (n <= 0) return hipSuccess;
  // 64 rows a workgroup once that gives every CU two of them
  const int big = (n + 63) / 64;
  if (big >= 512)
    hipLaunchKernelGGL((k_mlp<4, 4>), dim3((unsigned)big, 1), dim3(256), 0, st, X, mu, sd, n,
                       members, wp, w, y, ycap, bad);
  else if (big * members >= 512)
    hipLaunchKernelGGL((k_mlp<4, 4>), dim3((unsigned)big, (unsigned)members), dim3(256), 0, st, X,
                       mu, sd, n, 1, wp, w, y, ycap, bad);
  else
    hipLaunchKernelGGL((k_mlp<1, 8>), dim3((unsigned)((n + 15) / 16), (unsigned)members),
                       dim3(512), 0, st, X, mu, sd, n, 1, wp, w, y, ycap, bad);
  return hipGetLastError();
}

// ---- fixed-order block reduction (FP64) -------------------------------------
template <int NT>
__device__ __forceinline__ double block_sum(double v, double *sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(256) void k_col_stats(const double *X, int n, int cols, double *mu,
                                                   double *sd) {
  __shared__ double sh[256];
  const int c = blockIdx.x;
  double s = 0;
  for (int i = threadIdx.x; i < n; i += 256) s += X[(long long)i * cols + c];
  const double mean = block_sum<256>(s, sh) / n;
  double q = 0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double d = X[(long long)i * cols + c] - mean;
    q += d * d;
  }
  const double var = block_sum<256>(q, sh) / n;
  if (threadIdx.x == 0) {
    mu[c] = mean;
    const double s2 = sqrt(var);
    sd[c] = s2 < 1e-12 ? 1.0 : s2;
  }
}

hipError_t launch_col_stats(const double *X, int n, int cols, double *mu, double *sd,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_col_stats, dim3((unsigned)cols), dim3(256), 0, st, X, n, cols, mu, sd);
  return hipGetLastError();
}

__global__ void k_standardise(const double *X, long long total, int cols, const double *mu,
                              const double *sd, float *Y) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % cols);
  Y[i] = (float)((X[i] - mu[c]) / sd[c]);
}

hipError_t launch_standardise(const double *X, int n, int cols, const double *mu,
                              const double *sd, float *Y, hipStream_t st) {
  const long long total = (long long)n * cols;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_standardise, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X,
                     total, cols, mu, sd, Y);
  return hipGetLastError();
}

// ---- training -----------------------------------------------------------------
// Forward, loss gradient and backward of 16 batch rows of one member: nothing
// crosses rows, so a workgroup carries its rows down and up the four layers
// without leaving the CU.  The pre-activations stay in registers (the backward
// products leave d act in the lanes that hold the same z), activations and
// gradients in LDS; what the weight gradients need goes out in their operand
// layout.  The chain of seven dependent products bounds it, not their rate (5
// members x 64 rows are 20 workgroups): sixteen wavefronts of a tile each share
// a product, and the weights of a later product and the biases are loaded
// before the one that is being computed (each workgroup reads all weights, 0.6
// MB at 64 bytes a cycle 4 us).  5 members, batches of 64 rows on an MI355X:
// 17.1 us a batch (18.1 with eight wavefronts, 18.8 with two-byte stores of the
// operands too, 23 without the early loads) where a kernel per product,
// activation and bias gradient took eighteen launches and, with the download of
// the loss, 286 us (now 43 for both kernels and the host's share).
constexpr int kFbWaves = 16, kFbTiles = 16 / kFbWaves;

// four floats in a row, at any float's address
__device__ __forceinline__ void store4(float *p, const float (&x)[4]) {
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  *(f4 *)p = f4{x[0], x[1], x[2], x[3]};
}

// four values of column tile `tile` (columns 16 tile + 4 (lane / 16) + i) of
// batch row b into their fragments
__device__ __forceinline__ void put_frag(bf16 *frags, int tile, int cb, int b, int lane,
                                         const bf16 (&e)[4]) {
  bf16 *f = frags + ((long long)tile * cb + b / 32) * kFrag + (16 * ((b % 32) / 8)) * 8 + b % 8;
#pragma unroll
  for (int i = 0; i < 4; ++i) f[(4 * (lane >> 4) + i) * 8] = e[i];
}

// the 16 rows x 256 columns of `act` (LDS), rows b0 + r of the batch, into
// their fragments: eight rows of a column are one 16-byte store
__device__ __forceinline__ void put_frags(const bf16 *act, bf16 *frags, int tile0, int cb, int b0,
                                          int tid) {
#pragma unroll
  for (int e = tid; e < 16 * 32; e += 64 * kFbWaves) {
    const int l = e % 32, n = 16 * (e / 32) + l % 16;
    v8bf x;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      x[i] = __builtin_bit_cast(__bf16, act[(8 * (l / 16) + i) * LDA + n]);
    *(v8bf *)(frags + ((long long)(tile0 + e / 32) * cb + b0 / 32) * kFrag +
              (16 * ((b0 % 32) / 8 + l / 16) + l % 16) * 8) = x;
  }
}

template <int L>
__device__ __forceinline__ void fb_forward(const v4f (&acc)[kFbTiles][1],
                                           const float (&bias)[kFbTiles][4], bf16 *out,
                                           bf16 *actp, int cb, bool live, int wv, int lane,
                                           float (&z)[kFbTiles][4]) {
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kFbTiles; ++t) {
    const int tile = wv * kFbTiles + t, n = 16 * tile + 4 * (lane >> 4);
    bf16 e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float zz = acc[t][0][i] + bias[t][i];
      z[t][i] = zz;
      e[i] = live ? to_bf16(silu(zz)) : (bf16)0;
    }
    uint2 w2;
    w2.x = (uint32_t)e[0] | (uint32_t)e[1] << 16;
    w2.y = (uint32_t)e[2] | (uint32_t)e[3] << 16;
    *(uint2 *)(out + (lane & 15) * LDA + n) = w2;
  }
  __syncthreads();
  put_frags(out, actp, act_tile(L + 1), cb, blockIdx.x * 16, 64 * wv + lane);
}

// gradients of layer L - 1's pre-activations: d act of layer L's input (acc, in
// the lanes that hold the same z) times silu' of z
template <int L>
__device__ __forceinline__ void fb_backward(const v4f (&acc)[kFbTiles][1], bf16 *out, bf16 *gradp,
                                            float *gradf, int cb, int row, bool live, int wv,
                                            int lane, const float (&z)[kFbTiles][4]) {
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kFbTiles; ++t) {
    const int tile = wv * kFbTiles + t, n = 16 * tile + 4 * (lane >> 4);
    bf16 e[4];
    float d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      d[i] = acc[t][0][i] * dsilu(z[t][i]);
      e[i] = live ? to_bf16(d[i]) : (bf16)0;
    }
    if (live) store4(gradf + (long long)row * kGradCols + grad_col(L - 1) + n, d);
    uint2 w2;
    w2.x = (uint32_t)e[0] | (uint32_t)e[1] << 16;
    w2.y = (uint32_t)e[2] | (uint32_t)e[3] << 16;
    *(uint2 *)(out + (lane & 15) * LDA + n) = w2;
  }
  __syncthreads();
  put_frags(out, gradp, grad_tile(L - 1), cb, blockIdx.x * 16, 64 * wv + lane);
}

__global__ __launch_bounds__(64 * kFbWaves) void k_fb(Batch q, const float *w) {
  __shared__ __attribute__((aligned(16))) bf16 x0[16 * LDX];
  __shared__ __attribute__((aligned(16))) bf16 act[16 * LDA];
  __shared__ __attribute__((aligned(16))) bf16 dy[16 * (32 + 8)];
  __shared__ double sq[32];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int zm = blockIdx.y, cb = gridDim.x / 2;
  const int row = blockIdx.x * 16 + (lane & 15);  // of this lane's results
  const bool live = row < q.bsz;
  const bf16 *wz = q.wp + zm * kPack;
  const float *pz = w + zm * kParams;
  bf16 *actp = q.actp + (long long)zm * kActTiles * cb * kFrag;
  bf16 *gradp = q.gradp + (long long)zm * kGradTiles * cb * kFrag;
  float *gradf = q.gradf + (long long)zm * q.bsz * kGradCols;
  const int t0 = wv * kFbTiles;
  v8bf a0[kFbTiles][kChunksK[0]], a1[kFbTiles][kChunksK[1]], a2[kFbTiles][kChunksK[2]];
  v8bf a3[1][kChunksK[3]], r3[kFbTiles][kChunksN[3]], r2[kFbTiles][kChunksN[2]],
      r1[kFbTiles][kChunksN[1]];
  v4f acc[kFbTiles][1];
  frag_load<pack_off(0)>(wz, t0, lane, a0);
  frag_load<pack_off(1)>(wz, t0, lane, a1);
  float bias[3][kFbTiles][4];
#pragma unroll
  for (int l = 0; l < 3; ++l)
#pragma unroll
    for (int t = 0; t < kFbTiles; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        bias[l][t][i] = pz[b_off(l) + 16 * (t0 + t) + 4 * (lane >> 4) + i];
  for (int e = tid; e < 16 * 32 * kChunksK[0]; e += 64 * kFbWaves) {
    const int r = e / (32 * kChunksK[0]), c = e % (32 * kChunksK[0]), b = blockIdx.x * 16 + r;
    bf16 v = 0;
    if (c < kFeat && b < q.bsz) {
      const long long src = q.idx ? q.idx[zm * q.idx_stride + b] : b;
      v = to_bf16(q.X[src * kFeat + c]);
    }
    x0[r * LDX + c] = v;
    if (c < kFeat)
      actp[((long long)(c / 16) * cb + b / 32) * kFrag + (c % 16 + 16 * ((b % 32) / 8)) * 8 +
           b % 8] = v;
  }
  for (int e = tid; e < 16 * (32 + 8); e += 64 * kFbWaves) dy[e] = 0;
  __syncthreads();
  float z0[kFbTiles][4], z1[kFbTiles][4], z2[kFbTiles][4];
  frag_mul<kFbTiles, kChunksK[0], LDX>(a0, x0, lane, acc);
  fb_forward<0>(acc, bias[0], act, actp, cb, live, wv, lane, z0);
  frag_load<pack_off(2)>(wz, t0, lane, a2);
  frag_mul<kFbTiles, kChunksK[1], LDA>(a1, act, lane, acc);
  fb_forward<1>(acc, bias[1], act, actp, cb, live, wv, lane, z1);
  if (wv < kTilesN[3]) frag_load<pack_off(3)>(wz, wv, lane, a3);
  frag_load<packt_off(3)>(wz, t0, lane, r3);
  frag_mul<kFbTiles, kChunksK[2], LDA>(a2, act, lane, acc);
  fb_forward<2>(acc, bias[2], act, actp, cb, live, wv, lane, z2);
  frag_load<packt_off(2)>(wz, t0, lane, r2);
  if (wv < kTilesN[3]) {
    v4f out[1][1];
    frag_mul<1, kChunksK[3], LDA>(a3, act, lane, out);
    const float sc = 2.0f / (float)(q.bsz * kOut);
    const long long src = live ? (q.idx ? q.idx[zm * q.idx_stride + row] : row) : 0;
    double s = 0;
    bf16 e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 16 * wv + 4 * (lane >> 4) + i;
      e[i] = 0;
      if (o < kOut && live) {
        const float y = out[0][0][i] + pz[b_off(3) + o];
        const float d = y - q.T[src * kOut + o];
        const float gd = sc * d;
        gradf[(long long)row * kGradCols + grad_col(3) + o] = gd;
        e[i] = to_bf16(gd);
        dy[(lane & 15) * (32 + 8) + o] = e[i];
        s += (double)d * (double)d;
      }
    }
    put_frag(gradp, grad_tile(3) + wv, cb, row, lane, e);
    // squared errors in a fixed order: lanes 16 apart hold the same row
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) sq[wv] = s;
  }
  __syncthreads();
  if (tid == 0) q.lossp[zm * gridDim.x + blockIdx.x] = sq[0] + sq[1];
  frag_mul<kFbTiles, kChunksN[3], 32 + 8>(r3, dy, lane, acc);
  fb_backward<3>(acc, act, gradp, gradf, cb, row, live, wv, lane, z2);
  frag_load<packt_off(1)>(wz, t0, lane, r1);
  frag_mul<kFbTiles, kChunksN[2], LDA>(r2, act, lane, acc);
  fb_backward<2>(acc, act, gradp, gradf, cb, row, live, wv, lane, z1);
  frag_mul<kFbTiles, kChunksN[1], LDA>(r1, act, lane, acc);
  fb_backward<1>(acc, act, gradp, gradf, cb, row, live, wv, lane, z0);
}

hipError_t launch_fb(const Batch &q, const float *w, hipStream_t st) {
  const unsigned tiles = 2u * (unsigned)batch_chunks(q.bsz);
  hipLaunchKernelGGL(k_fb, dim3(tiles, (unsigned)q.members), dim3(64 * kFbWaves), 0, st, q, w);
  return hipGetLastError();
}

// One wavefront computes 32 inputs x 32 outputs of a layer's dW = D^T act over
// the whole batch and, while they are in its registers, takes the Adam step on
// those weights and refreshes their packed copies: gradients never go to
// memory.  The last workgroups sum the bias gradients (in batch order, so one
// chain per output) and the loss.  Bound by latency and by the accesses to the
// weights' rows: at a batch of 64, 9 MB of 5 members' weights and moments are
// read and written in 10.1 us; 13.9 with a store per float, 16.5 with a
// workgroup's wavefronts along the outputs, each line then written by two
// workgroups, 21.8 with the loads behind the products.
constexpr int wave_tiles(int l) { return ((kTilesK[l] + 1) / 2) * ((kTilesN[l] + 1) / 2); }
constexpr int kUpdWaves = wave_tiles(0) + wave_tiles(1) + wave_tiles(2) + wave_tiles(3);
static_assert(kUpdWaves % 4 == 0, "whole workgroups of four wavefronts");
constexpr int kBiasBlocks = 4;

// Adam on one weight: gradient g, first and second moments m, v
__device__ __forceinline__ float adam_step(const AdamStep &a, float g, float w, float &m,
                                           float &v) {
  // the two moments with one rounding of their last product and sum each,
  // written out so that every caller rounds alike
  m = fmaf(1.0f - a.b1, g, a.b1 * m);
  v = fmaf(g, (1.0f - a.b2) * g, a.b2 * v);
  return w - a.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.eps);
}

template <int L, bool ADAM>
__device__ __forceinline__ void update_tile(const Batch &q, int cb, int zm, int tile, int lane,
                                            float *g, float *w, float *m, float *v, bf16 *wp,
                                            const AdamStep &adam) {
  constexpr int KT = kTilesK[L], K = kWidth[L], N = kWidth[L + 1];
  // neighbouring wavefronts along the rows of W, which are contiguous
  const int kt = 2 * (tile % ((KT + 1) / 2)), nt = 2 * (tile / ((KT + 1) / 2));
  const bf16 *A = q.actp + ((long long)zm * kActTiles + act_tile(L) + kt) * cb * kFrag + lane * 8;
  const bf16 *B = q.gradp + ((long long)zm * kGradTiles + grad_tile(L) + nt) * cb * kFrag +
                  lane * 8;
  // (an odd last tile of inputs computes its partner on itself, unused)
  const long long ka = kt + 1 < KT ? (long long)cb * kFrag : 0;
  const long long kb = (long long)cb * kFrag;
  // weights and moments of this wavefront's 2 x 2 tiles, all in flight before
  // the products: four inputs of one output per lane and tile
  float w4[2][2][4], m4[2][2][4], v4[2][2][4];
  long long o[2][2];
  bool in[2][2];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
      const int k = 16 * (kt + ti) + 4 * (lane >> 4), n = 16 * (nt + tj) + (lane & 15);
      in[ti][tj] = kt + ti < KT && n < N;
      o[ti][tj] = (long long)zm * kParams + w_off(L) + (in[ti][tj] ? (long long)n * K + k : 0);
      if constexpr (ADAM)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          w4[ti][tj][i] = w[o[ti][tj] + i];
          m4[ti][tj][i] = m[o[ti][tj] + i];
          v4[ti][tj][i] = v[o[ti][tj] + i];
        }
    }
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < cb; ++c) {
    const v8bf a0 = *(const v8bf *)(A + (long long)c * kFrag);
    const v8bf a1 = *(const v8bf *)(A + ka + (long long)c * kFrag);
    const v8bf b0 = *(const v8bf *)(B + (long long)c * kFrag);
    const v8bf b1 = *(const v8bf *)(B + kb + (long long)c * kFrag);
    acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, acc[1][1], 0, 0, 0);
  }
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
      if (!in[ti][tj]) continue;
      const int k = 16 * (kt + ti) + 4 * (lane >> 4), n = 16 * (nt + tj) + (lane & 15);
      const long long at = o[ti][tj];
      if constexpr (!ADAM) {
        const float d[4] = {acc[ti][tj][0], acc[ti][tj][1], acc[ti][tj][2], acc[ti][tj][3]};
        store4(g + at, d);
      } else {
        bf16 e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          w4[ti][tj][i] = adam_step(adam, acc[ti][tj][i], w4[ti][tj][i], m4[ti][tj][i],
                                    v4[ti][tj][i]);
          e[i] = to_bf16(w4[ti][tj][i]);
        }
        store4(w + at, w4[ti][tj]);
        store4(m + at, m4[ti][tj]);
        store4(v + at, v4[ti][tj]);
        // four inputs in a row: one 8-byte store in the forward fragments, four
        // places in the transposed ones
        bf16 *p = wp + zm * kPack;
        uint2 w2;
        w2.x = (uint32_t)e[0] | (uint32_t)e[1] << 16;
        w2.y = (uint32_t)e[2] | (uint32_t)e[3] << 16;
        *(uint2 *)(p + (long long)(pack_off(L) + (n / 16) * kChunksK[L] + k / 32) * kFrag +
                   (n % 16 + 16 * ((k % 32) / 8)) * 8 + k % 8) = w2;
        if constexpr (L > 0) {
          bf16 *pt = p + (long long)(packt_off(L) + (k / 16) * kChunksN[L] + n / 32) * kFrag +
                     (k % 16 + 16 * ((n % 32) / 8)) * 8 + n % 8;
#pragma unroll
          for (int i = 0; i < 4; ++i) pt[8 * i] = e[i];
        }
      }
    }
}

template <bool ADAM>
__global__ __launch_bounds__(256) void k_update(Batch q, int cb, float *g, float *w, float *m,
                                                float *v, bf16 *wp, AdamStep adam, double *loss) {
  const int zm = blockIdx.y, lane = threadIdx.x & 63;
  int t = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (t < kUpdWaves) {
    if (t < wave_tiles(0)) return update_tile<0, ADAM>(q, cb, zm, t, lane, g, w, m, v, wp, adam);
    t -= wave_tiles(0);
    if (t < wave_tiles(1)) return update_tile<1, ADAM>(q, cb, zm, t, lane, g, w, m, v, wp, adam);
    t -= wave_tiles(1);
    if (t < wave_tiles(2)) return update_tile<2, ADAM>(q, cb, zm, t, lane, g, w, m, v, wp, adam);
    t -= wave_tiles(2);
    return update_tile<3, ADAM>(q, cb, zm, t, lane, g, w, m, v, wp, adam);
  }
  // biases: one layer per workgroup, one output per thread
  const int l = (int)blockIdx.x - kUpdWaves / 4, n = threadIdx.x;
  if (l == 3 && n == 255) {
    double s = 0;
    for (int i = 0; i < 2 * cb; ++i) s += q.lossp[zm * 2 * cb + i];
    loss[zm] = s / (q.bsz * kOut);
  }
  if (n >= kWidth[l + 1]) return;
  const float *d = q.gradf + (long long)zm * q.bsz * kGradCols + grad_col(l) + n;
  float s = 0.f;
  int b = 0;
  for (; b + 16 <= q.bsz; b += 16) {  // loads in flight together, added in order
    float e[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) e[i] = d[(long long)(b + i) * kGradCols];
#pragma unroll
    for (int i = 0; i < 16; ++i) s += e[i];
  }
  for (; b < q.bsz; ++b) s += d[(long long)b * kGradCols];
  const long long o = (long long)zm * kParams + b_off(l) + n;
  if constexpr (ADAM) {
    float mi = m[o], vi = v[o];
    w[o] = adam_step(adam, s, w[o], mi, vi);
    m[o] = mi;
    v[o] = vi;
  } else {
    g[o] = s;
  }
}

hipError_t launch_update(const Batch &q, float *g, float *w, float *m, float *v, bf16 *wp,
                         const AdamStep *adam, double *loss, hipStream_t st) {
  const dim3 grid(kUpdWaves / 4 + kBiasBlocks, (unsigned)q.members);
  const int cb = batch_chunks(q.bsz);
  if (adam)
    hipLaunchKernelGGL(k_update<true>, grid, dim3(256), 0, st, q, cb, g, w, m, v, wp, *adam, loss);
  else
    hipLaunchKernelGGL(k_update<false>, grid, dim3(256), 0, st, q, cb, g, w, m, v, wp, AdamStep{},
                       loss);
  return hipGetLastError();
}

__global__ void k_ensemble(const float *Y, int members, int n, long long cap, const double *mu,
                           const double *sd, double *mean, double *std) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= (long long)n * kOut) return;
  const int j = (int)(i % kOut);
  double s = 0;
  for (int z = 0; z < members; ++z) s += (double)Y[(long long)z * cap * kOut + i] * sd[j] + mu[j];
  const double mn = s / members;
  double q = 0;
  for (int z = 0; z < members; ++z) {
    const double d = (double)Y[(long long)z * cap * kOut + i] * sd[j] + mu[j] - mn;
    q += d * d;
  }
  mean[i] = mn;
  std[i] = sqrt(q / members);
}

hipError_t launch_ensemble(const float *Y, int members, int n, long long cap, const double *mu,
                           const double *sd, double *mean, double *std, hipStream_t st) {
  const long long total = (long long)n * kOut;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ensemble, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, Y,
                     members, n, cap, mu, sd, mean, std);
  return hipGetLastError();
}

// ---- descriptor -------------------------------------------------------------
// One workgroup per pooled cell (8^3 samples) and throat.  Sample i of an axis
// of length n sits at (i + 0.5) n / 32 - 0.5 lattice units; the point is solid
// if it is in a sphere or outside the prism over the throat spheres 0..2.
__global__ __launch_bounds__(512) void k_describe(const double *geo, double *feat) {
  const int cell = blockIdx.x, t = blockIdx.y;
  const double *G = geo + (long long)t * 19;
  const double *S = G;  // 4 spheres (cx, cy, cz, r), throat spheres first
  const double nx = G[16], ny = G[17], nz = G[18];
  const int k = kOcc / kPool;
  const int cx = cell % k, cy = (cell / k) % k, cz = cell / (k * k);
  const int tid = threadIdx.x;
  const int ix = cx * kPool + tid % kPool, iy = cy * kPool + (tid / kPool) % kPool,
            iz = cz * kPool + tid / (kPool * kPool);
  const double px = __dsub_rn(__dmul_rn(__dmul_rn((double)ix + 0.5, nx), 1.0 / kOcc), 0.5);
  const double py = __dsub_rn(__dmul_rn(__dmul_rn((double)iy + 0.5, ny), 1.0 / kOcc), 0.5);
  const double pz = __dsub_rn(__dmul_rn(__dmul_rn((double)iz + 0.5, nz), 1.0 / kOcc), 0.5);
  bool solid = !geom::in_prism(S, S + 4, S + 8, px, py);
  for (int i = 0; i < 4 && !solid; ++i) solid = geom::in_sphere(px, py, pz, S + 4 * i);
  const int cnt = __syncthreads_count(solid);
  double *f = feat + (long long)t * kFeat;
  if (tid == 0) f[16 + cell] = (double)cnt / (double)(kPool * kPool * kPool);
  if (cell == 0 && tid < 16) {
    const double rbar = __ddiv_rn(__dadd_rn(__dadd_rn(S[3], S[7]), S[11]), 3.0);
    if (tid < 4) {
      f[tid] = __ddiv_rn(S[4 * tid + 3], rbar);
    } else {
      const int s = (tid - 4) / 3, a = (tid - 4) % 3;
      const double c = __ddiv_rn(__dadd_rn(__dadd_rn(S[a], S[4 + a]), S[8 + a]), 3.0);
      f[tid] = __ddiv_rn(__dsub_rn(S[4 * s + a], c), rbar);
    }
  }
}

hipError_t launch_describe(const double *geo, int n, double *feat, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int k = kOcc / kPool;
  hipLaunchKernelGGL(k_describe, dim3((unsigned)(k * k * k), (unsigned)n), dim3(512), 0, st, geo,
                     feat);
  return hipGetLastError();
}

}  // namespace sg
