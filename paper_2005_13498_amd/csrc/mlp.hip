// FP32 multilayer perceptron of the learned Krylov controller:
//   x (8) -> 64 -> GELU -> 64 -> GELU -> 1  (exact erf GELU),
// forward, gradient of the mean squared error, and Adam.  The forward alone
// (a chunk's few predictions) takes one wavefront per row: lane k owns hidden
// unit k of both layers, and the previous layer's activations are broadcast
// with lane reads.  Training runs forward and backward on the matrix cores;
// gradient partial sums are kept per workgroup and reduced by the Adam kernel
// in a fixed order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "gelu.h"
#include "hub.h"
#include "mlp.h"

namespace hub {
namespace dev {

constexpr int kIn = HUB_MLP_IN, kHid = HUB_MLP_HID, kOut = HUB_MLP_OUT, kP = HUB_MLP_NPARAM;
constexpr int oW1 = 0, oB1 = oW1 + kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid, oW3 = oB2 + kHid,
              oB3 = oW3 + kOut * kHid;
static_assert(oB3 + kOut == kP, "parameter layout");
constexpr int kMlpBlock = 256, kMlpWaves = kMlpBlock / 64;
constexpr int kGradStride = kP + 1;  // partial row: gradient, then the loss

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
struct GeluOps {
  static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
  static __device__ __forceinline__ float exp2(float x) { return __builtin_amdgcn_exp2f(x); }
};
__device__ __forceinline__ float lane_bcast(float v, int src) { return __shfl(v, src, 64); }
__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Per-lane parameter slice: lane k holds row k of W1 and W2, column k of W3.
struct Slice {
  float w1[kIn], b1, w2[kHid], b2, w3[kOut], b3[kOut];
};

__device__ __forceinline__ void load_slice(const float* __restrict__ P, int k, Slice& S) {
#pragma unroll
  for (int i = 0; i < kIn; ++i) S.w1[i] = P[oW1 + k * kIn + i];
  S.b1 = P[oB1 + k];
#pragma unroll
  for (int j = 0; j < kHid; ++j) S.w2[j] = P[oW2 + k * kHid + j];
  S.b2 = P[oB2 + k];
#pragma unroll
  for (int o = 0; o < kOut; ++o) {
    S.w3[o] = P[oW3 + o * kHid + k];
    S.b3[o] = P[oB3 + o];
  }
}

// Forward of one row on one wavefront; every lane ends with both outputs.
__device__ __forceinline__ void forward_row(const Slice& S, const float* __restrict__ x, float& z1, float& h1,
                                            float& z2, float& h2, float (&out)[kOut]) {
  float xi[kIn];
#pragma unroll
  for (int i = 0; i < kIn; ++i) xi[i] = x[i];
  z1 = S.b1;
#pragma unroll
  for (int i = 0; i < kIn; ++i) z1 = fmaf(S.w1[i], xi[i], z1);
  h1 = gelu(z1);
  z2 = S.b2;
#pragma unroll
  for (int j = 0; j < kHid; ++j) z2 = fmaf(S.w2[j], lane_bcast(h1, j), z2);
  h2 = gelu(z2);
#pragma unroll
  for (int o = 0; o < kOut; ++o) out[o] = wave_sum_f(S.w3[o] * h2) + S.b3[o];
}

__global__ __launch_bounds__(kMlpBlock) void k_mlp_forward(const float* __restrict__ P, int n_rows,
                                                           const float* __restrict__ feats,
                                                           float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * kMlpWaves + (threadIdx.x >> 6);
  const int nw = gridDim.x * kMlpWaves;
  Slice S;
  load_slice(P, lane, S);
  for (int r = wave; r < n_rows; r += nw) {
    float z1, h1, z2, h2, o[kOut];
    forward_row(S, feats + (size_t)r * kIn, z1, h1, z2, h2, o);
#pragma unroll
    for (int q = 0; q < kOut; ++q)
      if (lane == q) out[(size_t)r * kOut + q] = o[q];
  }
}

// Gradient of L = (1/n) sum_r |out_r - y_r|^2 on the matrix cores, FP32
// throughout (v_mfma_f32_16x16x4f32).  A wavefront takes a tile of 16 rows
// through forward and backward with the hidden units on the matrix rows and
// the data rows on its columns,
//   Z1^T = W1 X^T,  Z2^T = W2 H1^T,  dH1^T = W2^T dZ2^T,
// so that lane l of every result holds, for data row l % 16, the units
// 16 t + 4 (l / 16) + r (t: matrix tile, r: register): exactly the operand of
// the next product when its contraction runs over the units in the order
// (t, r, l / 16), which the weight fragments follow.  Only the weight
// gradients, contracted over the data rows, need the transposed operands:
// H1, dZ2 and dZ1 pass through a 16-row LDS tile of the wavefront (row stride
// 80 words: the four row groups of a read fall on different banks).  Column 8
// of gW1's feature operand is 1, so its product also gives the bias gradient.
// Bound: 216 matrix instructions of 32 cycles per tile, about as much again
// in the two GELUs, two wavefronts per SIMD to overlap the two: 5 us per tile
// of a SIMD, after 14 us for the first tile of a workgroup with its staging
// and sums.  A workgroup adds its eight wavefronts through LDS, 16 bytes a
// lane, the second of two rounds by every thread, which stores what it added
// (pairwise in three rounds, one wavefront storing, 3 us more; in turn, each
// adding to sums in LDS, 30 us more), and leaves one partial row.  48,000
// rows: 775 us with one row per wavefront and lane broadcasts, 30 us now; 45
// TFLOP/s, the matrix cores busy 28 % and the VALU 35 % of it.
using f32x4 = __attribute__((ext_vector_type(4))) float;
constexpr int kGradWaves = 8, kGradBlock = 64 * kGradWaves;
constexpr int kTile = 16;         // data rows of a wavefront's tile
constexpr int kTStride = 80;      // words per row of a transposed tile
constexpr int kMaxGradRows = 256; // partial rows (workgroups) of one train step
constexpr int kSums = 28;         // 16-byte words of a lane's gradient sums: gW2 16, gW1 4, gb2 4, gW3 4
static_assert(kHid == 64 && kIn == 8 && kOut == 1, "fragment layout of the gradient kernel");

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Orders a wavefront's own LDS writes before its later reads of other lanes'.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the 16 lanes (data rows) of a lane's row group, by rotations
// within the group (DPP row_ror: vector operands, no LDS permute).
template <int CTRL>
__device__ __forceinline__ float row_rotated(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_sum(float v) {
  v += row_rotated<0x128>(v);
  v += row_rotated<0x124>(v);
  v += row_rotated<0x122>(v);
  v += row_rotated<0x121>(v);
  return v;
}

__global__ __launch_bounds__(kGradBlock) void k_mlp_grad(const float* __restrict__ P, int n_rows,
                                                         const float* __restrict__ feats,
                                                         const float* __restrict__ targets,
                                                         float* __restrict__ part) {
  // fragments [unit tile][k tile][lane] of W2 (component r) and of its
  // transpose, then H1 and dZ2 (later dZ1) of every wavefront's tile
  // [row][unit]; at the end the sums of half the wavefronts
  constexpr int kTileWords = kTile * kTStride / 4;
  __shared__ f32x4 sh[2 * 16 * 64 + 2 * kGradWaves * kTileWords];
  static_assert(sizeof(sh) >= kGradWaves / 2 * kSums * 64 * sizeof(f32x4), "the wavefronts' sums reuse the tiles");
  f32x4* const fw2 = sh;
  f32x4* const fw2t = sh + 16 * 64;
  __shared__ f32x4 vb[3][kHid / 4];  // b1, b2 and w3, read where they are used (registers are short)
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int c = lane & 15, g = lane >> 4;  // matrix column (or operand row) and lane group
  for (int q = tid; q < 16 * 64; q += kGradBlock) {
    const int l = q & 63, kt = (q >> 6) & 3, it = q >> 8;
    const int i = 16 * it + (l & 15), k = 16 * kt + 4 * (l >> 4);
    f32x4 a, b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[r] = P[oW2 + i * kHid + k + r];
      b[r] = P[oW2 + (k + r) * kHid + i];
    }
    fw2[q] = a;
    fw2t[q] = b;
  }
  if (tid < kHid / 4)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vb[0][tid][r] = P[oB1 + 4 * tid + r];
      vb[1][tid][r] = P[oB2 + 4 * tid + r];
      vb[2][tid][r] = P[oW3 + 4 * tid + r];
    }
  float w1[4][2];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int s = 0; s < 2; ++s) w1[t][s] = P[oW1 + (16 * t + c) * kIn + 4 * s + g];
  const float b3 = P[oB3];
  const float inv_n = 1.0f / static_cast<float>(n_rows);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 gw2[4][4], gw1[4], gb2[4], gw3[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    gw1[t] = gb2[t] = gw3[t] = zero;
#pragma unroll
    for (int k = 0; k < 4; ++k) gw2[t][k] = zero;
  }
  float gb3 = 0.f, loss = 0.f;
  float* const H = reinterpret_cast<float*>(sh + 2 * 16 * 64 + 2 * wv * kTileWords);
  float* const D = H + kTile * kTStride;
  __syncthreads();

  const int tiles = (n_rows + kTile - 1) / kTile;
  for (int tile = blockIdx.x + wv * gridDim.x; tile < tiles; tile += kGradWaves * gridDim.x) {
    const int row = tile * kTile + c;
    const bool live = row < n_rows;
    float x[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) x[s] = live ? feats[(size_t)row * kIn + 4 * s + g] : 0.f;
    const float y = live ? targets[row] : 0.f;
    // the same rows' features as the second operand of gW1: [row 4 s + g][c]
    float xb[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int rr = tile * kTile + 4 * s + g;
      xb[s] = (c < kIn && rr < n_rows) ? feats[(size_t)rr * kIn + c] : (c == kIn ? 1.f : 0.f);
    }
    f32x4 h1[4], g1[4], dz[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 z = vb[0][4 * t + g];
#pragma unroll
      for (int s = 0; s < 2; ++s) z = mfma4(w1[t][s], x[s], z);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Gelu q = gelu_both<GeluOps>(z[r]);
        h1[t][r] = q.h;
        g1[t][r] = q.d;
      }
      *reinterpret_cast<f32x4*>(H + c * kTStride + 16 * t + 4 * g) = h1[t];
    }
    float o = 0.f;
    f32x4 h2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 z = vb[1][4 * t + g];
      const f32x4 w3 = vb[2][4 * t + g];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f32x4 w = fw2[(t * 4 + k) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) z = mfma4(w[r], h1[k][r], z);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Gelu q = gelu_both<GeluOps>(z[r]);
        h2[t][r] = q.h;
        dz[t][r] = q.d;
        o = fmaf(w3[r], h2[t][r], o);
      }
    }
    o += __shfl_xor(o, 16, 64);
    o += __shfl_xor(o, 32, 64);
    const float e = live ? o + b3 - y : 0.f;
    const float d = 2.0f * e * inv_n;  // dL/d out of this lane's row
    loss += e * e * inv_n;
    gb3 += d;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 w3 = vb[2][4 * t + g];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        gw3[t][r] = fmaf(d, h2[t][r], gw3[t][r]);
        dz[t][r] *= w3[r] * d;  // dZ2
        gb2[t][r] += dz[t][r];
      }
      *reinterpret_cast<f32x4*>(D + c * kTStride + 16 * t + 4 * g) = dz[t];
    }
    wave_lds_sync();
    // gW2 += dZ2^T H1 over the tile's rows
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float a[4], b[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[t] = D[(4 * s + g) * kTStride + 16 * t + c];
        b[t] = H[(4 * s + g) * kTStride + 16 * t + c];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) gw2[t][k] = mfma4(a[t], b[k], gw2[t][k]);
    }
    wave_lds_sync();
    // dZ1^T = (W2^T dZ2^T) gelu'(Z1^T), transposed into D
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 z = zero;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f32x4 w = fw2t[(t * 4 + k) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) z = mfma4(w[r], dz[k][r], z);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) z[r] *= g1[t][r];
      *reinterpret_cast<f32x4*>(D + c * kTStride + 16 * t + 4 * g) = z;
    }
    wave_lds_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) gw1[t] = mfma4(D[(4 * s + g) * kTStride + 16 * t + c], xb[s], gw1[t]);
    wave_lds_sync();  // the next tile rewrites H and D
  }

  // the lanes' bias, output-layer and loss sums over the data rows
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      gb2[t][r] = row_sum(gb2[t][r]);
      gw3[t][r] = row_sum(gw3[t][r]);
    }
  gb3 = row_sum(gb3);
  loss = row_sum(loss);
  // the wavefronts' sums in a fixed order: the upper half is added to the
  // lower, then every thread adds those four for 3.5 of the words and stores
  f32x4 sums[kSums];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sums[4 * t + k] = gw2[t][k];
    sums[16 + t] = gw1[t];
    sums[20 + t] = gb2[t];
    sums[24 + t] = gw3[t];
  }
  __shared__ float scal[2][kGradWaves];
  if (lane == 0) {
    scal[0][wv] = gb3;
    scal[1][wv] = loss;
  }
  constexpr int kHalf = kGradWaves / 2;
  __syncthreads();  // the tiles are no longer read
  if (wv >= kHalf)
#pragma unroll
    for (int k = 0; k < kSums; ++k) sh[((wv - kHalf) * kSums + k) * 64 + lane] = sums[k];
  __syncthreads();
  if (wv < kHalf)  // each lane rewrites the words that it alone has read
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
      const int q = (wv * kSums + k) * 64 + lane;
      sh[q] = sums[k] + sh[q];
    }
  __syncthreads();
  float* const G = part + (size_t)blockIdx.x * kGradStride;
  for (int k = wv; k < kSums; k += kGradWaves) {
    f32x4 q = sh[k * 64 + lane];
#pragma unroll
    for (int w = 1; w < kHalf; ++w) q += sh[(w * kSums + k) * 64 + lane];
    const int t = k < 16 ? k >> 2 : k & 3;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 16 * t + 4 * g + r;  // matrix row: the unit of the outer layer
      if (k < 16) G[oW2 + u * kHid + 16 * (k & 3) + c] = q[r];
      else if (k < 20 && c < kIn) G[oW1 + u * kIn + c] = q[r];
      else if (k < 20 && c == kIn) G[oB1 + u] = q[r];
      else if (k >= 20 && c == 0) G[(k < 24 ? oB2 : oW3) + u] = q[r];
    }
  }
  if (wv != 0) return;
  if (lane < 2) {
    float q = 0.f;
    for (int w = 0; w < kGradWaves; ++w) q += scal[lane][w];
    G[lane == 0 ? oB3 : kP] = q;
  }
}

// Adam on the fixed-order sum of the workgroups' partials; parameter kP
// reports L.  kAdamSlices threads share a parameter, each with every
// kAdamSlices-th partial row (one thread per parameter waits out every row's
// load: 60 us for 256 rows; 5 us now, 7 with twice the parameters and half the
// threads each).
constexpr int kAdamCols = 32, kAdamSlices = 32;
__global__ __launch_bounds__(kAdamCols * kAdamSlices) void k_mlp_adam(const float* __restrict__ part, int n_part,
                                                                      float* __restrict__ P, float* __restrict__ m,
                                                                      float* __restrict__ v, int t, float lr,
                                                                      float* __restrict__ loss) {
  __shared__ float red[kAdamSlices][kAdamCols];
  const int c = threadIdx.x % kAdamCols, s = threadIdx.x / kAdamCols;
  const int p = blockIdx.x * kAdamCols + c;
  float sum = 0.f;
  if (p <= kP)
#pragma unroll 8
    for (int w = s; w < n_part; w += kAdamSlices) sum += part[(size_t)w * kGradStride + p];
  red[s][c] = sum;
  __syncthreads();
  if (s != 0 || p > kP) return;
  float g = 0.f;
#pragma unroll
  for (int k = 0; k < kAdamSlices; ++k) g += red[k][c];
  if (p == kP) {
    *loss = g;
    return;
  }
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mt = b1 * m[p] + (1.f - b1) * g;
  const float vt = b2 * v[p] + (1.f - b2) * g * g;
  m[p] = mt;
  v[p] = vt;
  const float mh = mt / (1.f - powf(b1, static_cast<float>(t)));
  const float vh = vt / (1.f - powf(b2, static_cast<float>(t)));
  P[p] -= lr * mh / (sqrtf(vh) + eps);
}

}  // namespace dev

// Partial rows (workgroups) of the gradient: one per tile of 16 rows up to a
// workgroup on every compute unit.
static int grad_parts(int n_rows) {
  const int tiles = (n_rows + dev::kTile - 1) / dev::kTile;
  return tiles < 1 ? 1 : (tiles > dev::kMaxGradRows ? dev::kMaxGradRows : tiles);
}

int64_t mlp_workspace_bytes(int n_rows) {
  const int64_t rows = (static_cast<int64_t>(n_rows) + 7) / 8;  // at least grad_parts
  return (rows > dev::kMaxGradRows ? dev::kMaxGradRows : (rows + 3) / 4 * 4) * dev::kGradStride * sizeof(float);
}

hipError_t launch_mlp_forward(const float* params, int n_rows, const float* feats, float* out, hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  int grid = (n_rows + dev::kMlpWaves - 1) / dev::kMlpWaves;
  grid = grid > 1024 ? 1024 : grid;
  hipLaunchKernelGGL(dev::k_mlp_forward, dim3(grid), dim3(dev::kMlpBlock), 0, s, params, n_rows, feats, out);
  return hipGetLastError();
}

hipError_t launch_mlp_train_step(float* params, float* m, float* v, int t, float lr, int n_rows, const float* feats,
                                 const float* targets, float* loss, void* workspace, hipStream_t s) {
  const int parts = grad_parts(n_rows);
  float* part = static_cast<float*>(workspace);
  hipLaunchKernelGGL(dev::k_mlp_grad, dim3(parts), dim3(dev::kGradBlock), 0, s, params, n_rows, feats, targets, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int grid = (dev::kP + 1 + dev::kAdamCols - 1) / dev::kAdamCols;
  hipLaunchKernelGGL(dev::k_mlp_adam, dim3(grid), dim3(dev::kAdamCols * dev::kAdamSlices), 0, s, part, parts, params,
                     m, v, t, lr, loss);
  return hipGetLastError();
}

}  // namespace hub
