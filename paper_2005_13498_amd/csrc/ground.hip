// Ground-state Lanczos kernels: complex double, one vector.  An iteration is
// the H v kernels and two launches, with no host wait in between: inner
// products and subtraction of the two vectors that H v overlaps with (and of
// the deflated one).  The last two iterations of a batch
// have the same two launches once more against every vector, which takes out
// what the three-term recurrence let grow back; gs_lanczos checks how much
// that was.  Vectors are stored as subtracted, with their norms beside them.
// Inner products of small sectors are latency-bound, so the (vector, chunk)
// pairs are spread over workgroups and the subtraction adds the few partial
// rows itself and reads the vectors in independent groups of eight.
// 10 sites (63,504 states): the subtraction of up to 60 vectors took 56 us on
// average when each vector's load waited for the last, 8 us now (4 TB/s out of
// the caches).  A whole ground state with its gap took 192 ms with a dense
// eigenproblem, three waits on the host per iteration and start vectors from
// the host, 12.6 ms with every product against every vector of up to 60, and
// 5.5 ms now (240 iterations, whose three launches of 5 to 7 us bound it).
#include "ground.h"

#include <algorithm>

#include "kernels_common.h"

namespace hub {
namespace dev {

namespace {

constexpr int kDotVecs = 4;   // vectors per inner-product workgroup
constexpr int kSubVecs = 8;   // vectors whose loads a subtraction issues together
constexpr int kSubMost = 1024;  // vectors of one subtraction launch (coefficients in LDS)

__device__ __forceinline__ int gs_index(const GsBasis& B, int k) {  // in V, or -1: deflate
  return B.deflate ? (k == 0 ? -1 : B.first + k - 1) : B.first + k;
}
__device__ __forceinline__ const double2* gs_vec(const GsBasis& B, int k) {
  const int i = gs_index(B, k);
  return i < 0 ? B.deflate : B.V + static_cast<int64_t>(i) * B.dim;
}
__device__ __forceinline__ double gs_inv(const GsBasis& B, int k) {
  const int i = gs_index(B, k);
  return i > 0 ? B.it[i - 1].inv : 1.0;
}

// beta = sqrt(sum of normp) and its inverse, by a workgroup.
__device__ __forceinline__ void gs_beta(const double* normp, int nrows, GsIter* it, double* red) {
  const double n = sqrt(reduce_column(normp, nrows, 1, 0, red));
  if (threadIdx.x == 0) {
    it->beta = n;
    it->inv = n > 0.0 ? 1.0 / n : 0.0;
  }
}

// Workgroup sum of |w|^2 into normp[blockIdx.x].
__device__ __forceinline__ void store_norm(double n2, double* red, double* normp) {
  const double s = block_sum(n2, red);
  if (threadIdx.x == 0) normp[blockIdx.x] = s;
}

}  // namespace

__global__ __launch_bounds__(kBlock) void k_gs_dot(GsBasis B, const double2* __restrict__ w, int64_t len,
                                                   double* dotp, const double* __restrict__ normp, int nrows,
                                                   GsIter* prev) {
  __shared__ double red[kWaves * 2 * kDotVecs];
  if (prev && blockIdx.x == 0 && blockIdx.y == 0) {  // the subtraction after this launch needs it first
    gs_beta(normp, nrows, prev, red);
    __syncthreads();
  }
  const int k0 = blockIdx.y * kDotVecs, K = min(kDotVecs, B.nb - k0);
  const double2* vp[kDotVecs];
#pragma unroll
  for (int k = 0; k < kDotVecs; ++k) vp[k] = gs_vec(B, k0 + min(k, K - 1));
  double acc[2 * kDotVecs];
#pragma unroll
  for (int q = 0; q < 2 * kDotVecs; ++q) acc[q] = 0.0;
  const int64_t i0 = blockIdx.x * len, i1 = min(B.dim, i0 + len);
#pragma unroll 2
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) {
    const double2 b = w[i];
#pragma unroll
    for (int k = 0; k < kDotVecs; ++k) {
      const double2 a = vp[k][i];
      acc[2 * k] += a.x * b.x + a.y * b.y;  // conj(a) b
      acc[2 * k + 1] += a.x * b.y - a.y * b.x;
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 2 * kDotVecs; ++q) {
    const double t = wave_sum(acc[q]);
    if (lane == 0) red[wv * 2 * kDotVecs + q] = t;
  }
  __syncthreads();
  if (threadIdx.x < 2 * K) {
    double t = 0.0;
    for (int k = 0; k < kWaves; ++k) t += red[k * 2 * kDotVecs + threadIdx.x];
    dotp[static_cast<size_t>(blockIdx.x) * 2 * B.nb + 2 * k0 + threadIdx.x] = t;
  }
}

// Vectors k0 .. k0 + kn of the basis; the last launch of a subtraction also
// leaves the norm partials and the coefficient of the last vector.  A
// workgroup takes 64 elements at a time and its wavefronts a quarter of the
// groups of kSubVecs vectors each, so that a small sector still has a few
// wavefronts per SIMD waiting on loads.
__global__ __launch_bounds__(kBlock) void k_gs_subtract(GsBasis B, int k0, int kn, double2* __restrict__ w,
                                                        const double* __restrict__ dotp, int rows, double* normp,
                                                        GsIter* it, int all) {
  __shared__ double2 part[kWaves][64];
  extern __shared__ double sc[];  // [2 kn], padded to a whole group of vectors
  const int groups = (kn + kSubVecs - 1) / kSubVecs;
  const bool last = k0 + kn == B.nb;
  const double inv = gs_inv(B, B.nb - 1);
  const double f = all || k0 > 0 ? 1.0 : inv;  // w's factor: once
  double l2 = 0.0;
  for (int t = threadIdx.x; t < 2 * kSubVecs * groups; t += kBlock) {
    double s = 0.0;
    if (t < 2 * kn) {
#pragma unroll 8
      for (int r = 0; r < rows; ++r) s += dotp[static_cast<size_t>(r) * 2 * B.nb + 2 * k0 + t];
      const double ik = gs_inv(B, k0 + (t >> 1));
      s *= ik * (all ? 1.0 : inv);  // <v_k, f w>
      l2 += s * s;
      if (last && t == 2 * (kn - 1) && blockIdx.x == 0) it->alpha = (all ? it->alpha : 0.0) + s;
      s *= ik;
    }
    sc[t] = s;
  }
  if (all && blockIdx.x == 0) {
    l2 = block_sum(l2, &part[0][0].x);
    if (threadIdx.x == 0) it->loss = k0 > 0 ? hypot(it->loss, sqrt(l2)) : sqrt(l2);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double n2 = 0.0;
  for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * 64; i0 < B.dim; i0 += static_cast<int64_t>(gridDim.x) * 64) {
    const int64_t i = i0 + lane;
    double2 t = double2{0.0, 0.0};
    if (i < B.dim)
      for (int g = wv; g < groups; g += kWaves) {
        double2 a[kSubVecs];
#pragma unroll
        for (int q = 0; q < kSubVecs; ++q) a[q] = gs_vec(B, k0 + min(g * kSubVecs + q, kn - 1))[i];
#pragma unroll
        for (int q = 0; q < kSubVecs; ++q) {  // padded vectors have zero coefficients
          const double cx = sc[2 * (g * kSubVecs + q)], cy = sc[2 * (g * kSubVecs + q) + 1];
          t.x += cx * a[q].x - cy * a[q].y;
          t.y += cx * a[q].y + cy * a[q].x;
        }
      }
    __syncthreads();  // the previous elements' parts are read
    part[wv][lane] = t;
    __syncthreads();
    if (wv == 0 && i < B.dim) {
      double2 o = w[i];
      o.x *= f;
      o.y *= f;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) {
        o.x -= part[q][lane].x;
        o.y -= part[q][lane].y;
      }
      w[i] = o;
      n2 += o.x * o.x + o.y * o.y;
    }
  }
  if (last && wv == 0) {
    n2 = wave_sum(n2);
    if (lane == 0) normp[blockIdx.x] = n2;
  }
}

__global__ __launch_bounds__(kBlock) void k_gs_combine(const double2* __restrict__ V, int64_t dim, int m,
                                                       const double* __restrict__ c, double2* __restrict__ out,
                                                       double* normp) {
  __shared__ double red[kWaves];
  double n2 = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    double2 t = double2{0.0, 0.0};
#pragma unroll 8
    for (int k = 0; k < m; ++k) {
      const double2 a = V[static_cast<int64_t>(k) * dim + i];
      t.x += c[k] * a.x;
      t.y += c[k] * a.y;
    }
    out[i] = t;
    n2 += t.x * t.x + t.y * t.y;
  }
  store_norm(n2, red, normp);
}

__global__ __launch_bounds__(kBlock) void k_gs_beta(const double* __restrict__ normp, int nrows, GsIter* it) {
  __shared__ double red[kWaves];
  gs_beta(normp, nrows, it, red);
}

__global__ __launch_bounds__(kBlock) void k_gs_scale(int64_t dim, const double2* x, const double* __restrict__ normp,
                                                     int nrows, double2* dst, double2* dst2) {
  __shared__ double red[kWaves];
  const double n = sqrt(reduce_column(normp, nrows, 1, 0, red));
  const double f = n > 0.0 ? 1.0 / n : 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const double2 t = x[i];
    const double2 o = double2{f * t.x, f * t.y};
    dst[i] = o;
    if (dst2) dst2[i] = o;
  }
}

// Counter-based: element i mixes (seed, i) to 64 random bits twice (the
// finaliser of Steele, Lea and Flood's SplitMix64) and takes the pair of normal
// numbers of Box and Muller.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
  return z ^ (z >> 31);
}

__global__ __launch_bounds__(kBlock) void k_gs_start(int64_t dim, uint64_t seed, double2* x, double* normp) {
  __shared__ double red[kWaves];
  double n2 = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const uint64_t a = mix64(mix64(seed) + 0x9e3779b97f4a7c15ULL * (2 * static_cast<uint64_t>(i) + 1));
    const uint64_t b = mix64(mix64(seed) + 0x9e3779b97f4a7c15ULL * (2 * static_cast<uint64_t>(i) + 2));
    const double u = (static_cast<double>(a >> 11) + 0.5) * 0x1p-53, p = static_cast<double>(b >> 11) * 0x1p-53;
    const double r = sqrt(-2.0 * log(u));
    double sn, cs;
    sincospi(2.0 * p, &sn, &cs);
    const double2 t = double2{r * cs, r * sn};
    x[i] = t;
    n2 += t.x * t.x + t.y * t.y;
  }
  store_norm(n2, red, normp);
}

__global__ __launch_bounds__(kBlock) void k_gs_absmax(int64_t dim, const double2* x, double* partials) {
  __shared__ double red[kWaves];
  double m = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const double2 t = x[i];
    m = fmax(m, t.x * t.x + t.y * t.y);
  }
  m = wave_max(m);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kWaves; ++k) m = fmax(m, red[k]);
    partials[blockIdx.x] = m;
  }
}

// first[workgroup]: the workgroup's lowest index with |x_i| within 1e-12 of
// the largest modulus (dim: none).
__global__ __launch_bounds__(kBlock) void k_gs_first(int64_t dim, const double2* x, const double* partials, int nrows,
                                                     int64_t* first) {
  __shared__ double red[kWaves];
  __shared__ int64_t best[kWaves];
  double m = 0.0;
  for (int b = threadIdx.x; b < nrows; b += kBlock) m = fmax(m, partials[b]);
  m = wave_max(m);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) red[wv] = m;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kWaves; ++k) m = fmax(m, red[k]);
  const double th = m * (1.0 - 1e-12) * (1.0 - 1e-12);
  int64_t r = dim;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim && r == dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const double2 t = x[i];
    if (t.x * t.x + t.y * t.y >= th) r = i;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) r = min(r, static_cast<int64_t>(__shfl_xor(static_cast<long long>(r), off)));
  if (lane == 0) best[wv] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kWaves; ++k) r = min(r, best[k]);
    first[blockIdx.x] = r;
  }
}

// factor = conj(c) / |c| of the first component c found.
__global__ void k_gs_factor(int64_t dim, const double2* x, const int64_t* first, int nrows, double* factor) {
  int64_t r = dim;
  for (int b = threadIdx.x; b < nrows; b += 64) r = min(r, first[b]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) r = min(r, static_cast<int64_t>(__shfl_xor(static_cast<long long>(r), off)));
  if (threadIdx.x == 0) {
    const double2 c = r < dim ? x[r] : double2{1.0, 0.0};
    const double mag = hypot(c.x, c.y);
    factor[0] = c.x / mag;
    factor[1] = -c.y / mag;
  }
}

__global__ __launch_bounds__(kBlock) void k_gs_rotate(int64_t dim, double2* x, const double* factor) {
  const double fx = factor[0], fy = factor[1];
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; i < dim;
       i += static_cast<int64_t>(gridDim.x) * kBlock) {
    const double2 t = x[i];
    x[i] = double2{fx * t.x - fy * t.y, fx * t.y + fy * t.x};
  }
}

}  // namespace dev
using namespace dev;

// One element per thread until every compute unit has four workgroups.
static int gs_grid(int64_t dim) {
  return static_cast<int>(std::min<int64_t>((dim + kBlock - 1) / kBlock, kGsNormRows));
}

hipError_t launch_gs_dot(const GsBasis& B, const double2* w, double* dotp, int* rows, const double* normp, int nrows,
                         GsIter* prev, hipStream_t s) {
  // about 512 workgroups of at least 1,024 elements
  const int groups = (B.nb + kDotVecs - 1) / kDotVecs;
  const int64_t most = std::max<int64_t>(1, (B.dim + 1023) / 1024);
  const int c = static_cast<int>(std::min<int64_t>({most, kGsDotRows, std::max(1, 512 / groups)}));
  const int64_t len = ((B.dim + c - 1) / c + kBlock - 1) / kBlock * kBlock;
  hipLaunchKernelGGL(k_gs_dot, dim3(c, groups), dim3(kBlock), 0, s, B, w, len, dotp, normp, nrows, prev);
  *rows = c;
  return hipGetLastError();
}

hipError_t launch_gs_subtract(const GsBasis& B, double2* w, const double* dotp, int rows, double* normp, int* nrows,
                              GsIter* it, bool all, hipStream_t s) {
  const int grid = static_cast<int>(std::min<int64_t>((B.dim + 63) / 64, kGsNormRows));
  for (int k0 = 0; k0 < B.nb; k0 += kSubMost) {
    const int kn = std::min(kSubMost, B.nb - k0);
    const size_t lds = static_cast<size_t>((kn + kSubVecs - 1) / kSubVecs) * kSubVecs * 2 * sizeof(double);
    hipLaunchKernelGGL(k_gs_subtract, dim3(grid), dim3(kBlock), lds, s, B, k0, kn, w, dotp, rows, normp, it,
                       all ? 1 : 0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  *nrows = grid;
  return hipSuccess;
}

hipError_t launch_gs_combine(const double2* V, int64_t dim, int m, const double* c, double2* out, double* normp,
                             int* nrows, hipStream_t s) {
  *nrows = gs_grid(dim);
  hipLaunchKernelGGL(k_gs_combine, dim3(*nrows), dim3(kBlock), 0, s, V, dim, m, c, out, normp);
  return hipGetLastError();
}

hipError_t launch_gs_beta(const double* normp, int nrows, GsIter* it, hipStream_t s) {
  hipLaunchKernelGGL(k_gs_beta, dim3(1), dim3(kBlock), 0, s, normp, nrows, it);
  return hipGetLastError();
}

hipError_t launch_gs_scale(int64_t dim, const double2* x, const double* normp, int nrows, double2* dst, double2* dst2,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_gs_scale, dim3(gs_grid(dim)), dim3(kBlock), 0, s, dim, x, normp, nrows, dst, dst2);
  return hipGetLastError();
}

hipError_t launch_gs_start(int64_t dim, uint64_t seed, double2* x, double* normp, int* nrows, hipStream_t s) {
  *nrows = gs_grid(dim);
  hipLaunchKernelGGL(k_gs_start, dim3(*nrows), dim3(kBlock), 0, s, dim, seed, x, normp);
  return hipGetLastError();
}

hipError_t launch_gs_phase(int64_t dim, double2* x, double* partials, int64_t* first, hipStream_t s) {
  const int grid = gs_grid(dim);
  hipLaunchKernelGGL(k_gs_absmax, dim3(grid), dim3(kBlock), 0, s, dim, x, partials);
  hipLaunchKernelGGL(k_gs_first, dim3(grid), dim3(kBlock), 0, s, dim, x, partials, grid, first);
  // the partials are read; their first two entries take the factor
  hipLaunchKernelGGL(k_gs_factor, dim3(1), dim3(64), 0, s, dim, x, first, grid, partials);
  hipLaunchKernelGGL(k_gs_rotate, dim3(grid), dim3(kBlock), 0, s, dim, x, partials);
  return hipGetLastError();
}

}  // namespace hub
