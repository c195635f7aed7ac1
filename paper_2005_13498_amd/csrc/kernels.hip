// HIP kernels for gfx950 (CDNA4, wave64): matrix-free Peierls-Hubbard apply
// with fused Lanczos epilogue and Krylov decision, Lanczos update, Krylov
// combine, and BLAS-1 helpers.
//
// Cross-workgroup reductions never use in-kernel fences (an agent-scope
// release writes back the whole L2 of an XCD).  Every kernel writes
// per-workgroup partial sums; the NEXT kernel on the stream sums them in a
// fixed order (kernel boundaries make them visible), so results are
// deterministic and bitwise reproducible.
#include "kernels_common.h"

#include <algorithm>
#include <cstdint>

namespace hub {
namespace dev {

// u_{j+1} = w - alpha_j s_j u_j in place (w holds s_j H u_j - beta s u_{j-1}),
// with alpha_j the fixed-order total of the apply's partials; |u_{j+1}|^2
// partials for the next apply.  Workgroup 0 records alpha_j and, after the
// step's first apply, the observables.
template <typename R, int NV>
__global__ __launch_bounds__(kBlock) void k_update(int64_t n, typename CT<R>::T* w,
                                                   const typename CT<R>::T* uj, VecState* st,
                                                   StepCtl* ctl, int j, const double* apply_partials,
                                                   int apply_nblk, int apply_nq, const double* row_obs,
                                                   int row_nblk, double* partials) {
  using V = typename CT<R>::T;
  __shared__ double red[kWaves * kMaxNV];
  __shared__ double sh_alpha[kMaxNV];
  if (ctl->all_done) return;
  const int tid = threadIdx.x;
  const int qn = apply_nq * NV;
  // alpha of vector v is column v
  cols_total<NV, kWaves>(cols_partial<NV, kBlock>(apply_partials, apply_nblk, qn), red, sh_alpha);
  if (blockIdx.x == 0) {
    if (tid < NV && st[tid].status == 0) st[tid].alpha[j] = sh_alpha[tid];
    if (!row_obs) {
      for (int t = NV; t < qn; ++t) {  // observables of the step's first vector
        const double s = reduce_column(apply_partials, apply_nblk, qn, t, red);
        if (tid == 0) st[t % NV].obs[t / NV - 1] = s;
      }
    } else {
      // two-pass apply: [diag, docc, n2, down-hop part] from the row pass,
      // the up-hop part of <x|K(t_obs)|x> in column 1 of the column pass
      for (int t = 0; t < kObsQ * NV; ++t) {
        double s = reduce_column(row_obs, row_nblk, kObsQ * NV, t, red);
        if (t / NV == kObsQ - 1) s += reduce_column(apply_partials, apply_nblk, qn, NV + t % NV, red);
        if (tid == 0) st[t % NV].obs[t / NV] = s;
      }
    }
  }
  const int v = tid % NV;
  const R c = static_cast<R>(sh_alpha[v] * st[v].scale[j]);
  double n2 = 0.0;
  const int64_t total = n * NV;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + tid; i < total; i += (int64_t)gridDim.x * kBlock) {
    const V u = uj[i];
    V t = w[i];
    t.x -= c * u.x;
    t.y -= c * u.y;
    w[i] = t;
    n2 += (double)t.x * t.x + (double)t.y * t.y;
  }
  block_partials<NV>(&n2, 1, red, partials + (size_t)blockIdx.x * NV);
}

// Records a finished step (workgroup 0 of its combine, or k_step_log):
// Krylov report into log, first-apply observables into obs_log, and a cleared
// control block; after a step where a vector hit m_max, the combines from
// sequence number seq + 1 on do nothing and the Lanczos kernels stay idle.
template <int NV>
__device__ void record_step(const VecState* st, StepCtl* ctl, CombineLog* log, double* obs_log, int nobs, int seq) {
  const int v = threadIdx.x;
  if (v < NV) {
    const VecState& S = st[v];
    if (log) {
      log[v].m = S.m;
      log[v].status = S.status;
      log[v].eps = S.eps;
      log[v].beta_last = S.m > 0 ? S.beta[S.m - 1] : 0.0;
    }
    if (obs_log)
      for (int k = 0; k < nobs; ++k) obs_log[v * nobs + k] = S.obs[k];
  }
  if (v == 0) {
    ctl->all_done = 0;
    ctl->any_maxed = 0;
    ctl->iter = 0;
    ctl->steps_done += 1;
    int maxed = 0;
    for (int w = 0; w < NV; ++w) maxed |= (st[w].status >= 3);
    if (maxed && log) {  // a vector hit m_max (or went non-finite): later enqueued steps do nothing
      ctl->halt_from = seq + 1;
      ctl->all_done = 1;
    }
  }
}

// One word of the state: VPL consecutive values.
template <typename R, int VPL>
struct __align__(sizeof(typename CT<R>::T) * VPL) StateWord {
  typename CT<R>::T v[VPL];
};

// |v|^2 partials of a state read word by word (the combine's result, or the
// input of a call's first step and of a step that is run again): both kernels
// add the same terms in the same order, so a step run again starts from the
// same bits.
template <int VPL, typename W>
__device__ __forceinline__ void word_norm(const W& o, double (&n2)[VPL]) {
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const double x = o.v[i].x, y = o.v[i].y;
    n2[i] = fma(x, x, fma(y, y, n2[i]));
  }
}
// Workgroup sums per vector, fixed order: partials[workgroup][NV].
template <int NV, int VPL>
__device__ __forceinline__ void word_norm_store(const double (&n2)[VPL], double* red, double* partials) {
  constexpr int L = NV > VPL ? NV / VPL : 1, kP = NV == 1 ? 1 : VPL;  // words per element, sums per word
  double s[kP];
#pragma unroll
  for (int i = 0; i < kP; ++i) s[i] = n2[i];
  if constexpr (NV == 1)
#pragma unroll
    for (int i = 1; i < VPL; ++i) s[0] += n2[i];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < kP; ++i) {
    double t = s[i];
#pragma unroll
    for (int off = 32; off >= L; off >>= 1) t += __shfl_xor(t, off);
    if (lane < L) red[wv * kMaxNV + lane * kP + i] = t;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double t = 0.0;
    for (int k = 0; k < kWaves; ++k) t += red[k * kMaxNV + threadIdx.x];
    partials[(size_t)blockIdx.x * NV + threadIdx.x] = t;
  }
}

// v <- beta0 sum_{k<m_v} s_k y_k u_k into slot 0, and |v|^2 partials for the
// next step's first apply; workgroup 0 then records the step (its other
// workgroups read the control block only at their start, and the record's
// halt applies from the next sequence number on).  Slot 0 is the state, slots
// 1, 2, .. lie `stride` words apart from `slots` on.  A thread takes a word of
// VPL values (16 bytes where the vectors are so aligned, else one value) and
// issues the loads of kCombineAhead slots together.  Eight vectors of 12
// sites (complex64, groups of 4 on two lanes, about seven slots): 119 us per
// group with one 8-byte value per thread and a pointer load per slot, 54 us
// now; one complex128 vector 21.9 and 19.3 us.
constexpr int kCombineAhead = 4;

template <typename R, int NV, int VPL>
__global__ __launch_bounds__(kBlock) void k_combine(int64_t words, typename CT<R>::T* state,
                                                    const typename CT<R>::T* slots, int64_t stride,
                                                    const VecState* st, StepCtl* ctl, double* partials, int seq,
                                                    CombineLog* log, double* obs_log, int nobs,
                                                    typename CT<R>::T* out2) {
  using V = typename CT<R>::T;
  using Word = StateWord<R, VPL>;
  constexpr int L = NV > VPL ? NV / VPL : 1;  // words per element (a word of one vector: consecutive elements)
  __shared__ double red[kWaves * kMaxNV];
  __shared__ double cr[kMaxNV][kMMax], ci[kMaxNV][kMMax];
  __shared__ int mv[kMaxNV];
  const int tid = threadIdx.x;
  // A step whose launches ended before every vector was decided is abandoned
  // with slot 0 unchanged; the flag makes the rest of the enqueued work idle.
  if (ctl->abort || (ctl->halt_from > 0 && seq >= ctl->halt_from)) return;
  bool undecided = false;
#pragma unroll
  for (int v = 0; v < NV; ++v) undecided |= (st[v].status == 0);
  if (undecided) {
    if (blockIdx.x == 0 && tid == 0) {
      ctl->abort = 1;
      ctl->all_done = 1;
    }
    return;
  }
  for (int t = tid; t < NV * kMMax; t += kBlock) {
    const int vv = t / kMMax, k = t % kMMax;
    const VecState& S = st[vv];
    const double f = S.beta0 * S.scale[k];
    cr[vv][k] = (k < S.m) ? f * S.y[2 * k] : 0.0;
    ci[vv][k] = (k < S.m) ? f * S.y[2 * k + 1] : 0.0;
    if (k == 0) mv[vv] = S.m;
  }
  __syncthreads();
  // vector of value i of this thread's words (kBlock and the grid's stride are multiples of L)
  int vec[VPL], m = 0;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    vec[i] = NV == 1 ? 0 : (tid % L) * VPL + i;
    m = max(m, mv[vec[i]]);
  }
  double n2[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) n2[i] = 0.0;
  Word* const out = reinterpret_cast<Word*>(state);
  const Word* const sl = reinterpret_cast<const Word*>(slots);
  for (int64_t w = (int64_t)blockIdx.x * kBlock + tid; w < words; w += (int64_t)gridDim.x * kBlock) {
    double ar[VPL], ai[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) ar[i] = ai[i] = 0.0;
    for (int k0 = 0; k0 < m; k0 += kCombineAhead) {
      Word u[kCombineAhead];
#pragma unroll
      for (int q = 0; q < kCombineAhead; ++q) {
        const int k = min(k0 + q, m - 1);
        u[q] = k == 0 ? out[w] : sl[(k - 1) * stride + w];
      }
#pragma unroll
      for (int q = 0; q < kCombineAhead; ++q)
#pragma unroll
        for (int i = 0; i < VPL; ++i)
          if (k0 + q < mv[vec[i]]) {  // slots past a vector's own m hold no vector of it
            const double c = cr[vec[i]][k0 + q], d = ci[vec[i]][k0 + q];
            ar[i] += c * u[q].v[i].x - d * u[q].v[i].y;
            ai[i] += c * u[q].v[i].y + d * u[q].v[i].x;
          }
    }
    Word o;
#pragma unroll
    for (int i = 0; i < VPL; ++i) o.v[i] = V{static_cast<R>(ar[i]), static_cast<R>(ai[i])};
    word_norm<VPL>(o, n2);
    out[w] = o;
    if (out2) reinterpret_cast<Word*>(out2)[w] = o;
  }
  word_norm_store<NV, VPL>(n2, red, partials);
  if (blockIdx.x == 0) record_step<NV>(st, ctl, log, obs_log, nobs, seq);
}

// |v|^2 partials of the step's input (first step of a call), tau for every
// vector, and a cleared control block.
template <typename R, int NV, int VPL>
__global__ __launch_bounds__(kBlock) void k_step_begin(int64_t words, const typename CT<R>::T* x, VecState* st,
                                                       StepCtl* ctl, double tau, int norm, double* partials) {
  using Word = StateWord<R, VPL>;
  __shared__ double red[kWaves * kMaxNV];
  if (ctl->abort) return;
  const int tid = threadIdx.x;
  if (norm) {
    double n2[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) n2[i] = 0.0;
    for (int64_t w = (int64_t)blockIdx.x * kBlock + tid; w < words; w += (int64_t)gridDim.x * kBlock)
      word_norm<VPL>(reinterpret_cast<const Word*>(x)[w], n2);
    word_norm_store<NV, VPL>(n2, red, partials);
  }
  if (blockIdx.x == 0 && tid < NV) st[tid].tau = tau;
  if (blockIdx.x == 0 && tid == 0) {
    ctl->all_done = 0;
    ctl->any_maxed = 0;
    ctl->iter = 0;
  }
}

// Records the observables of the last sample time (no log): a cleared
// control block and obs_log; nothing after an abandoned step.
template <int NV>
__global__ void k_step_log(const VecState* st, StepCtl* ctl, CombineLog* log, double* obs_log, int nobs) {
  if (ctl->abort) return;
  record_step<NV>(st, ctl, log, obs_log, nobs, 0);
}

// Column sums of a [nrows][ncols] partial array, one workgroup per column,
// fixed order.
__global__ __launch_bounds__(kBlock) void k_finalize(const double* partials, int nrows, int ncols, double* out) {
  __shared__ double red[kWaves];
  const double s = reduce_column(partials, nrows, ncols, blockIdx.x, red);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// Observables of an apply in kObsOnly mode: finalize its partials
// [nrows][kObsQ][NV] into st, the block kernels' up-hop parts [ncols][NV] with
// them (all columns in one pass: 4 vectors of 12 sites took 20 us one column
// after another).
template <int NV>
__global__ __launch_bounds__(kBlock) void k_finalize_obs(const double* partials, int nrows, const double* hops,
                                                         int ncols, VecState* st) {
  constexpr int NC = kObsQ * NV;
  __shared__ double red[kWaves * NC], so[NC], su[NV];
  const double rows = cols_partial<NC, kBlock>(partials, nrows, NC);
  const double cols = ncols > 0 ? cols_partial<NV, kBlock>(hops, ncols, NV) : 0.0;
  cols_total<NC, kWaves>(rows, red, so);
  cols_total<NV, kWaves>(cols, red, su);
  const int t = threadIdx.x, q = t / NV;
  if (t < NC) st[t % NV].obs[q] = so[t] + (q == kObsQ - 1 ? su[t % NV] : 0.0);
}

template <typename R>
__global__ void k_interleave(int64_t n, int nv, const typename CT<R>::T* src, typename CT<R>::T* dst,
                             int to_block) {
  const int64_t total = n * nv;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = i / nv, v = i % nv;  // block layout i = k*nv + v ; ABI layout v*n + k
    if (to_block) dst[i] = src[v * n + k];
    else dst[v * n + k] = src[i];
  }
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_site_docc(int dim_up, int dim_dn, int n_sites, const uint32_t* up,
                                                      const uint32_t* dn, const typename CT<R>::T* x,
                                                      double* partials) {
  __shared__ double red[kWaves * kMaxSites];
  double acc[kMaxSites];
#pragma unroll
  for (int i = 0; i < kMaxSites; ++i) acc[i] = 0.0;
  const int64_t n = (int64_t)dim_up * dim_dn;
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n; k += (int64_t)gridDim.x * kBlock) {
    const auto t = x[k];
    const double m2 = (double)t.x * t.x + (double)t.y * t.y;
    const uint32_t d = up[k / dim_dn] & dn[k % dim_dn];
#pragma unroll
    for (int i = 0; i < kMaxSites; ++i)
      if ((d >> i) & 1u) acc[i] += m2;
  }
  block_partials<1>(acc, n_sites, red, partials + (size_t)blockIdx.x * n_sites);
}

// y = sign * x at the mapped source element: a creation or annihilation
// operator between two sectors.  For an up operator the map acts on tile rows
// (map[a'] = source row, -1 = no source), for a down operator on columns.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_cop(int64_t n_t, int dim_dn_t, int dim_dn_s, int64_t n_s, int nvec,
                                                 int down, const int32_t* map, const int8_t* sgn,
                                                 const typename CT<R>::T* x, typename CT<R>::T* y) {
  using V = typename CT<R>::T;
  const int64_t total = n_t * nvec;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
    const int64_t k = i / n_t, e = i % n_t;
    const int a = static_cast<int>(e / dim_dn_t), b = static_cast<int>(e % dim_dn_t);
    const int r = down ? b : a;
    const int src = map[r];
    V out = V{0, 0};
    if (src >= 0) {
      const int64_t se = down ? (int64_t)a * dim_dn_s + src : (int64_t)src * dim_dn_s + b;
      const V v = x[k * n_s + se];
      const R f = static_cast<R>(sgn[r]);
      out = V{f * v.x, f * v.y};
    }
    y[i] = out;
  }
}

// <x_k | y_k> partials for nvec vector pairs (ABI layout), [grid][2 * nvec].
template <typename R>
__global__ __launch_bounds__(kBlock) void k_dots(int64_t n, int nvec, const typename CT<R>::T* x,
                                                  const typename CT<R>::T* y, double* partials) {
  __shared__ double red[kWaves];
  for (int k = 0; k < nvec; ++k) {
    double re = 0.0, im = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
      const auto a = x[k * n + i];
      const auto b = y[k * n + i];
      re += (double)a.x * b.x + (double)a.y * b.y;
      im += (double)a.x * b.y - (double)a.y * b.x;
    }
    re = block_sum(re, red);
    im = block_sum(im, red);
    if (threadIdx.x == 0) {
      partials[(size_t)blockIdx.x * 2 * nvec + 2 * k] = re;
      partials[(size_t)blockIdx.x * 2 * nvec + 2 * k + 1] = im;
    }
  }
}

// Overlaps of NV members with the state they were made from (Sec. 2.5,
// Eq. (Glg)): member v, in the target sector, with operator map map_v (tile
// rows for an up operator, columns for a down one; -1 = no source) and signs
// sgn_v, and psi_v the source-sector state at its time,
//   o_v = <c_v psi_v | phi_v> = sum_y sgn_v(y) conj(psi_v[src_v(y)]) phi_v[y],
// gathered straight from psi_v (no copy of c_v psi_v).  phi is interleaved
// ([y][NV]) or in the ABI layout ([v][n_t]).  Partials [NV][grid][2]; the
// kernel does nothing after an abandoned step (ctl->abort).
// A thread takes the VPL members of one 16-byte word of an interleaved
// element (one member otherwise), so that the record's gathers of a block
// spread over the chip; 8 members of 10 sites (complex64): 32 us with one
// thread per element on 52 workgroups and a reduction per sum, 10 us now.
template <typename R, int NV, int VPL>
__global__ __launch_bounds__(kBlock) void k_overlaps(OverlapArgs p) {
  using V = typename CT<R>::T;
  struct __align__(sizeof(V) * VPL) Word {
    V v[VPL];
  };
  constexpr int L = NV / VPL;  // words per element
  __shared__ double red[kWaves * 2 * NV];
  if (p.ctl && p.ctl->abort) return;
  const V* const psi = static_cast<const V*>(p.traj);
  const int tid = threadIdx.x, k = tid % L;
  double acc[2 * VPL];
#pragma unroll
  for (int q = 0; q < 2 * VPL; ++q) acc[q] = 0.0;
  int64_t off[VPL];
  const int32_t* map[VPL];
  const int8_t* sgn[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int v = k * VPL + i;
    off[i] = p.psi_off[v];
    map[i] = p.maps + static_cast<size_t>(v) * p.map_len;
    sgn[i] = p.sgns + static_cast<size_t>(v) * p.map_len;
  }
  const uint32_t ddt = static_cast<uint32_t>(p.dim_dn_t);
  for (int64_t w = (int64_t)blockIdx.x * kBlock + tid; w < p.n_t * L; w += (int64_t)gridDim.x * kBlock) {
    const int64_t y = w / L;
    const int a = static_cast<int>(static_cast<uint32_t>(y) / ddt), b = static_cast<int>(y - (int64_t)a * ddt);
    const int r = p.down ? b : a;
    Word f;
    if (VPL > 1 || p.interleaved) f = static_cast<const Word*>(p.phi)[w];
    else f.v[0] = static_cast<const V*>(p.phi)[k * p.n_t + y];
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int src = map[i][r];
      if (src < 0) continue;
      const int64_t se = p.down ? (int64_t)a * p.dim_dn_s + src : (int64_t)src * p.dim_dn_s + b;
      const V x = psi[off[i] + se];
      const double sg = static_cast<double>(sgn[i][r]);
      acc[2 * i] += sg * ((double)x.x * f.v[i].x + (double)x.y * f.v[i].y);
      acc[2 * i + 1] += sg * ((double)x.x * f.v[i].y - (double)x.y * f.v[i].x);
    }
  }
  // workgroup sums, fixed order; member v's pair goes to partials + (v grid + workgroup) 2
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int q = 0; q < 2 * VPL; ++q) {
    double t = acc[q];
#pragma unroll
    for (int o = 32; o >= L; o >>= 1) t += __shfl_xor(t, o);
    if (lane < L) red[wv * 2 * NV + lane * 2 * VPL + q] = t;
  }
  __syncthreads();
  if (tid < 2 * NV) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += red[w * 2 * NV + tid];
    p.partials[((size_t)(tid >> 1) * gridDim.x + blockIdx.x) * 2 + (tid & 1)] = t;
  }
}

// Deterministic test vector: x[i] = (sin(0.618 i), cos(0.377 i + 1)).
template <typename R>
__global__ __launch_bounds__(kBlock) void k_fill_probe(int64_t n, typename CT<R>::T* x) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
    x[i] = typename CT<R>::T{static_cast<R>(sin(0.618 * (double)i)), static_cast<R>(cos(0.377 * (double)i + 1.0))};
}

// out[s * out_stride + q] = sum over r < rows of part[s * set_stride + r * cols + q]
// for q < cols, one workgroup per set s (fixed order).
__global__ __launch_bounds__(kBlock) void k_reduce_sets(const double* part, int64_t set_stride, int rows, int cols,
                                                        double* out, int64_t out_stride) {
  __shared__ double red[kWaves];
  const double* P = part + (int64_t)blockIdx.x * set_stride;
  for (int q = 0; q < cols; ++q) {
    const double s = reduce_column(P, rows, cols, q, red);
    if (threadIdx.x == 0) out[(int64_t)blockIdx.x * out_stride + q] = s;
  }
}

// --------------------- CGS2 re-orthogonalisation ---------------------------
// One classical Gram-Schmidt pass of w = u_{j+1} against the Krylov vectors
// v_k = s_k u_k, k = 0..j (FP64 coefficients):  w <- w - sum_k v_k <v_k, w>.
// Three kernels: partial inner products, their fixed-order reduction into
// coefficients s_k^2 <u_k, w>, and the subtraction with |w|^2 partials.
// All exit at once after the step's decision.
constexpr int kReorthK = 4;  // inner products accumulated per pass over w

template <typename R, int NV>
__global__ __launch_bounds__(kBlock) void k_reorth_dot(int64_t n, void* const* slots, int j, const StepCtl* ctl,
                                                       double* partials) {
  using V = typename CT<R>::T;
  __shared__ double red[kWaves * 2 * kReorthK * kMaxNV];
  if (ctl->all_done) return;
  const V* w = static_cast<const V*>(slots[j + 1]);
  const int64_t total = n * NV;
  const int tid = threadIdx.x;
  for (int kb = 0; kb <= j; kb += kReorthK) {
    const int kn = min(kReorthK, j + 1 - kb);
    double acc[2 * kReorthK];
#pragma unroll
    for (int q = 0; q < 2 * kReorthK; ++q) acc[q] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + tid; i < total; i += (int64_t)gridDim.x * kBlock) {
      const V x = w[i];
#pragma unroll
      for (int q = 0; q < kReorthK; ++q) {
        if (q < kn) {
          const V u = static_cast<const V*>(slots[kb + q])[i];
          acc[2 * q] += (double)u.x * x.x + (double)u.y * x.y;      // conj(u) w
          acc[2 * q + 1] += (double)u.x * x.y - (double)u.y * x.x;
        }
      }
    }
    block_partials<NV>(acc, 2 * kn, red, partials + ((size_t)blockIdx.x * (j + 1) * 2 + 2 * kb) * NV);
  }
}

template <int NV>
__global__ __launch_bounds__(kBlock) void k_reorth_coef(const double* partials, int nrows, int j, const VecState* st,
                                                        const StepCtl* ctl, double* coef) {
  __shared__ double red[kWaves];
  if (ctl->all_done) return;
  const int ncols = (j + 1) * 2 * NV;  // column (k * 2 + c) * NV + v
  for (int t = 0; t < ncols; ++t) {
    const double s = reduce_column(partials, nrows, ncols, t, red);
    if (threadIdx.x == 0) {
      const int v = t % NV, c = (t / NV) % 2, k = t / (2 * NV);
      const double sc = st[v].scale[k];
      coef[(k * NV + v) * 2 + c] = s * sc * sc;
    }
  }
}

template <typename R, int NV>
__global__ __launch_bounds__(kBlock) void k_reorth_axpy(int64_t n, void* const* slots, int j, const double* coef,
                                                        const StepCtl* ctl, double* partials) {
  using V = typename CT<R>::T;
  __shared__ double red[kWaves * kMaxNV];
  __shared__ double cr[kMMax + 1][kMaxNV], ci[kMMax + 1][kMaxNV];
  if (ctl->all_done) return;
  const int tid = threadIdx.x;
  for (int t = tid; t < (j + 1) * NV; t += kBlock) {
    cr[t / NV][t % NV] = coef[2 * t];
    ci[t / NV][t % NV] = coef[2 * t + 1];
  }
  __syncthreads();
  V* w = static_cast<V*>(slots[j + 1]);
  const int v = tid % NV;
  const int64_t total = n * NV;
  double n2 = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + tid; i < total; i += (int64_t)gridDim.x * kBlock) {
    const V x = w[i];
    double ar = x.x, ai = x.y;
    for (int k = 0; k <= j; ++k) {
      const V u = static_cast<const V*>(slots[k])[i];
      ar -= cr[k][v] * u.x - ci[k][v] * u.y;
      ai -= cr[k][v] * u.y + ci[k][v] * u.x;
    }
    const V o = V{static_cast<R>(ar), static_cast<R>(ai)};
    w[i] = o;
    n2 += (double)o.x * o.x + (double)o.y * o.y;
  }
  block_partials<NV>(&n2, 1, red, partials + (size_t)blockIdx.x * NV);
}

// ------------------- broadened spectral functions ---------------------------
// A(nu) = (1/pi) Re sum_k w_k e^{-eps s_k} e^{i nu s_k} z_k on s_k = k dt with
// trapezoidal weights, z = conj(o) for removal (lesser) members and z = o for
// addition (greater) members; one thread per (member, frequency), FP64.
__global__ __launch_bounds__(kBlock) void k_spectral(int n_s, const double2* __restrict__ o,
                                                     unsigned long long lesser_mask, double dt, double eps,
                                                     int n_nu, const double* __restrict__ nu,
                                                     double* __restrict__ out) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  const int m = blockIdx.y;
  if (f >= n_nu) return;
  const double w = nu[f];
  const double cj = ((lesser_mask >> m) & 1ull) ? -1.0 : 1.0;
  const double2* om = o + (size_t)m * n_s;
  double acc = 0.0;
  for (int k = 0; k < n_s; ++k) {
    const double s = k * dt;
    const double wt = (k == 0 || k == n_s - 1) ? 0.5 * dt : dt;
    double sn, cs;
    sincos(w * s, &sn, &cs);
    const double2 z = om[k];
    acc += wt * exp(-eps * s) * (cs * z.x - sn * (cj * z.y));
  }
  out[(size_t)m * n_nu + f] = n_s > 1 ? acc / M_PI : 0.0;
}

}  // namespace dev
using namespace dev;

hipError_t launch_apply_c128(const ApplyLaunch& L, int grid, size_t lds, int* pgrid);
hipError_t launch_apply_c64(const ApplyLaunch& L, int grid, size_t lds, int* pgrid);
hipError_t launch_batch_c128(const ApplyLaunch& L, int nvec, int cw);
hipError_t launch_batch_c64(const ApplyLaunch& L, int nvec, int cw);
hipError_t launch_block_c128(const ApplyLaunch& L, int* pgrid);
hipError_t launch_block_c64(const ApplyLaunch& L, int* pgrid);

int elem_grid(int64_t n) {
  // four workgroups per CU at most (16 waves) for these memory-bound passes;
  // every Lanczos apply workgroup sums the partials they leave
  const int64_t g = (n + 4 * kBlock - 1) / (4 * kBlock);
  return static_cast<int>(g < 1 ? 1 : (g > 1024 ? 1024 : g));
}

int apply_chunks(const DevBasis& db, int prec, int nv) {
  // Several column chunks per row would keep more up-hop gathers in flight
  // (measured: at most ~15% faster for plain applies at 12 sites, and slower
  // inside the Lanczos loop, whose first phase sums the previous kernel's
  // partials in every workgroup) -- one chunk per row.  The fused Lanczos row
  // pass requires one chunk (it updates and sums whole rows); its launcher
  // refuses anything else.
  (void)db;
  (void)prec;
  (void)nv;
  return 1;
}

// Column block of the column pass: kColW columns, staged as +x and -x, or as
// +x alone (sign from the stage index) when two copies do not fit; 2 columns
// of one copy when 4 do not fit either.
static size_t colpass_copy_bytes(const DevBasis& db, int prec, int w) {
  return (static_cast<size_t>(db.dim_up) + 1) * w * (prec == 0 ? 16 : 8);
}
int colpass_width(const DevBasis& db, int prec) {
  return colpass_copy_bytes(db, prec, kColW) <= 150 * 1024 ? kColW : 2;
}
bool colpass_single(const DevBasis& db, int prec) {
  return 2 * colpass_copy_bytes(db, prec, colpass_width(db, prec)) > 150 * 1024;
}
int colpass_grid(const DevBasis& db, int prec) {
  const int w = colpass_width(db, prec);
  return (db.dim_dn + w - 1) / w;
}

size_t colpass_lds_bytes(const DevBasis& db, int prec) {
  const size_t copy = colpass_copy_bytes(db, prec, colpass_width(db, prec));
  return colpass_single(db, prec) ? copy : 2 * copy;
}

bool apply_global_rows(const DevBasis& db, int prec, int nv) {
  return nv == 1 && apply_lds_bytes(db, prec, 1, 1) > 150 * 1024;
}

// Larger than the eight XCDs' L2s together: one vector, changing buffers, one
// pass / gathered columns, in us: 47 MB (13 sites, complex128) 104 / 72, 94 MB
// (14 sites, complex64) 228 / 142, 188 MB (14 sites, complex128) 287 / 243, 331
// MB (15 sites, complex64) 894 / 590, 2.6 GB (16 sites, complex128) 5,033 /
// 4,423.  Staged columns: 24 MB (13 sites, complex64) as fast as gathered ones,
// 14 sites, complex64, 200 where those then took 140, 15 and 16 sites do not fit.
bool apply_gathers(const DevBasis& db, int prec) {
  if (apply_global_rows(db, prec, 1) && db.dn_gslots == 0) return false;  // no grouped table for the row pass
  return static_cast<double>(db.dim) * (prec == 0 ? 16 : 8) > 32.0 * 1024 * 1024;
}

bool apply_two_pass(const DevBasis& db, int prec, int nv, int mode, bool obs) {
  if (nv != 1 || !(mode == kPlain || mode == kLanczos) || db.two_pass == 0 || !db.up_tab) return false;
  if (obs && mode != kLanczos) return false;
  const bool gather = mode == kPlain && apply_gathers(db, prec);
  // rows too long for LDS have a row pass of their own only where the column
  // pass gathers (k_rowgather); their other kernels do it all in one pass
  if (!gather && (apply_global_rows(db, prec, 1) || colpass_lds_bytes(db, prec) > 150 * 1024)) return false;
  if (db.two_pass == 1) return true;
  const int tuned = mode == kPlain ? db.tuned_single[prec] : db.tuned_lanczos[prec];
  if (tuned >= 0) return tuned == 1;
  // automatic: when a vector is larger than one XCD's L2 the up-hop row
  // gathers of the one-pass kernel stream from the Infinity Cache.  With 2
  // staged columns only the Lanczos iterations gain (fused updates), not a
  // plain apply.
  if (mode == kPlain && !gather && colpass_width(db, prec) < kColW) return false;
  // Lanczos iterations, whose update the row pass then takes in, gain from 1
  // MiB on where the column pass has a workgroup for every fourth unit, 256
  // columns, and the row pass 64 rows: us per step, one pass / two, 10 sites
  // complex128 (1.0 MB) 111 / 112, 11 sites complex64 (1.7 MB) 142 / 134 and
  // complex128 (3.4 MB) 152 / 143, 12 sites 4 + 5 complex64 (3.1 MB) 192 / 149;
  // tall tiles, complex64, 3 steps: 3,432 x 91 (14 sites, 2.4 MB) 830 / 1,013,
  // 3,003 x 105 764 / 906, 1,716 x 286 (13 sites, 3.7 MB) 810 / 705; 16 x 4,368
  // (complex128, 1.1 MB), 8 vectors on concurrent lanes, 1,910 / 2,133.
  const bool spread = mode != kPlain && db.dim_dn >= 256 && db.dim_up >= 64;
  const double least = spread ? 1.0 : 4.0;
  return static_cast<double>(db.dim) * (prec == 0 ? 16 : 8) >= least * 1024 * 1024;
}

int apply_grid(const DevBasis& db, int prec, int nv) {
  return std::max({db.dim_up * apply_chunks(db, prec, nv), colpass_grid(db, prec), db.dim_dn});
}

static bool block_slots_ok(int g) { return g == 8 || g == 12 || g == 16 || g == 20 || g == 24; }

size_t block_lds_bytes(const DevBasis& db, int prec, int nv) {
  const size_t es = prec == 0 ? 16 : 8;
  return (static_cast<size_t>(std::max(db.dim_up, db.dim_dn)) + 1) * nv * es;
}

bool block_two_pass(const DevBasis& db, int prec, int nv) {
  if (!(nv == 2 || nv == 4 || nv == 8) || db.block_path == 0 || !db.dn_tabg || !db.up_tabg) return false;
  const int gi = nv == 2 ? 1 : (nv == 4 ? 2 : 3);
  if (db.block_path == -1 && db.tuned_block[prec][gi] == 0) return false;
  if (!block_slots_ok(db.dn_gslots) || !block_slots_ok(db.up_gslots)) return false;
  return block_lds_bytes(db, prec, nv) <= 150 * 1024;
}

int apply_nq_two_pass(bool obs) { return obs ? 2 : 1; }  // column pass: alpha [, up-hop obs part]

int apply_nq(int mode, bool obs, int nc) {
  const bool kL = mode == kLanczos;
  const bool kO = mode == kObsOnly || (kL && obs);
  (void)nc;
  return (kL ? 1 : 0) + (kO ? kObsQ : 0);
}

size_t apply_lds_bytes(const DevBasis& db, int prec, int nv, int rows) {
  (void)rows;
  const size_t elem = prec == 0 ? 16 : 8;
  return 2 * (static_cast<size_t>(db.dim_dn) + 1) * nv * elem;  // +x and -x copies with zero slots
}

bool apply_fits(const DevBasis& db, int prec, int nv) {
  return nv == 1 || apply_lds_bytes(db, prec, nv, 1) <= 150 * 1024;
}

hipError_t launch_apply(const ApplyLaunch& L, int* grid_out) {
  if (L.nv > 1 && block_two_pass(*L.db, L.prec, L.nv)) {
    int pgrid = 0;
    const hipError_t e = L.prec == 0 ? launch_block_c128(L, &pgrid) : launch_block_c64(L, &pgrid);
    if (grid_out) *grid_out = pgrid;
    return e;
  }
  const int grid = L.db->dim_up * apply_chunks(*L.db, L.prec, L.nv);
  int pgrid = grid;
  const size_t lds = apply_lds_bytes(*L.db, L.prec, L.nv, L.rows);
  const hipError_t e = L.prec == 0 ? launch_apply_c128(L, grid, lds, &pgrid) : launch_apply_c64(L, grid, lds, &pgrid);
  if (grid_out) *grid_out = pgrid;
  return e;
}

int batch_columns(const DevBasis& db, int prec, int nvec) {
  if (nvec < 2 || nvec > kMaxNV) return -1;
  // One pass up to 11 sites (8 complex64 / complex128 vectors, one vs two
  // passes: 10 sites 10.6 / 10.6 vs 13.2 / 13.6 us, 11 sites 23.4 / 29.0 vs
  // 21.5 / 31.9; 12 sites 99.7 / 145.6 vs 68.8 / 124.0: a vector no longer
  // fits an XCD's L2 and its up hops miss).
  constexpr size_t kLds = 150 * 1024;
  if (db.dim <= (1 << 18) && db.maxs_pad <= 24 && apply_lds_bytes(db, prec, 1, 1) <= kLds) return 0;
  auto slots_ok = [](int g) { return g >= 4 && g <= 24; };
  if (!slots_ok(db.dn_gslots) || !slots_ok(db.up_gslots) || (static_cast<size_t>(db.dim_dn) + 1) * 16 > kLds) return -1;
  const size_t col = (static_cast<size_t>(db.dim_up) + 1) * 16;
  const int groups = prec == 0 ? nvec : (nvec + 1) / 2;
  // 8 columns per workgroup, one workgroup per compute unit, where that makes
  // nearly whole rounds of them (of 256: 12 sites, 8 complex64 vectors, 464
  // workgroups: 82.6 us vs 90.9 with 4 columns; 3 complex128 vectors, 348:
  // 60.7 vs 54.5), else 4, or 2 where 4 do not fit (14 sites)
  const int w8 = groups * ((db.dim_dn + 7) / 8), rounds = (w8 + db.n_cu - 1) / db.n_cu;
  if (8 * col <= kLds && 20 * w8 >= 17 * db.n_cu * rounds) return 8;
  return 4 * col <= kLds ? 4 : (2 * col <= kLds ? 2 : -1);
}

hipError_t launch_batch(const ApplyLaunch& L, int columns) {
  if (L.nv < 1 || L.nv > kMaxNV) return hipErrorInvalidValue;
  return L.prec == 0 ? launch_batch_c128(L, L.nv, columns) : launch_batch_c64(L, L.nv, columns);
}

#define HUB_NV_SWITCH(nv, CALL)                         \
  switch (nv) {                                         \
    case 1: { constexpr int NVC = 1; CALL; } break;     \
    case 2: { constexpr int NVC = 2; CALL; } break;     \
    case 4: { constexpr int NVC = 4; CALL; } break;     \
    case 8: { constexpr int NVC = 8; CALL; } break;     \
    default: return hipErrorInvalidValue;               \
  }

hipError_t launch_reorth(int prec, int nv, int64_t n, void* const* slots_dev, int j, const VecState* st,
                         const StepCtl* ctl, double* dot_partials, double* coef, double* norm_partials,
                         hipStream_t s) {
  const int grid = elem_grid(n * nv);
  if (prec == 0) {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_reorth_dot<double, NVC>), dim3(grid), dim3(kBlock), 0, s, n, slots_dev,
                                         j, ctl, dot_partials));
  } else {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_reorth_dot<float, NVC>), dim3(grid), dim3(kBlock), 0, s, n, slots_dev,
                                         j, ctl, dot_partials));
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_reorth_coef<NVC>), dim3(1), dim3(kBlock), 0, s, dot_partials, grid, j, st,
                                       ctl, coef));
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (prec == 0) {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_reorth_axpy<double, NVC>), dim3(grid), dim3(kBlock), 0, s, n,
                                         slots_dev, j, coef, ctl, norm_partials));
  } else {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_reorth_axpy<float, NVC>), dim3(grid), dim3(kBlock), 0, s, n,
                                         slots_dev, j, coef, ctl, norm_partials));
  }
  return hipGetLastError();
}

hipError_t launch_spectral(int n_members, int n_s, const void* overlaps, const int32_t* lesser, double dt, double eps,
                           int n_nu, const double* nu, double* out, hipStream_t s) {
  for (int m0 = 0; m0 < n_members; m0 += 64) {
    const int mc = std::min(64, n_members - m0);
    unsigned long long mask = 0;
    for (int k = 0; k < mc; ++k)
      if (lesser[m0 + k]) mask |= 1ull << k;
    const dim3 grid((n_nu + kBlock - 1) / kBlock, mc);
    hipLaunchKernelGGL(k_spectral, grid, dim3(kBlock), 0, s, n_s,
                       static_cast<const double2*>(overlaps) + static_cast<size_t>(m0) * n_s, mask, dt, eps, n_nu,
                       nu, out + static_cast<size_t>(m0) * n_nu);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_update(int prec, int nv, int64_t n, void* w, const void* uj, VecState* st, StepCtl* ctl, int j,
                         const double* apply_partials, int apply_nblk, int apply_nq, const double* row_obs,
                         int row_nblk, double* partials, hipStream_t s) {
  const int grid = elem_grid(n * nv);
  if (prec == 0) {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_update<double, NVC>), dim3(grid), dim3(kBlock), 0, s, n,
                                         static_cast<double2*>(w), static_cast<const double2*>(uj), st, ctl, j,
                                         apply_partials, apply_nblk, apply_nq, row_obs, row_nblk, partials));
  } else {
    HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_update<float, NVC>), dim3(grid), dim3(kBlock), 0, s, n,
                                         static_cast<float2*>(w), static_cast<const float2*>(uj), st, ctl, j,
                                         apply_partials, apply_nblk, apply_nq, row_obs, row_nblk, partials));
  }
  return hipGetLastError();
}

// 16-byte words where every vector's storage is made of whole ones (an odd
// number of complex64 values, or a caller's vector at an odd one, is not).
template <typename R, int NV>
static bool whole_words(int64_t n, const void* state, const void* a = nullptr, const void* b = nullptr) {
  constexpr int VPL = 16 / sizeof(typename CT<R>::T);
  auto odd = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 != 0; };
  return (n * NV) % VPL == 0 && !odd(state) && !odd(a) && !odd(b);
}

template <typename R, int NV>
static hipError_t combine_t(int64_t n, void* state, void* slots, const VecState* st, StepCtl* ctl, double* partials,
                            int seq, CombineLog* log, double* obs_log, int nobs, hipStream_t s, void* copy_to) {
  using V = typename CT<R>::T;
  constexpr int VPL = 16 / sizeof(V);
  const int grid = elem_grid(n * NV);
  V* const x = static_cast<V*>(state);
  const V* const sl = static_cast<const V*>(slots);
  if (whole_words<R, NV>(n, state, slots, copy_to))
    hipLaunchKernelGGL((k_combine<R, NV, VPL>), dim3(grid), dim3(kBlock), 0, s, n * NV / VPL, x, sl, n * NV / VPL, st,
                       ctl, partials, seq, log, obs_log, nobs, static_cast<V*>(copy_to));
  else
    hipLaunchKernelGGL((k_combine<R, NV, 1>), dim3(grid), dim3(kBlock), 0, s, n * NV, x, sl, n * NV, st, ctl, partials,
                       seq, log, obs_log, nobs, static_cast<V*>(copy_to));
  return hipGetLastError();
}

template <typename R, int NV>
static void step_begin_t(int64_t n, const void* v, VecState* st, StepCtl* ctl, double tau, bool norm, double* partials,
                         hipStream_t s) {
  using V = typename CT<R>::T;
  constexpr int VPL = 16 / sizeof(V);
  const int grid = elem_grid(n * NV);
  const V* const x = static_cast<const V*>(v);
  if (whole_words<R, NV>(n, v))
    hipLaunchKernelGGL((k_step_begin<R, NV, VPL>), dim3(grid), dim3(kBlock), 0, s, n * NV / VPL, x, st, ctl, tau,
                       norm ? 1 : 0, partials);
  else
    hipLaunchKernelGGL((k_step_begin<R, NV, 1>), dim3(grid), dim3(kBlock), 0, s, n * NV, x, st, ctl, tau, norm ? 1 : 0,
                       partials);
}

hipError_t launch_combine(int prec, int nv, int64_t n, void* state, void* slots, const VecState* st, StepCtl* ctl,
                          double* partials, int seq, CombineLog* log, double* obs_log, int nobs, hipStream_t s,
                          void* copy_to) {
  if (prec == 0) {
    HUB_NV_SWITCH(nv, return (combine_t<double, NVC>(n, state, slots, st, ctl, partials, seq, log, obs_log, nobs, s,
                                                     copy_to)));
  } else {
    HUB_NV_SWITCH(nv, return (combine_t<float, NVC>(n, state, slots, st, ctl, partials, seq, log, obs_log, nobs, s,
                                                    copy_to)));
  }
}

template <typename R, int NV>
static void overlaps_t(const OverlapArgs& a, hipStream_t s) {
  constexpr int VPL = 16 / sizeof(typename CT<R>::T);
  const int grid = overlap_grid(a.n_t);
  if constexpr (VPL > 1 && NV % VPL == 0)  // a block's words are whole and aligned (its buffer is the library's)
    if (a.interleaved) {
      hipLaunchKernelGGL((k_overlaps<R, NV, VPL>), dim3(grid), dim3(kBlock), 0, s, a);
      return;
    }
  hipLaunchKernelGGL((k_overlaps<R, NV, 1>), dim3(grid), dim3(kBlock), 0, s, a);
}

hipError_t launch_overlaps(int prec, int nv, const OverlapArgs& a, hipStream_t s) {
  if (a.n_t > INT32_MAX) return hipErrorInvalidValue;  // tile positions are 32-bit (16 sites: 1.7e8)
  if (prec == 0) {
    HUB_NV_SWITCH(nv, (overlaps_t<double, NVC>(a, s)));
  } else {
    HUB_NV_SWITCH(nv, (overlaps_t<float, NVC>(a, s)));
  }
  return hipGetLastError();
}

hipError_t launch_reduce_sets(const double* part, int64_t set_stride, int n_sets, int rows, int cols, double* out,
                              int64_t out_stride, hipStream_t s) {
  if (n_sets < 1) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_sets, dim3(n_sets), dim3(kBlock), 0, s, part, set_stride, rows, cols, out, out_stride);
  return hipGetLastError();
}

hipError_t launch_fill_probe(int prec, int64_t n, void* x, hipStream_t s) {
  const int grid = elem_grid(n);
  if (prec == 0) hipLaunchKernelGGL(k_fill_probe<double>, dim3(grid), dim3(kBlock), 0, s, n, static_cast<double2*>(x));
  else hipLaunchKernelGGL(k_fill_probe<float>, dim3(grid), dim3(kBlock), 0, s, n, static_cast<float2*>(x));
  return hipGetLastError();
}

int overlap_grid(int64_t n_t) {
  const int64_t g = (n_t + kBlock - 1) / kBlock;
  return static_cast<int>(g < 1 ? 1 : (g > 1024 ? 1024 : g));
}

hipError_t launch_step_log(int nv, const VecState* st, StepCtl* ctl, void* log, double* obs_log, int nobs,
                           hipStream_t s) {
  HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_step_log<NVC>), dim3(1), dim3(64), 0, s, st, ctl,
                                       static_cast<CombineLog*>(log), obs_log, nobs));
  return hipGetLastError();
}

hipError_t launch_step_begin(int prec, int nv, int64_t n, const void* v, VecState* st, StepCtl* ctl, double tau,
                             bool norm, double* partials, hipStream_t s) {
  if (prec == 0) {
    HUB_NV_SWITCH(nv, (step_begin_t<double, NVC>(n, v, st, ctl, tau, norm, partials, s)));
  } else {
    HUB_NV_SWITCH(nv, (step_begin_t<float, NVC>(n, v, st, ctl, tau, norm, partials, s)));
  }
  return hipGetLastError();
}

hipError_t launch_finalize_obs(int nv, const double* partials, int nrows, const double* hops, int ncols, VecState* st,
                               hipStream_t s) {
  HUB_NV_SWITCH(nv, hipLaunchKernelGGL((k_finalize_obs<NVC>), dim3(1), dim3(kBlock), 0, s, partials, nrows, hops,
                                       ncols, st));
  return hipGetLastError();
}

hipError_t launch_finalize(const double* partials, int nrows, int ncols, double* out, hipStream_t s) {
  if (ncols < 1) return hipSuccess;
  hipLaunchKernelGGL(k_finalize, dim3(ncols), dim3(kBlock), 0, s, partials, nrows, ncols, out);
  return hipGetLastError();
}

hipError_t launch_interleave(int prec, int nv, int64_t n, const void* src, void* dst, bool to_block,
                             hipStream_t s) {
  const int grid = elem_grid(n * nv);
  if (prec == 0)
    hipLaunchKernelGGL(k_interleave<double>, dim3(grid), dim3(kBlock), 0, s, n, nv,
                       static_cast<const double2*>(src), static_cast<double2*>(dst), to_block ? 1 : 0);
  else
    hipLaunchKernelGGL(k_interleave<float>, dim3(grid), dim3(kBlock), 0, s, n, nv,
                       static_cast<const float2*>(src), static_cast<float2*>(dst), to_block ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_site_docc(int prec, const DevBasis& db, const void* x, double* out, double* partials,
                            hipStream_t s) {
  const int grid = elem_grid(db.dim);
  if (prec == 0)
    hipLaunchKernelGGL(k_site_docc<double>, dim3(grid), dim3(kBlock), 0, s, db.dim_up, db.dim_dn, db.n_sites,
                       db.up_bits, db.dn_bits, static_cast<const double2*>(x), partials);
  else
    hipLaunchKernelGGL(k_site_docc<float>, dim3(grid), dim3(kBlock), 0, s, db.dim_up, db.dim_dn, db.n_sites,
                       db.up_bits, db.dn_bits, static_cast<const float2*>(x), partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_finalize(partials, grid, db.n_sites, out, s);
}

hipError_t launch_cop(int prec, int64_t n_t, int dim_dn_t, int dim_dn_s, int64_t n_s, int nvec, bool down,
                      const int32_t* map, const int8_t* sgn, const void* x, void* y, hipStream_t s) {
  const int grid = elem_grid(n_t * nvec) * 4;
  if (prec == 0)
    hipLaunchKernelGGL(k_cop<double>, dim3(grid), dim3(kBlock), 0, s, n_t, dim_dn_t, dim_dn_s, n_s, nvec,
                       down ? 1 : 0, map, sgn, static_cast<const double2*>(x), static_cast<double2*>(y));
  else
    hipLaunchKernelGGL(k_cop<float>, dim3(grid), dim3(kBlock), 0, s, n_t, dim_dn_t, dim_dn_s, n_s, nvec,
                       down ? 1 : 0, map, sgn, static_cast<const float2*>(x), static_cast<float2*>(y));
  return hipGetLastError();
}

hipError_t launch_dots(int prec, int64_t n, int nvec, const void* x, const void* y, double* out, double* partials,
                       hipStream_t s) {
  const int grid = elem_grid(n);
  if (prec == 0)
    hipLaunchKernelGGL(k_dots<double>, dim3(grid), dim3(kBlock), 0, s, n, nvec, static_cast<const double2*>(x),
                       static_cast<const double2*>(y), partials);
  else
    hipLaunchKernelGGL(k_dots<float>, dim3(grid), dim3(kBlock), 0, s, n, nvec, static_cast<const float2*>(x),
                       static_cast<const float2*>(y), partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_finalize(partials, grid, 2 * nvec, out, s);
}

}  // namespace hub
