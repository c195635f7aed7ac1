// Plain products of several vectors in the caller's layout (hub_apply_H with
// nvec > 1), templated; instantiated per precision by batch_c128.hip and
// batch_c64.hip.
#pragma once

#include <hip/hip_ext.h>

#include "block_impl.h"
#include "kernels_common.h"

namespace hub {
namespace dev {

// y_v = H(A_v) x_v with the vectors one after another, as the caller holds
// them: no interleaved copies are made (two passes over 110 MB took 50 of 126
// us for eight complex64 vectors of 12 sites).
//   One pass (k_apply_batch), small tiles: a workgroup per (vector, tile row),
//     the row staged as +x and -x, up hops as whole rows from the caches;
//     launch-bound (8 vectors of 10 sites: 31 us in interleaved blocks, 11 us).
//   Two passes, larger tiles: a row pass (k_batch_row: diagonal and down hops)
//     and a column pass (k_batch_col: up hops) over VPL vectors at a time, two
//     complex64 or one complex128, interleaved in LDS only, so that a hop is
//     one 16-byte read and its table entry is decoded once for both.  Eight
//     complex64 vectors of 12 sites 126 -> 83 us (1.3 TB/s of x and y; the
//     row pass keeps the VALU busy 59 % and the LDS 55 % of its 40 us, three
//     fifths of that bank conflicts of the random 16-byte gathers, the column
//     pass 51 % and 34 % of 43 us), eight
//     complex128 ones 209 -> 139 us; 14 sites 2,045 -> 1,689 and 3,770 ->
//     2,265 us.  More words per element in the row pass (2 or 4, as the block
//     kernels) conflict less but leave too few wavefronts: 100-112 us.
template <typename R>
struct BatchArgs {
  int dim_up, dim_dn, nvec;
  double U;
  const uint32_t* up_bits;
  const uint32_t* dn_bits;
  const double* eps_up;
  const double* eps_dn;
  const int32_t* up_ptr;     // one pass: up hops of every row
  const uint32_t* up_hops;
  const uint16_t* tab;       // one pass: padded down table; two passes: the pass's grouped table
  uint8_t slot_class[64];    // class of every slot (one pass) or group; kMaxClasses: none
  R coef[2 * kMaxNV * (kMaxClasses + 1)];  // [v][class] complex, class kMaxClasses zero
  const void* x;
  void* y;
};

// v with the sign bit of e flipped in (e the same on every lane: scalar code).
__device__ __forceinline__ float flip(float v, uint32_t e) {
  return __uint_as_float(__float_as_uint(v) ^ (e & 0x80000000u));
}
__device__ __forceinline__ double flip(double v, uint32_t e) {
  return __hiloint2double(__double2hiint(v) ^ static_cast<int>(e & 0x80000000u), __double2loint(v));
}

constexpr int kBatchBlock = 256;

template <typename R, int MAXS>
__global__ __launch_bounds__(kBatchBlock) void k_apply_batch(BatchArgs<R> p) {
  using V = typename CT<R>::T;
  constexpr int kQ2 = MAXS / 4, kUB = 8;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  V* xs = reinterpret_cast<V*>(smem_raw);
  const uint32_t dd = p.dim_dn;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int v = lb / p.dim_up, a = lb % p.dim_up;
  const V* __restrict__ x = static_cast<const V*>(p.x) + static_cast<size_t>(v) * p.dim_up * dd;
  V* __restrict__ y = static_cast<V*>(p.y) + static_cast<size_t>(lb) * dd;
  const int hb = p.up_ptr[a], hcnt = p.up_ptr[a + 1] - hb;
  const uint32_t ua = p.up_bits[a];
  const double ea = p.eps_up ? p.eps_up[a] : 0.0;
  const uint2* tab2 = reinterpret_cast<const uint2*>(p.tab);
  const R* cv = p.coef + 2 * v * (kMaxClasses + 1);
  V cf[MAXS];
#pragma unroll
  for (int s = 0; s < MAXS; ++s) cf[s] = V{cv[2 * p.slot_class[s]], cv[2 * p.slot_class[s] + 1]};
  uint2 ev[kQ2];
  V tu[kUB];
  uint32_t q = threadIdx.x;
  auto up_row = [&](uint32_t e) { return x + static_cast<size_t>(e & 0xFFFFu) * dd; };
  auto up_coef = [&](uint32_t e) {
    const R* c = cv + 2 * ((e >> 16) & 0xFFu);
    return V{flip(c[0], e), flip(c[1], e)};
  };
  auto load_column = [&](uint32_t qq) {
#pragma unroll
    for (int k = 0; k < kQ2; ++k) ev[k] = tab2[qq * kQ2 + k];
#pragma unroll
    for (int k = 0; k < kUB; ++k) tu[k] = k < hcnt ? up_row(p.up_hops[hb + k])[qq] : V{0, 0};
  };
  if (q < dd) load_column(q);
  const V* xr = x + static_cast<size_t>(a) * dd;
  for (uint32_t t = threadIdx.x; t <= dd; t += kBatchBlock) {
    const V val = t < dd ? xr[t] : V{0, 0};
    xs[t] = val;
    xs[dd + 1 + t] = V{-val.x, -val.y};
  }
  __syncthreads();
  while (q < dd) {
    const double nd = static_cast<double>(__popc(ua & p.dn_bits[q]));
    const double dg = p.U * nd + ea + (p.eps_dn ? p.eps_dn[q] : 0.0);
    const V xv = xs[q];
    V acc = V{static_cast<R>(dg) * xv.x, static_cast<R>(dg) * xv.y};
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
      const uint32_t w2 = (s & 3) < 2 ? ev[s >> 2].x : ev[s >> 2].y;
      acc = cfma(cf[s], xs[(s & 1) ? (w2 >> 16) : (w2 & 0xFFFFu)], acc);
    }
#pragma unroll
    for (int k = 0; k < kUB; ++k)
      if (k < hcnt) acc = cfma(up_coef(p.up_hops[hb + k]), tu[k], acc);
    for (int h0 = kUB; h0 < hcnt; h0 += 8) {
      V t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] = h0 + k < hcnt ? up_row(p.up_hops[hb + h0 + k])[q] : V{0, 0};
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (h0 + k < hcnt) acc = cfma(up_coef(p.up_hops[hb + h0 + k]), t[k], acc);
    }
    y[q] = acc;
    q += kBatchBlock;
    if (q < dd) load_column(q);
  }
}

// The VPL vectors from v0 on of one workgroup: the i-th one's offset in the
// batch (the last vector again where the batch ends before: not stored) and
// its coefficients per group of slots.
template <typename R, int kG, int VPL>
__device__ __forceinline__ void batch_coefs(const BatchArgs<R>& p, int v0, typename CT<R>::T (&cf)[kG][VPL]) {
  using V = typename CT<R>::T;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const R* c = p.coef + 2 * min(v0 + i, p.nvec - 1) * (kMaxClasses + 1);
#pragma unroll
    for (int g = 0; g < kG; ++g) cf[g][i] = V{c[2 * p.slot_class[g]], c[2 * p.slot_class[g] + 1]};
  }
}

template <typename R, int MAXS, int BLK>
__global__ __launch_bounds__(BLK) void k_batch_row(BatchArgs<R> p) {
  using V = typename CT<R>::T;
  constexpr int VPL = 16 / sizeof(V), kG = MAXS / 4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  uint4* xs = reinterpret_cast<uint4*>(smem_raw);
  const uint32_t dd = p.dim_dn;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int v0 = lb / p.dim_up * VPL, a = lb % p.dim_up;
  const V* xr[VPL];
  V* yr[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const size_t o = (static_cast<size_t>(min(v0 + i, p.nvec - 1)) * p.dim_up + a) * dd;
    xr[i] = static_cast<const V*>(p.x) + o;
    yr[i] = static_cast<V*>(p.y) + o;
  }
  V cf[kG][VPL];
  batch_coefs<R, kG, VPL>(p, v0, cf);
  const uint2* tab2 = reinterpret_cast<const uint2*>(p.tab);
  uint2 ev[kG];
  uint32_t db = 0;
  auto fetch = [&](uint32_t b) {
#pragma unroll
    for (int g = 0; g < kG; ++g) ev[g] = tab2[b * kG + g];
    db = p.dn_bits[b];
  };
  if (threadIdx.x < dd) fetch(threadIdx.x);
#pragma unroll 4
  for (uint32_t t = threadIdx.x; t < dd; t += BLK) {
    V w[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) w[i] = xr[i][t];
    xs[t] = to_word<V>(w);
  }
  if (threadIdx.x == 0) xs[dd] = make_uint4(0u, 0u, 0u, 0u);
  const uint32_t ua = p.up_bits[a];
  const double ea = p.eps_up ? p.eps_up[a] : 0.0;
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < dd; b += BLK) {
    const double dg = p.U * static_cast<double>(__popc(ua & db)) + ea + (p.eps_dn ? p.eps_dn[b] : 0.0);
    uint2 ec[kG];
#pragma unroll
    for (int g = 0; g < kG; ++g) ec[g] = ev[g];
    if (b + BLK < dd) fetch(b + BLK);
    V acc[VPL];
    from_word<V>(xs[b], acc);
#pragma unroll
    for (int i = 0; i < VPL; ++i) acc[i] = V{static_cast<R>(dg) * acc[i].x, static_cast<R>(dg) * acc[i].y};
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      V sum[VPL];
      group_sum<R, 1>(ec[g], xs, 0, sum);
#pragma unroll
      for (int i = 0; i < VPL; ++i) acc[i] = cfma(cf[g][i], sum[i], acc[i]);
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (v0 + i < p.nvec) yr[i][b] = acc[i];
  }
}

// CW tile columns of VPL vectors per workgroup.
template <typename R, int MAXS, int BLK, int CW>
__global__ __launch_bounds__(BLK) void k_batch_col(BatchArgs<R> p) {
  using V = typename CT<R>::T;
  constexpr int VPL = 16 / sizeof(V), kG = MAXS / 4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  uint4* xs = reinterpret_cast<uint4*>(smem_raw);
  const uint32_t dd = p.dim_dn, du = p.dim_up;
  const int nb = (p.dim_dn + CW - 1) / CW;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int v0 = lb / nb * VPL;
  const uint32_t c = threadIdx.x % CW, b = lb % nb * CW + c;  // this thread's column
  const bool in = b < dd;
  const V* xc[VPL];
  V* yc[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const size_t o = static_cast<size_t>(min(v0 + i, p.nvec - 1)) * du * dd + (in ? b : 0);
    xc[i] = static_cast<const V*>(p.x) + o;
    yc[i] = static_cast<V*>(p.y) + o;
  }
  V cf[kG][VPL];
  batch_coefs<R, kG, VPL>(p, v0, cf);
  const uint2* tab2 = reinterpret_cast<const uint2*>(p.tab);
  uint2 ev[kG];
  V z[VPL];
  auto fetch = [&](uint32_t a) {
#pragma unroll
    for (int g = 0; g < kG; ++g) ev[g] = tab2[a * kG + g];
#pragma unroll
    for (int i = 0; i < VPL; ++i) z[i] = yc[i][static_cast<size_t>(a) * dd];
  };
  const uint32_t a0 = threadIdx.x / CW, astep = BLK / CW;
#pragma unroll 4
  for (uint32_t a = a0; a < du; a += astep) {
    V w[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) w[i] = xc[i][static_cast<size_t>(a) * dd];
    xs[a * CW + c] = to_word<V>(w);
  }
  if (threadIdx.x < CW) xs[du * CW + c] = make_uint4(0u, 0u, 0u, 0u);
  if (a0 < du) fetch(a0);
  __syncthreads();
  for (uint32_t a = a0; a < du; a += astep) {
    uint2 ec[kG];
#pragma unroll
    for (int g = 0; g < kG; ++g) ec[g] = ev[g];
    V acc[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) acc[i] = z[i];
    if (a + astep < du) fetch(a + astep);
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      V sum[VPL];
      group_sum<R, CW>(ec[g], xs, c, sum);
#pragma unroll
      for (int i = 0; i < VPL; ++i) acc[i] = cfma(cf[g][i], sum[i], acc[i]);
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (in && v0 + i < p.nvec) yc[i][static_cast<size_t>(a) * dd] = acc[i];
  }
}

// ---------------------------------------------------------------------------
// Launchers.

template <typename R>
BatchArgs<R> batch_args(const ApplyLaunch& L, int nvec) {
  const DevBasis& db = *L.db;
  BatchArgs<R> p{};
  p.dim_up = db.dim_up;
  p.dim_dn = db.dim_dn;
  p.nvec = nvec;
  p.U = db.U;
  p.up_bits = db.up_bits;
  p.dn_bits = db.dn_bits;
  p.eps_up = db.eps_up;
  p.eps_dn = db.eps_dn;
  p.up_ptr = db.up_ptr;
  p.up_hops = db.up_hops;
  for (int v = 0; v < nvec; ++v)
    for (int c = 0; c < 2 * db.nc; ++c)
      p.coef[2 * v * (kMaxClasses + 1) + c] = static_cast<R>(L.coef[2 * v * db.nc + c]);
  p.x = L.x;
  p.y = L.y;
  return p;
}

template <typename R, int MAXS>
hipError_t batch_one_t(const ApplyLaunch& L, int nvec) {
  const DevBasis& db = *L.db;
  BatchArgs<R> p = batch_args<R>(L, nvec);
  p.tab = db.dn_tab;
  for (int s = 0; s < 64; ++s) p.slot_class[s] = s < db.nslots ? db.slot_class[s] : kMaxClasses;
  auto fn = k_apply_batch<R, MAXS>;
  static const int max_dyn = dyn_lds_opt_in(reinterpret_cast<const void*>(fn));
  const size_t lds = apply_lds_bytes(db, sizeof(R) == 8 ? 0 : 1, 1, 1);
  if (lds > static_cast<size_t>(max_dyn)) return hipErrorInvalidValue;
  return launch_ev(fn, nvec * db.dim_up, kBatchBlock, lds, L.stream, L.ev_start, L.ev_stop, p);
}

template <typename R>
hipError_t batch_one(const ApplyLaunch& L, int nvec) {
  switch (L.db->maxs_pad) {
    case 4: return batch_one_t<R, 4>(L, nvec);
    case 8: return batch_one_t<R, 8>(L, nvec);
    case 12: return batch_one_t<R, 12>(L, nvec);
    case 16: return batch_one_t<R, 16>(L, nvec);
    case 20: return batch_one_t<R, 20>(L, nvec);
    case 24: return batch_one_t<R, 24>(L, nvec);
    default: return hipErrorInvalidValue;
  }
}

// Threads of the two passes' workgroups (12 sites, 8 complex64 vectors: row
// pass with 128, 256, 512 threads 87, 88, 90 us in all; column pass with 8
// columns, 512 and 1,024 threads 91 and 83 us).
constexpr int kBatchRowBlk = 256, kBatchColBlk = 1024;

template <typename R, int MAXS>
hipError_t batch_row_t(const ApplyLaunch& L, int nvec) {
  const DevBasis& db = *L.db;
  constexpr int VPL = 16 / sizeof(typename CT<R>::T);
  BatchArgs<R> p = batch_args<R>(L, nvec);
  p.tab = db.dn_tabg;
  for (int g = 0; g < 8; ++g) p.slot_class[g] = db.dn_gclass[g];
  auto fn = k_batch_row<R, MAXS, kBatchRowBlk>;
  static const int max_dyn = dyn_lds_opt_in(reinterpret_cast<const void*>(fn));
  const size_t lds = (static_cast<size_t>(db.dim_dn) + 1) * 16;
  if (lds > static_cast<size_t>(max_dyn)) return hipErrorInvalidValue;
  return launch_ev(fn, (nvec + VPL - 1) / VPL * db.dim_up, kBatchRowBlk, lds, L.stream, L.ev_start, L.ev_stop, p);
}

template <typename R, int MAXS, int CW>
hipError_t batch_col_t(const ApplyLaunch& L, int nvec) {
  const DevBasis& db = *L.db;
  constexpr int VPL = 16 / sizeof(typename CT<R>::T);
  BatchArgs<R> p = batch_args<R>(L, nvec);
  p.tab = db.up_tabg;
  for (int g = 0; g < 8; ++g) p.slot_class[g] = db.up_gclass[g];
  auto fn = k_batch_col<R, MAXS, kBatchColBlk, CW>;
  static const int max_dyn = dyn_lds_opt_in(reinterpret_cast<const void*>(fn));
  const size_t lds = (static_cast<size_t>(db.dim_up) + 1) * CW * 16;
  if (lds > static_cast<size_t>(max_dyn)) return hipErrorInvalidValue;
  return launch_ev(fn, (nvec + VPL - 1) / VPL * ((db.dim_dn + CW - 1) / CW), kBatchColBlk, lds, L.stream, L.ev2_start,
                   L.ev2_stop, p);
}

template <typename R, int CW>
hipError_t batch_col(const ApplyLaunch& L, int nvec) {
  switch (L.db->up_gslots) {
    case 4: return batch_col_t<R, 4, CW>(L, nvec);
    case 8: return batch_col_t<R, 8, CW>(L, nvec);
    case 12: return batch_col_t<R, 12, CW>(L, nvec);
    case 16: return batch_col_t<R, 16, CW>(L, nvec);
    case 20: return batch_col_t<R, 20, CW>(L, nvec);
    case 24: return batch_col_t<R, 24, CW>(L, nvec);
    default: return hipErrorInvalidValue;
  }
}

template <typename R>
hipError_t batch_two(const ApplyLaunch& L, int nvec, int cw) {
  hipError_t e = hipErrorInvalidValue;
  switch (L.db->dn_gslots) {
    case 4: e = batch_row_t<R, 4>(L, nvec); break;
    case 8: e = batch_row_t<R, 8>(L, nvec); break;
    case 12: e = batch_row_t<R, 12>(L, nvec); break;
    case 16: e = batch_row_t<R, 16>(L, nvec); break;
    case 20: e = batch_row_t<R, 20>(L, nvec); break;
    case 24: e = batch_row_t<R, 24>(L, nvec); break;
    default: break;
  }
  if (e != hipSuccess) return e;
  return cw == 8 ? batch_col<R, 8>(L, nvec) : (cw == 4 ? batch_col<R, 4>(L, nvec) : batch_col<R, 2>(L, nvec));
}

}  // namespace dev
}  // namespace hub
