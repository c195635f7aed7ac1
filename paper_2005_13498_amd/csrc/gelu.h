// GELU and its derivative in FP32 for the controller's training kernel:
// h = z Phi(z), d = Phi(z) + z phi(z).  No HIP of its own: the reciprocal and
// the power of two come from the caller (Ops::rcp, Ops::exp2), so that a host
// program can measure it.
#pragma once

#include <cmath>

#ifdef __HIPCC__
#define HUB_GELU_FN __host__ __device__ __forceinline__
#else
#define HUB_GELU_FN inline
#endif

namespace hub {

struct Gelu {
  float h, d;
};

// Branch-free, so that the 32 evaluations of a lane per tile interleave with
// each other and the matrix instructions (the library's erff branches on its
// argument).  F = Phi(-|z|) = 1/2 - |z| p(z^2) for z^2 < 2, else phi-weighted,
// e^{-z^2/2} q r(q) with q = 1 / (1 + |z| / sqrt 8); p and r are least-maximum
// fits of those functions (to 3e-10 and 2e-9), p's constant 1 / sqrt(2 pi) in
// two parts.  F is at most 1/2, and both results take it in one rounding of
// their own: h = max(z, 0) - |z| F, d = F - |z| phi or, for z > 0, one less
// that.  Against 64 bits on the GPU, at most and rms: h over [-8, 8] 2.4e-7 and
// 5.1e-8 (with erff and expf 4.5e-7, 6.8e-8), over [-2, 2] 1.1e-7, 2.0e-8 (1.6e-7,
// 2.8e-8); d 1.2e-7, 2.2e-8 (1.4e-7, 2.6e-8) and 1.2e-7, 2.5e-8 (1.5e-7, 2.9e-8).
template <typename Ops>
HUB_GELU_FN Gelu gelu_both(float z) {
  const float u = z * z, a = fabsf(z);
  float p = 4.20559104e-07f;
  p = fmaf(p, u, -8.76378544e-06f);
  p = fmaf(p, u, 0.000114431277f);
  p = fmaf(p, u, -0.00118652277f);
  p = fmaf(p, u, 0.00997322239f);
  p = fmaf(p, u, -0.0664903149f);
  const float al = a * -1.13352e-8f;  // |z| times what the constant below has too much
  const float near = fmaf(a, -0.398942292f, 0.5f) - fmaf(a * u, p, al);
  const float q = Ops::rcp(fmaf(a, 0.35355338f, 1.0f));
  float r = -0.101734042f;
  r = fmaf(r, q, 0.278311163f);
  r = fmaf(r, q, 0.0145136295f);
  r = fmaf(r, q, 0.171200514f);
  r = fmaf(r, q, 0.137736544f);
  const float e = Ops::exp2(u * -0.72134752f);
  const float F = u < 2.0f ? near : r * q * e;
  const float ah = a * -0.398942292f;
  const float g = fmaf(ah, e, fmaf(fmaf(a, -0.398942292f, -ah) - al, e, F));
  // (an infinite z > 0 is kept from 0 times infinity: h = z)
  const float b = fmaxf(-a, z > 0.0f ? -3.402823466e38f : z);
  return {fmaf(b, F, fmaxf(z, 0.0f)), z > 0.0f ? 1.0f - g : g};
}

}  // namespace hub
