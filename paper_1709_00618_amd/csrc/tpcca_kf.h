// Kalman-filter primitives of the gfx950 tracker (GPU library internal),
// shared by the sector tracker's kernels and the second phase.
//
// Track model of Sec. 2 (Rohr, LHCP 2017): state (y, z, sin phi,
// tan lambda, q/pT) at a pad-row plane x of a sector frame, propagated with
// Bz only.  Compiled with -ffp-contract=off and correctly rounded FP32
// division and square root: fused multiply-adds appear only where written.
#pragma once
#include <hip/hip_runtime.h>

#include "tpcca_internal.h"

namespace tpcca {

// Correctly rounded division and square root in fewer instructions than the
// general ones (quotient 4 after 3 for the reciprocal, which quotients by the
// same number share, against 11; root 7 against 16), for operands in the
// middle of the exponent range.  A step holds seven quotients by four numbers
// and three roots, and its instructions are what bounds the fit of few
// tracklets and keeps its VALU half busy on many.
//   reciprocal  v_rcp_f32 (1 ulp) and one Newton step; equal to the correctly
//               rounded one for every 24-bit significand (all checked)
//   quotient    Markstein's: with the correctly rounded reciprocal r, q = n r
//               corrected once by its exact residual is correctly rounded
//               (IBM J. Res. Dev. 34, 1990); v_div_fixup_f32 gives zeros,
//               infinities and NaN their results.  Exact while n and the
//               quotient lie above 2^-102 (below, the residual underflows).
//   root        v_sqrt_f32 (1 ulp) corrected once by its exact residual over
//               twice the root; equal to the correctly rounded one for every
//               float from 2^-96 to 2^120 (all checked), 0 and infinity.
// Checked on the device by tests/test_gpu_arithmetic.py.  Where an operand may
// lie outside, the callers below take the general operations.
struct KRecip {
  float d, r;
};
__device__ __forceinline__ KRecip kf_recip(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return {d, __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r)};
}
__device__ __forceinline__ float kf_div(float n, const KRecip &k) {
  const float q = n * k.r;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-k.d, q, n), k.r, q), k.d, n);
}
__device__ __forceinline__ float kf_sqrt(float x) {
  const float g = __builtin_amdgcn_sqrtf(x), h = 0.5f * __builtin_amdgcn_rsqf(x);
  const float q = __builtin_fmaf(__builtin_fmaf(-g, g, x), h, g);
  return __builtin_amdgcn_classf(x, 0x260) ? x : q;  // +-0, +infinity
}

// Track state at plane x: p = (y, z, sin phi, tan lambda, q/pT), C lower
// triangle (00,10,11,20,21,22,30,31,32,33,40,41,42,43,44).
struct KState {
  float p[5];
  float C[15];
  float x;
};

// Propagation x -> x1 with Bz only (Sec. 2).  sin(phi) is linear in x
// along a circle of curvature kB q/pT; dy = dx (s0 + s1) / (c0 + c1); the
// arc length (signed like dx) is the chord times the Maclaurin series of
// asin(u)/u to u^8, u = chord |k| / 2.  The Jacobian is the simplified one
// that drops the curvature term of the arc length.  C <- F C F^T.
//
// What a step takes of the two directions sin phi = s0, s1 and of dx: the
// displacement dy, the chord and its square, the Jacobian's a and b, and dy
// over the chord.  In the short forms above or, kShort false, by the general
// division and root.
struct KGeo {
  float dy, ch2, chs, a, b, dych;
};
template <bool kShort>
__device__ __forceinline__ KGeo kf_geometry(const ParamsDev &P, float dx, float s0, float s1) {
  auto root = [](float x) { return kShort ? kf_sqrt(x) : sqrtf(x); };
  auto div = [](float n, const KRecip &k) { return kShort ? kf_div(n, k) : n / k.d; };
  KGeo q;
  const float c0 = root(__builtin_fmaf(-s0, s0, 1.0f));
  const float c1 = root(__builtin_fmaf(-s1, s1, 1.0f));
  const KRecip rc0 = kf_recip(c0), rc1 = kf_recip(c1), rcc = kf_recip(c0 + c1);
  const float tt = div(s0 + s1, rcc);
  q.dy = dx * tt;
  q.ch2 = __builtin_fmaf(q.dy, q.dy, dx * dx);
  const float ch = root(q.ch2);
  q.chs = dx < 0.0f ? -ch : ch;
  q.a = div(dx * (2.0f + tt * (div(s0, rc0) + div(s1, rc1))), rcc);
  q.b = div(dx * P.kB * dx * (1.0f + div(tt * s1, rc1)), rcc);
  q.dych = div(q.dy, kf_recip(q.chs));
  return q;
}

// The step itself, for a caller that has no use for the state once the track
// turned back (|sin phi| beyond the limit, where the state ends up undefined):
// without a way round it, the new state takes the old one's registers.
//
// Where dx and kB keep the short forms exact (P.tiny), what is left to look at is
// s0 + s1 (c0 and c1 are 0, NaN or 2^-12 to 1): from 2^-60 on, dy and its
// quotient lie above 2^-92, and quotients of a smaller s0 or s1 only enter sums
// with 1 or 2.  Below it the wave takes the general forms, which give its other
// lanes the same.  One compare: a lone wave's time goes by its instructions.
__device__ __forceinline__ bool kf_step(const ParamsDev &P, KState &s, float x1) {
  const float dx = x1 - s.x;
  const float kk = P.kB * s.p[4];
  const float s0 = s.p[2];
  const float s1 = __builtin_fmaf(kk, dx, s0);
  KGeo q = kf_geometry<true>(P, dx, s0, s1);
  if (__builtin_expect(__ballot(fabsf(s0 + s1) < P.tiny) != 0ull, 0)) q = kf_geometry<false>(P, dx, s0, s1);
  const float u2 = q.ch2 * kk * kk * 0.25f;
  float h = (float)(35.0 / 1152.0);
  h = __builtin_fmaf(u2, h, (float)(5.0 / 112.0));
  h = __builtin_fmaf(u2, h, (float)(3.0 / 40.0));
  h = __builtin_fmaf(u2, h, (float)(1.0 / 6.0));
  h = __builtin_fmaf(u2, h, 1.0f);
  const float dS = q.chs * h;
  const float t = s.p[3];

  const float a = q.a, b = q.b;
  const float g = fabsf(q.chs) > 0.0f ? t * q.dych : 0.0f;
  const float cz = g * a;
  const float dzq = g * b;
  const float e = dS;
  const float f = P.kB * dx;

  s.p[0] = s.p[0] + q.dy;
  s.p[1] = s.p[1] + t * dS;
  s.p[2] = s1;
  s.x = x1;

  float *C = s.C;
  const float c00 = C[0], c10 = C[1], c11 = C[2], c20 = C[3], c21 = C[4], c22 = C[5];
  const float c30 = C[6], c31 = C[7], c32 = C[8], c33 = C[9];
  const float c40 = C[10], c41 = C[11], c42 = C[12], c43 = C[13], c44 = C[14];
  const float fc00 = c00 + a * c20 + b * c40;
  const float fc02 = c20 + a * c22 + b * c42;
  const float fc04 = c40 + a * c42 + b * c44;
  const float fc10 = c10 + cz * c20 + e * c30 + dzq * c40;
  const float fc11 = c11 + cz * c21 + e * c31 + dzq * c41;
  const float fc12 = c21 + cz * c22 + e * c32 + dzq * c42;
  const float fc13 = c31 + cz * c32 + e * c33 + dzq * c43;
  const float fc14 = c41 + cz * c42 + e * c43 + dzq * c44;
  const float fc20 = c20 + f * c40;
  const float fc21 = c21 + f * c41;
  const float fc22 = c22 + f * c42;
  const float fc23 = c32 + f * c43;
  const float fc24 = c42 + f * c44;
  C[0] = fc00 + a * fc02 + b * fc04;
  C[1] = fc10 + a * fc12 + b * fc14;
  C[2] = fc11 + cz * fc12 + e * fc13 + dzq * fc14;
  C[3] = fc20 + a * fc22 + b * fc24;
  C[4] = fc21 + cz * fc22 + e * fc23 + dzq * fc24;
  C[5] = fc22 + f * fc24;
  C[6] = c30 + a * c32 + b * c43;
  C[7] = c31 + cz * c32 + e * c33 + dzq * c43;
  C[8] = c32 + f * c43;
  C[9] = c33;
  C[10] = c40 + a * c42 + b * c44;
  C[11] = c41 + cz * c42 + e * c43 + dzq * c44;
  C[12] = c42 + f * c44;
  C[13] = c43;
  C[14] = c44;
  return fabsf(s1) <= P.max_sin;
}

// As kf_step, the state left as it is when the step fails.
__device__ __forceinline__ bool kf_propagate(const ParamsDev &P, KState &s, float x1) {
  const float s1 = __builtin_fmaf(P.kB * s.p[4], x1 - s.x, s.p[2]);
  if (!(fabsf(s1) <= P.max_sin)) return false;
  return kf_step(P, s, x1);
}

// 1 / det.  The short form is exact for 2^-126 to 2^126 and gives no normal
// number outside (checked for every float): there the wave divides.
__device__ __forceinline__ float kf_inverse(float det) {
  float inv = kf_div(1.0f, kf_recip(det));
  if (__builtin_expect(__ballot(!__builtin_amdgcn_classf(inv, 0x108)) != 0ull, 0)) inv = 1.0f / det;  // +-normal
  return inv;
}

// A 2-D measurement against the state: residual, inverse of S = C_yz + R and
// chi2.  The test of a searched hit and the update with it share it.  Fails
// (its values undefined) unless det S > 0.
struct KMeas {
  float r0, r1, i00, i10, i11, chi2;
};
__device__ __forceinline__ bool kf_meas(const ParamsDev &P, const KState &s, float ym, float zm, KMeas &m) {
  m.r0 = ym - s.p[0];
  m.r1 = zm - s.p[1];
  const float s00 = s.C[0] + P.ery;
  const float s10 = s.C[1];
  const float s11 = s.C[2] + P.erz;
  const float det = s00 * s11 - s10 * s10;
  const float inv = kf_inverse(det);
  m.i00 = s11 * inv;
  m.i10 = -s10 * inv;
  m.i11 = s00 * inv;
  const float v0 = m.i00 * m.r0 + m.i10 * m.r1;
  const float v1 = m.i10 * m.r0 + m.i11 * m.r1;
  m.chi2 = m.r0 * v0 + m.r1 * v1;
  return det > 0.0f;
}

// Kalman gain with a measurement: K = C H^T S^-1, p += K r, C -= K H C.
__device__ __forceinline__ void kf_gain(KState &s, const KMeas &m) {
  // first two columns of C (old values), row k = (C_k0, C_k1)
  const float cj0[5] = {s.C[0], s.C[1], s.C[3], s.C[6], s.C[10]};
  const float cj1[5] = {s.C[1], s.C[2], s.C[4], s.C[7], s.C[11]};
  float k0[5], k1[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    k0[k] = cj0[k] * m.i00 + cj1[k] * m.i10;
    k1[k] = cj0[k] * m.i10 + cj1[k] * m.i11;
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) s.p[k] = s.p[k] + k0[k] * m.r0 + k1[k] * m.r1;
  int idx = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j) {
      s.C[idx] = s.C[idx] - (k0[i] * cj0[j] + k1[i] * cj1[j]);
      ++idx;
    }
}

__device__ __forceinline__ bool kf_chi2(const ParamsDev &P, const KState &s, float ym, float zm, float &chi2) {
  KMeas m;
  if (!kf_meas(P, s, ym, zm, m)) return false;
  chi2 = m.chi2;
  return true;
}

__device__ __forceinline__ bool kf_update(const ParamsDev &P, KState &s, float ym, float zm, float &chi2) {
  KMeas m;
  if (!kf_meas(P, s, ym, zm, m)) return false;
  chi2 = m.chi2;
  kf_gain(s, m);
  return true;
}

}  // namespace tpcca
