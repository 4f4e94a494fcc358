#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

// The FP32 Kalman filter shared by the tracklet constructor (tpc_track.hip)
// and the track refit (tpc_refit.hip): one track per lane.  Internal header of
// the library.
//
// State at plane x: (y, z, sin(phi), tan(lambda), q/pT); curvature C = k q/pT.
// Exact helix transport: sin2 = sin1 + C dx, dy = dx (sin1+sin2)/(cos1+cos2),
// dz = tan(lambda) s_T with s_T = sign(dx) L asin(u)/u, L = |(dx,dy)|, u = |C|L/2;
// analytic Jacobian for the covariance; no process noise.

namespace tpc_kf {

// Two forms of the state, which differ only in where the covariance (lower
// triangle, row-major, 15 entries) lives: KState keeps it in LDS, entry k at
// c[k * 64] (the lane's column of a [15][64] block, so the lanes of a wave
// hit distinct banks); KStateR keeps it in registers.  The functions below
// take either and reach entry k through cv(s, k).
struct KState {
  float p[5];
  float *c;
  float x, chi2;
};
struct KStateR {
  float p[5];
  float c[15];
  float x, chi2;
};
__device__ __forceinline__ float &cv(KState &s, int k) { return s.c[k * 64]; }
__device__ __forceinline__ float &cv(KStateR &s, int k) { return s.c[k]; }

// Square root, reciprocal and quotient of normal numbers far from overflow,
// without the scaling and fix-up steps that the general forms spend on the
// rest (5, 3 and 3 instructions here against about 13, 10 and 10): a hardware
// approximation (1 ulp), one Newton step whose residual an FMA forms exactly,
// and for the quotient one correction by its remainder (Markstein, Computation
// of elementary functions on the IBM RISC System/6000 processor, 1990).
// tests/test_gpu_kalman_roots.py compares them with sqrtf, 1.f / x and a / b:
// the same bits on every float between the limits of is_mid, and on 2^32
// quotients by either kind of reciprocal, the divisor's own and the one refined
// from its square root's approximation.
__device__ __forceinline__ float sqrt_n(float x, float &rs) {  // rs: about 1 / sqrt(x)
  rs = __builtin_amdgcn_rsqf(x);
  const float g = x * rs;
  return fmaf(fmaf(-g, g, x), 0.5f * rs, g);
}
__device__ __forceinline__ float refine_rcp(float x, float r) { return fmaf(fmaf(-x, r, 1.f), r, r); }
__device__ __forceinline__ float rcp_n(float x) { return refine_rcp(x, __builtin_amdgcn_rcpf(x)); }
__device__ __forceinline__ float div_by(float a, float b, float rb) {  // a / b, rb = rcp_n(b) or a refined one
  const float q = a * rb;
  return fmaf(fmaf(-b, q, a), rb, q);
}
// whether a value may go to the functions above
__device__ __forceinline__ bool is_mid(float x) { return fabsf(x) > 1e-25f && fabsf(x) < 1e25f; }

__device__ __forceinline__ float asin_over(float u) {  // asin(u)/u
#pragma clang fp contract(off)
  const float u2 = u * u;
  if (u < 0.03f) return fmaf(u2, fmaf(u2, 3.f / 40.f, 1.f / 6.f), 1.f);
  return asinf(u) / u;
}
__device__ __forceinline__ float asin_over_dd(float u) {  // (d/du asin(u)/u) / u
#pragma clang fp contract(off)
  const float u2 = u * u;
  if (u < 0.2f) return fmaf(u2, fmaf(u2, fmaf(u2, 35.f / 144.f, 15.f / 56.f), 0.3f), 1.f / 3.f);
  return (u / sqrtf(1.f - u2) - asinf(u)) / (u2 * u);
}

// How the transport, the update and the seed round is written out: contraction
// is off and each FMA is named.  Left to the compiler, which product of a sum
// enters an FMA depends on what surrounds the inlined code, and the tracklet
// fit alone compiles it into six bodies, chosen by the size of the batch: a
// unit's fit may not depend on what else the batch holds.  The forms are those
// the compiler had taken for all six (so at i == 1 below, where q0[1] * I01 is
// also a product of K0[0]).

// Transport of the state to a plane x2, parameter part; kept so that the
// covariance part can follow once a hit is found in that row.
struct Step {
  float dx, C, s1, s2, c1, c2, D, N, iD, dy, L, u, fu, sT, sg;
  float r1, r2, rL;  // about 1 / c1, 1 / c2, 1 / L
};

// ROWS: the two planes are pad rows of one geometry (1 .. 8192 cm, apart).
template <bool ROWS = false, class S>
__device__ __forceinline__ bool step_prepare(const S &s, float x2, float k, float sinmax, Step &t) {
#pragma clang fp contract(off)
  t.dx = x2 - s.x;
  t.C = k * s.p[4];
  t.s1 = s.p[2];
  t.s2 = fmaf(t.C, t.dx, t.s1);
  if (!(fabsf(t.s1) < sinmax) || !(fabsf(t.s2) < sinmax)) return false;
  t.c1 = sqrt_n(fmaf(-t.s1, t.s1, 1.f), t.r1);  // 1 - sinmax^2 or more
  t.c2 = sqrt_n(fmaf(-t.s2, t.s2, 1.f), t.r2);
  t.D = t.c1 + t.c2;
  t.N = t.s1 + t.s2;
  t.iD = rcp_n(t.D);
  t.dy = t.dx * t.N * t.iD;
  const float LL = fmaf(t.dx, t.dx, t.dy * t.dy);
  if (ROWS || is_mid(LL)) {
    t.L = sqrt_n(LL, t.rL);
  } else {  // planes that (nearly) coincide
    t.L = sqrtf(LL);
    t.rL = t.L > 0.f ? 1.f / t.L : 0.f;
  }
  t.u = fabsf(t.C) * t.L * 0.5f;
  if (!(t.u < 1.f)) return false;
  t.sg = t.dx < 0.f ? -1.f : 1.f;
  t.fu = asin_over(t.u);
  t.sT = t.sg * t.L * t.fu;
  return true;
}

// The position a prepared step leads to.
template <class S>
__device__ __forceinline__ float y_after(const S &s, const Step &t) {
  return s.p[0] + t.dy;
}
template <class S>
__device__ __forceinline__ float z_after(const S &s, const Step &t) {
  return fmaf(s.p[3], t.sT, s.p[1]);
}

// Apply a prepared step: parameters, and the covariance through the analytic
// Jacobian.
template <class S>
__device__ __forceinline__ void step_apply(S &s, const Step &t, float x2, float k) {
#pragma clang fp contract(off)
  const float dx = t.dx, s1 = t.s1, s2 = t.s2, c1 = t.c1, c2 = t.c2, D = t.D, N = t.N, iD = t.iD;
  const float dy = t.dy, L = t.L, u = t.u, fu = t.fu, sT = t.sT, sg = t.sg, C = t.C;
  const float tgl = s.p[3];
  const float iD2 = iD * iD;
  const float i2 = refine_rcp(c2, t.r2);
  const float a = dx * fmaf(2.f, D, N * (div_by(s1, c1, refine_rcp(c1, t.r1)) + div_by(s2, c2, i2))) * iD2;
  const float b = dx * k * dx * (D + div_by(N * s2, c2, i2)) * iD2;
  const float g = asin_over_dd(u);
  const float dsdy = L > 0.f ? sg * div_by(dy, L, refine_rcp(L, t.rL)) * fmaf(u * u, g, fu) : 0.f;
  const float dsdC = sg * C * L * L * L * g * 0.25f;
  const float cc = tgl * dsdy * a;
  const float d = sT;
  const float e = tgl * fmaf(dsdC, k, dsdy * b);
  const float f = k * dx;
  s.p[0] += dy;
  s.p[1] = fmaf(tgl, sT, s.p[1]);
  s.p[2] = s2;
  s.x = x2;
  // cov <- F cov F^T, F = I + {(0,2)=a, (0,4)=b, (1,2)=cc, (1,3)=d, (1,4)=e, (2,4)=f}
  const float P00 = cv(s, 0), P10 = cv(s, 1), P11 = cv(s, 2), P20 = cv(s, 3), P21 = cv(s, 4),
              P22 = cv(s, 5), P30 = cv(s, 6), P31 = cv(s, 7), P32 = cv(s, 8), P33 = cv(s, 9),
              P40 = cv(s, 10), P41 = cv(s, 11), P42 = cv(s, 12), P43 = cv(s, 13), P44 = cv(s, 14);
  // T = F P, rows 0..2
  const float T00 = fmaf(b, P40, fmaf(a, P20, P00));
  const float T02 = fmaf(b, P42, fmaf(a, P22, P20));
  const float T04 = fmaf(b, P44, fmaf(a, P42, P40));
  const float T10 = fmaf(e, P40, fmaf(d, P30, fmaf(cc, P20, P10)));
  const float T11 = fmaf(e, P41, fmaf(d, P31, fmaf(cc, P21, P11)));
  const float T12 = fmaf(e, P42, fmaf(d, P32, fmaf(cc, P22, P21)));
  const float T13 = fmaf(e, P43, fmaf(d, P33, fmaf(cc, P32, P31)));
  const float T14 = fmaf(e, P44, fmaf(d, P43, fmaf(cc, P42, P41)));
  const float T20 = fmaf(f, P40, P20);
  const float T21 = fmaf(f, P41, P21);
  const float T22 = fmaf(f, P42, P22);
  const float T23 = fmaf(f, P43, P32);
  const float T24 = fmaf(f, P44, P42);
  cv(s, 0) = fmaf(b, T04, fmaf(a, T02, T00));
  cv(s, 1) = fmaf(b, T14, fmaf(a, T12, T10));
  cv(s, 2) = fmaf(e, T14, fmaf(d, T13, fmaf(cc, T12, T11)));
  cv(s, 3) = fmaf(b, T24, fmaf(a, T22, T20));
  cv(s, 4) = fmaf(e, T24, fmaf(d, T23, fmaf(cc, T22, T21)));
  cv(s, 5) = fmaf(f, T24, T22);
  cv(s, 6) = fmaf(b, P43, fmaf(a, P32, P30));
  cv(s, 7) = fmaf(e, P43, fmaf(d, P33, fmaf(cc, P32, P31)));
  cv(s, 8) = fmaf(f, P43, P32);
  cv(s, 10) = fmaf(b, P44, fmaf(a, P42, P40));
  cv(s, 11) = fmaf(e, P44, fmaf(d, P43, fmaf(cc, P42, P41)));
  cv(s, 12) = fmaf(f, P44, P42);
}

// The measurement of residuals (r0, r1).  Z_FUSED: which product of a sum of
// two with the residuals enters the FMA unrounded, the y one's or the z one's
// (the chain fit's).  P_FIRST: the parameters before the covariance; the bits
// are the same.  The next row waits for them, and the fit with several lanes a
// seed has no other wave to run meanwhile: one chunk 451 us the whole call, 455
// with the covariance first.  The row loop of k_fit needs no scratch with the
// covariance first: 50 collisions 8.13 ms, so 8.25.
template <bool Z_FUSED = false, bool P_FIRST = false, class S>
__device__ __forceinline__ void kf_update(S &s, float r0, float r1, float sy2, float sz2) {
#pragma clang fp contract(off)
  const float S00 = cv(s, 0) + sy2, S01 = cv(s, 1), S11 = cv(s, 2) + sz2;
  const float det = fmaf(S00, S11, -(S01 * S01));
  const float idet = is_mid(det) ? rcp_n(det) : 1.f / det;
  const float I00 = S11 * idet, I01 = -S01 * idet, I11 = S00 * idet;
  // columns 0 and 1 of P (P_i0, P_i1)
  const float q0[5] = {cv(s, 0), cv(s, 1), cv(s, 3), cv(s, 6), cv(s, 10)};
  const float q1[5] = {cv(s, 1), cv(s, 2), cv(s, 4), cv(s, 7), cv(s, 11)};
  float K0[5], K1[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    K0[i] = fmaf(q0[i], I00, q1[i] * I01);
    K1[i] = i == 1 ? fmaf(q1[i], I11, q0[i] * I01) : fmaf(q0[i], I01, q1[i] * I11);
  }
  auto parameters = [&]() {
#pragma clang fp contract(off)
#pragma unroll
    for (int i = 0; i < 5; ++i) s.p[i] += Z_FUSED ? fmaf(K1[i], r1, K0[i] * r0) : fmaf(K0[i], r0, K1[i] * r1);
  };
  if (P_FIRST) parameters();
  int k = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j, ++k) cv(s, k) -= fmaf(K0[i], q0[j], K1[i] * q1[j]);
  if (!P_FIRST) parameters();
  if (Z_FUSED)
    s.chi2 += fmaf(r0, fmaf(r1, I01, r0 * I00), r1 * fmaf(r1, I11, r0 * I01));
  else
    s.chi2 += fmaf(r0, fmaf(I00, r0, I01 * r1), r1 * fmaf(I01, r0, I11 * r1));
}

template <class S>
__device__ __forceinline__ void cov_reset(S &s, const float *cov0) {
#pragma unroll
  for (int i = 0; i < 15; ++i) cv(s, i) = 0.f;
  cv(s, 0) = cov0[0];
  cv(s, 2) = cov0[1];
  cv(s, 5) = cov0[2];
  cv(s, 9) = cov0[3];
  cv(s, 14) = cov0[4];
}

// measurement of hit h relative to the reference (exact: integer difference)
template <bool Z_FUSED = false, bool P_FIRST = false, class S>
__device__ __forceinline__ void upd_hit(S &s, int2 yz, int Yr, int Zr, float sy2, float sz2) {
  kf_update<Z_FUSED, P_FIRST>(s, fmaf(float(yz.x - Yr), 1.f / 256.f, -s.p[0]), fmaf(float(yz.y - Zr), 1.f / 256.f, -s.p[1]), sy2, sz2);
}

// Length of (x, y); X_FUSED: which of the squares enters the FMA unrounded.
template <bool X_FUSED>
__device__ __forceinline__ float chord(float x, float y) {
#pragma clang fp contract(off)
  return sqrtf(X_FUSED ? fmaf(x, x, y * y) : fmaf(y, y, x * x));
}

// Three-point seed: the circle through (x0, 0), (x1, y1), (x2, y2) gives the
// curvature C and sin(phi) at the first point; tan(lambda) = z2 / s_T, with s_T
// the transverse arc length from the first point to the third.  y and z are
// relative to the first point.  The state starts at x0 with the diagonal
// covariance cov0.  False when the points are not distinct, the circle cannot
// join them or |sin(phi)| reaches smx.
template <bool X_FUSED = false, class S>
__device__ __forceinline__ bool seed3(S &s, float x0, float x1, float x2, float y1, float y2, float z2,
                                      float k, float smx, const float *cov0) {
#pragma clang fp contract(off)
  const float ax = x1 - x0, ay = y1, bx = x2 - x0, by = y2, cx = x2 - x1, cy = y2 - y1;
  const float d12 = chord<X_FUSED>(ax, ay), d13 = chord<X_FUSED>(bx, by), d23 = chord<X_FUSED>(cx, cy);
  bool ok = d12 > 0.f && d13 > 0.f && d23 > 0.f;
  const float C = ok ? 2.f * fmaf(ax, by, -(ay * bx)) / (d12 * d13 * d23) : 0.f;
  const float sa = ok ? C * d13 * 0.5f : 0.f;
  ok = ok && fabsf(sa) < 1.f;
  const float ca = sqrtf(fmaxf(0.f, fmaf(-sa, sa, 1.f)));
  const float sphi = ok ? fmaf(by / d13, ca, -(bx / d13 * sa)) : 0.f;
  ok = ok && fabsf(sphi) < smx;
  const float sT = ok ? d13 * asin_over(fabsf(sa)) : 1.f;
  s.p[0] = 0.f;
  s.p[1] = 0.f;
  s.p[2] = sphi;
  s.p[3] = z2 / sT;
  s.p[4] = k != 0.f ? C / k : 0.f;
  s.x = x0;
  s.chi2 = 0.f;
  cov_reset(s, cov0);
  return ok;
}

}  // namespace tpc_kf
