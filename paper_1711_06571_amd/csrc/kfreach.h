// Geometry of the barrel builder's hit search (section 3.1): the z rows and
// stored-phi intervals of a search window, and of the part of it where hits
// of at most a given chi2 can lie.  Host and device code (a CPU test runs it).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace kfreach {

#define KFR __host__ __device__ inline

KFR float bits_f(uint32_t u) { return __builtin_bit_cast(float, u); }
KFR uint32_t f_bits(float f) { return __builtin_bit_cast(uint32_t, f); }

constexpr float kTwoPiF = 6.283185307179586f;
// Margins of a window's stored-value intervals (rad, cm).
constexpr float kEpsPhi = 1e-5f, kEpsZ = 1e-4f;

// z rows lo..hi a window overlaps, and the row of its middle; at(i) counts
// them from the middle row on.
struct Rows {
  int lo, hi, mid;
  KFR int at(int i) const { return i == 0 ? mid : lo + i - (i <= mid - lo ? 1 : 0); }
  KFR int n() const { return hi - lo + 1; }
};
KFR int row_of(float v, float zh, int nz) {
  const int i = (int)floorf((v + zh) * (float)nz / (2.f * zh));
  return i < 0 ? 0 : (i > nz - 1 ? nz - 1 : i);
}
KFR Rows rows_of(float z, float dz, float zh, int nz) {
  const int lo = row_of(z - dz, zh, nz), hi = row_of(z + dz, zh, nz), m = row_of(z, zh, nz);
  return {lo, hi, m < lo ? lo : (m > hi ? hi : m)};
}

// Part i (0, 1) of the stored phi in [lo, hi] (hi - lo below a turn), which
// may wrap at 0 or 2 pi; a > b: empty.  The parts are disjoint.
KFR void wrap_part(float lo, float hi, int i, float& a, float& b) {
  if (i & 1) {
    a = lo < 0.f ? lo + kTwoPiF : (hi >= kTwoPiF ? 0.f : 1.f);
    b = lo < 0.f ? kTwoPiF : (hi >= kTwoPiF ? hi - kTwoPiF : 0.f);
  } else {
    a = lo < 0.f ? 0.f : lo;
    b = hi >= kTwoPiF ? kTwoPiF : hi;
  }
}
// The intervals of stored phi within hw of phip (3.14159 and more: the whole
// circle): log2 of their number, and interval i.
KFR int phi_parts(float phip, float hw) {
  return hw < 3.14159f && (phip - hw < 0.f || phip + hw >= kTwoPiF) ? 1 : 0;
}
KFR void phi_part(float phip, float hw, int i, float& a, float& b) {
  if (hw >= 3.14159f) { a = 0.f; b = kTwoPiF; }
  else wrap_part(phip - hw, phip + hw, i, a, b);
}

// Two non-negative floats as the upper halves of one word, rounded up.
KFR uint32_t bound_word(float a, float b) {
  const uint32_t ua = (f_bits(a) + 0xFFFFu) >> 16, ub = (f_bits(b) + 0xFFFFu) >> 16;
  return (ua << 16) | ub;
}

// Where a layer's hits of chi2 at most c2 can lie: with S = [s00 s01; s01
// s11] and residuals r0 (along the arc) and r1 (z),
//   chi2 = r1^2 / s11 + (r0 - s01/s11 r1)^2 / (s00 - s01^2/s11),
// so per z row r0 lies in a strip, and r0 = radius * sin(angle from the
// prediction): up to two arcs of stored phi, the second mirrored about the
// quarter turn.  s01 is the prediction's; s00 and s11 are the prediction's
// (suu, sww) plus at most the largest variances of the hits looked at, whose
// covariances couple z neither to x nor to y.
struct Reach {
  float c2;      // (with the margin below)
  uint32_t v;    // largest transverse and z variances of the hits (bound_word)
  uint32_t rad;  // smallest and largest radius, upper halves
  KFR float lam() const { return bits_f(v & 0xFFFF0000u); }
  KFR float vzz() const { return bits_f(v << 16); }
  KFR float dz(float sww) const { return sqrtf(c2 * (sww + vzz())) * 1.0001f + kEpsZ; }
};
// 1 - rho^2 of S at least (without the hit's own variances), or 0 where no
// bound can be given.
KFR float reach_del(const Reach& q, float suu, float suw, float sww) {
  const float e = suu - 1e-5f * q.lam();
  const float d = 1.f - suw * suw / (e * sww) - 2e-7f;
  return e > 0.f && sww > 0.f && d > 1e-5f && q.lam() < 1e30f && q.vzz() < 1e30f && (q.rad >> 16) != 0u ? d : 0.f;
}
// The chi2 computed in FP32 may fall below its exact value by a part of
// 1.5e-6 / (1 - rho^2): the numerator's terms lose 10 ulp of their sum, of
// which at least 1 - |rho| remains, the determinant 4 ulp of s00 s11.
KFR float reach_margin(float del) { return (1.f + 4e-6f / del) * 1.0001f; }

// Part i (0..3) of row `row`: arc i / 2, cut where it wraps; a > b: empty.
// The parts are disjoint.  phip, z: the prediction; rc its radius; hw, dzw:
// the window's half-widths.
KFR void reach_part(const Reach& q, float suu, float suw, float sww, float rc, float z, float phip, float hw, float dzw,
                    int row, int nz, float zh, int i, float& a, float& b) {
  const float pi = 3.1415927f, eps = 4e-5f;
  const float lam = q.lam(), s11 = sww + q.vzz();
  const float rh = 2.f * zh / (float)nz, zb = q.dz(sww), zm = zb < dzw ? zb : dzw;
  a = 1.f;
  b = 0.f;
  // residuals in z of the row's hits (the end rows hold all hits beyond)
  float l1 = row == 0 ? -zm : (float)row * rh - zh - z - kEpsZ;
  float h1 = row == nz - 1 ? zm : (float)(row + 1) * rh - zh - z + kEpsZ;
  l1 = l1 < -zm ? -zm : l1;
  h1 = h1 > zm ? zm : h1;
  const float m1 = l1 > 0.f ? l1 : (h1 < 0.f ? -h1 : 0.f);
  const float rem = q.c2 - m1 * m1 / s11 * 0.9999f;
  if (!(l1 <= h1) || !(rem >= 0.f)) return;
  const float cond = suu + lam - suw * suw / s11 + 2e-6f * (suu + lam);
  const float ka = suw / sww, kb = suw / s11;
  const float x0 = ka * l1, x1 = ka * h1, x2 = kb * l1, x3 = kb * h1;
  const float h = sqrtf(rem * cond) * 1.0001f + 4e-6f * rc + 1e-5f * (fabsf(x0) + fabsf(x1));
  const float r0l = fminf(fminf(x0, x1), fminf(x2, x3)) - h, r0h = fmaxf(fmaxf(x0, x1), fmaxf(x2, x3)) + h;
  const float rlo = bits_f(q.rad & 0xFFFF0000u), rhi = bits_f(q.rad << 16);
  const float sl = r0l / (r0l < 0.f ? rlo : rhi), su = r0h / (r0h > 0.f ? rlo : rhi);
  if (!(sl < 1.f) || !(su > -1.f)) return;
  const bool ol = sl < -0.9999f, ou = su > 0.9999f;
  const float dl = ol ? -0.5f * pi : asinf(sl) - eps, dh = ou ? 0.5f * pi : asinf(su) + eps;
  float u0, u1;  // the arc, as angles from the prediction
  if (ol && ou) {  // every angle
    if (i & 2) return;
    if (hw >= 3.14159f) {
      a = i == 0 ? 0.f : 1.f;
      b = i == 0 ? kTwoPiF : 0.f;
      return;
    }
    u0 = -hw;
    u1 = hw;
  } else if (ol || ou) {  // the two arcs meet at a quarter turn
    if (i & 2) return;
    u0 = ou ? dl : -pi - dh;
    u1 = ou ? pi - dl : dh;
    if (hw < 0.5f * pi) {
      u0 = fmaxf(u0, -hw);
      u1 = fminf(u1, hw);
    }
  } else if (i & 2) {
    if (!(pi - dh <= hw + eps) && !(pi + dl <= hw + eps)) return;  // the window does not reach it
    u0 = pi - dh;
    u1 = pi - dl;
  } else {
    u0 = fmaxf(dl, -hw);
    u1 = fminf(dh, hw);
  }
  if (!(u0 <= u1)) return;
  float lo = phip + u0, hi = phip + u1;
  if (lo >= kTwoPiF) { lo -= kTwoPiF; hi -= kTwoPiF; }
  if (hi < 0.f) { lo += kTwoPiF; hi += kTwoPiF; }
  wrap_part(lo, hi, i, a, b);
}

}  // namespace kfreach
