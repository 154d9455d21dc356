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
// Margins of a window's stored-value intervals (rad, cm), and of the z rows'
// edges by the barrel's half-length: the edges and a position's row are formed
// in FP32 from up to twice that (some 4 roundings of 6e-8).
constexpr float kEpsPhi = 1e-5f, kEpsZ = 1e-4f, kEpsRow = 5e-7f;

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
  const float e = dz + kEpsRow * zh;
  const int lo = row_of(z - e, zh, nz), hi = row_of(z + e, zh, nz), m = row_of(z, zh, nz);
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
// s11] and residuals r0 (along the arc) and r1 (z), D = det S and k = s01/s11,
//   D chi2 = num = s11 (r0 - k r1)^2 + D/s11 r1^2,
// so per z row r0 lies in a strip, and r0 = radius * sin(angle from the
// prediction): up to two arcs of stored phi, the second mirrored about the
// quarter turn.  s01 is the prediction's; s00 and s11 are the prediction's
// (suu, sww) plus at most the largest variances of the hits looked at, whose
// covariances couple z neither to x nor to y.
//
// The builder computes num and D in FP32: num loses at most 10 ulp of
// s11 r0^2 + s00 r1^2 and D gains at most 4 ulp of s00 s11, so a hit whose
// computed chi2 is at most c2 has
//   (r0 - k r1)^2 <= c2 (C + 4u s00) - C r1^2 / s11 + 10u (r0^2 + s00/s11 r1^2)
// with C = D / s11, which near full correlation may be negative (u = 2^-24;
// twice the factors are used).  The same bounds r1 where 1 - rho^2 is not
// lost in rounding: c2_z is c2 with that margin, else infinite.
struct Reach {
  float c2, c2_z;
  uint32_t v;    // largest transverse and z variances of the hits (bound_word)
  uint32_t rad;  // smallest and largest radius, upper halves
  KFR float lam() const { return bits_f(v & 0xFFFF0000u); }
  KFR float vzz() const { return bits_f(v << 16); }
  KFR float rlo() const { return bits_f(rad & 0xFFFF0000u); }
  KFR float rhi() const { return bits_f(rad << 16); }
  KFR float dz(float sww) const { return sqrtf(c2_z * (sww + vzz())) * 1.0001f + kEpsZ; }
  // whether a bound can be given at all
  KFR bool usable(float suu, float sww) const {
    return lam() < 1e30f && vzz() < 1e30f && (rad >> 16) != 0u && fabsf(suu) < 1e30f && sww > 0.f && sww < 1e30f;
  }
  // whether no hit can have a positive determinant (an FP32 covariance that
  // lost its positivity): the builder then accepts none
  KFR bool none(float suu, float suw, float sww) const {
    const float s00 = fabsf(suu) + lam();
    return suu + lam() - suw * suw / (sww + vzz()) < -3e-6f * s00;
  }
  // sets the bound (>= 0); rho^2 is largest without the hit's own variances
  KFR void set(float bound, float suu, float suw, float sww) {
    const float e = suu - 1e-5f * lam(), d = 1.f - suw * suw / (e * sww) - 2e-7f;
    c2 = bound;
    c2_z = e > 0.f && d > 1e-5f ? bound * (1.f + 4e-6f / d) * 1.0001f : 1e30f;
  }
};

// The arcs of row `row` as angles from the prediction, clipped to the window:
// [lo[0], hi[0]] and [lo[1], hi[1]], empty where lo > hi; an arc of [-4, 4] is
// the whole circle.  rc, z: the prediction's radius and z; hw, dzw: the
// window's half-widths.
KFR void reach_arcs(const Reach& q, float suu, float suw, float sww, float rc, float z, float hw, float dzw, int row, int nz,
                    float zh, float lo[2], float hi[2]) {
  const float pi = 3.1415927f, eps = 4e-5f;
  const float lam = q.lam(), s00 = fabsf(suu) + lam, s11 = sww + q.vzz();
  const float rh = 2.f * zh / (float)nz, zb = q.dz(sww), zm = zb < dzw ? zb : dzw;
  lo[0] = lo[1] = 1.f;
  hi[0] = hi[1] = 0.f;
  // residuals in z of the row's hits (the end rows hold all hits beyond)
  const float er = kEpsZ + kEpsRow * zh;
  float l1 = row == 0 ? -zm : (float)row * rh - zh - z - er;
  float h1 = row == nz - 1 ? zm : (float)(row + 1) * rh - zh - z + er;
  l1 = l1 < -zm ? -zm : l1;
  h1 = h1 > zm ? zm : h1;
  if (!(zm < 1e9f)) {  // (nothing to gain, and the squares below stay finite)
    lo[0] = hw < 3.14159f ? -hw : -4.f;
    hi[0] = hw < 3.14159f ? hw : 4.f;
    return;
  }
  if (!(l1 <= h1)) return;
  const float m1 = l1 > 0.f ? l1 : (h1 < 0.f ? -h1 : 0.f), M1 = fmaxf(fabsf(l1), fabsf(h1));
  const float rhi = q.rhi(), rlo = q.rlo();
  const float cmax = suu + lam - suw * suw / s11 + 2e-6f * s00, cmin = suu - 1e-5f * lam - suw * suw / sww - 2e-6f * s00;
  const float w2 = q.c2 * (fmaxf(cmax, 0.f) + 5e-7f * s00) * 1.0002f -
                   (cmin > 0.f ? cmin * m1 * m1 / s11 : cmin * M1 * M1 / sww) +
                   1.2e-6f * (rhi * rhi + s00 / sww * M1 * M1);
  if (!(w2 >= 0.f)) return;
  const float ka = suw / sww, kb = suw / s11;
  const float x0 = ka * l1, x1 = ka * h1, x2 = kb * l1, x3 = kb * h1;
  const float h = sqrtf(w2) * 1.0001f + 4e-6f * rc + 1e-5f * (fabsf(x0) + fabsf(x1));
  const float r0l = fminf(fminf(x0, x1), fminf(x2, x3)) - h, r0h = fmaxf(fmaxf(x0, x1), fmaxf(x2, x3)) + h;
  const float sl = r0l / (r0l < 0.f ? rlo : rhi), su = r0h / (r0h > 0.f ? rlo : rhi);
  if (!(sl < 1.f) || !(su > -1.f)) return;
  const bool ol = sl < -0.9999f, ou = su > 0.9999f;
  const float dl = ol ? -0.5f * pi : asinf(sl) - eps, dh = ou ? 0.5f * pi : asinf(su) + eps;
  if (ol && ou) {  // every angle
    lo[0] = hw < 3.14159f ? -hw : -4.f;
    hi[0] = hw < 3.14159f ? hw : 4.f;
  } else if (ol || ou) {  // the two arcs meet at a quarter turn
    lo[0] = ou ? dl : -pi - dh;
    hi[0] = ou ? pi - dl : dh;
    if (hw < 0.5f * pi) {
      lo[0] = fmaxf(lo[0], -hw);
      hi[0] = fminf(hi[0], hw);
    }
  } else {
    lo[0] = fmaxf(dl, -hw);
    hi[0] = fminf(dh, hw);
    if (pi - dh <= hw + eps || pi + dl <= hw + eps) {  // the window reaches the second
      lo[1] = pi - dh;
      hi[1] = pi - dl;
    }
  }
}
// Part i (0, 1) of an arc in stored phi, cut where it wraps; a > b: empty.
// The parts of a row's arcs are disjoint.
KFR void arc_part(float phip, float lo, float hi, int i, float& a, float& b) {
  a = 1.f;
  b = 0.f;
  if (!(lo <= hi)) return;
  if (hi - lo > 7.f) {
    a = i == 0 ? 0.f : 1.f;
    b = i == 0 ? kTwoPiF : 0.f;
    return;
  }
  float u0 = phip + lo, u1 = phip + hi;
  if (u0 >= kTwoPiF) { u0 -= kTwoPiF; u1 -= kTwoPiF; }
  if (u1 < 0.f) { u0 += kTwoPiF; u1 += kTwoPiF; }
  wrap_part(u0, u1, i, a, b);
}

}  // namespace kfreach
