"""Where hits of at most a given chi2 can lie (csrc/kfreach.h), checked on
the CPU against brute force: for random predictions (narrow to far wider than
the layer, correlated up to and past what FP32 resolves, anywhere in phi and
beyond the barrel's end) and hits all over the layer, every hit inside
the search window whose chi2, computed in FP32 as the builder does, is within
the bound lies in exactly one part of its own row.  The bounds are strict
inequalities with margins, so no hit may be missed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include "kfreach.h"
using namespace kfreach;
int main(int argc, char** argv) {
  const int nz = atoi(argv[1]);
  const float radius = atof(argv[2]), zh = 100.f;
  std::mt19937_64 g(nz * 1000 + (int)radius);
  auto U = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(g); };
  long nones = 0, missed = 0, twice = 0, inside = 0, all = 0, given = 0;
  for (int c = 0; c < 600; ++c) {
    const float sig = 0.01f, sz = 0.1f;
    // prediction and its covariance along the arc and in z
    const double ph = U(0, 2 * M_PI), su = std::exp(U(std::log(0.01), std::log(3000.))),
                 sw = std::exp(U(std::log(0.05), std::log(3000.)));
    // (every fourth nearer to full correlation than FP32 can tell, or past it)
    double rho = c % 4 == 3 ? 1 - (c & 8 ? U(-3e-7, 1e-6) : U(-1e-2, 1e-4)) : 1 - std::exp(U(std::log(3e-6), 0.));
    if (c & 1) rho = -rho;
    const float fx = radius * std::cos(ph), fy = radius * std::sin(ph), fz = U(-130, 130);
    const float suu = su * su, sww = sw * sw, suw = rho * su * sw;
    const float irr = 1.f / sqrtf(fx * fx + fy * fy);
    const float hwin = 3.f * sqrtf(suu + sig * sig) / radius, dz = 3.f * sqrtf(sww + sz * sz);
    float phip = atan2f(fy, fx);
    if (phip < 0.f) phip += kTwoPiF;
    Reach q;
    q.v = bound_word(sig * sig * 1.00001f, sz * sz);
    q.rad = (f_bits(radius * 0.98f) & 0xFFFF0000u) | bound_word(0.f, radius * 1.02f);
    if (!q.usable(suu, sww)) continue;
    const bool none = q.none(suu, suw, sww);
    nones += none;
    ++given;
    const float bound = std::exp(U(std::log(1e-4), std::log(30.)));
    q.set(bound, suu, suw, sww);
    const float hw = hwin + kEpsPhi, dzw = dz + kEpsZ;
    const Rows rw = rows_of(fz, fminf(dzw, q.dz(sww)), zh, nz);
    for (int k = 0; k < 4000; ++k) {
      // hits near the prediction (in its own metric) and anywhere
      const double a = k & 1 ? U(-1, 1) * std::fmin(5 * su, M_PI * radius) : U(-M_PI, M_PI) * radius;
      const double hr = radius * U(0.98, 1.02), hp = ph + a / radius;
      float hx = hr * std::cos(hp), hy = hr * std::sin(hp);
      float hz = k & 1 ? fz + (float)(U(-5, 5) * std::fmin(sw, 60.)) + (k & 2 ? (float)(rho * sw / su * a) : 0.f) : (float)U(-120, 120);
      double ph64 = std::atan2((double)hy, (double)hx);
      if (ph64 < 0) ph64 += 2 * M_PI;
      const float sp = (float)ph64;
      // window test and chi2 in FP32
      const float cr = fx * hy - fy * hx, dt = fx * hx + fy * hy;
      if (!(fabsf(hz - fz) <= dz) || !(fabsf(atan2f(cr, dt)) <= hwin)) continue;
      const float ctx = -fy * irr, cty = fx * irr;
      const float r0 = ctx * (hx - fx) + cty * (hy - fy), r1 = hz - fz;
      const float c0 = cosf(sp), s0 = sinf(sp), v = sig * sig;
      const float V0 = v * s0 * s0, V1 = -v * s0 * c0, V3 = v * c0 * c0, V5 = sz * sz;
      const float s00 = suu + ctx * ctx * V0 + 2.f * ctx * cty * V1 + cty * cty * V3, s01 = suw, s11 = sww + V5;
      const float det = s00 * s11 - s01 * s01;
      if (!(s00 > 0.f) || !(det > 0.f)) continue;
      const float c2 = (s11 * r0 * r0 - 2.f * s01 * r0 * r1 + s00 * r1 * r1) * (1.0f / det);
      if (none) ++missed;  // (a positive determinant after all)
      ++all;
      if (!(c2 <= bound)) continue;
      ++inside;
      double fr = std::floor(((double)hz + (double)zh) * nz / (2.0 * (double)zh));
      const int row = fr < 0 ? 0 : (fr > nz - 1 ? nz - 1 : (int)fr);
      int n = 0;
      if (row >= rw.lo && row <= rw.hi)
        {
          float al[2], ah[2];
          reach_arcs(q, suu, suw, sww, sqrtf(fx * fx + fy * fy), fz, hw, dzw, row, nz, zh, al, ah);
          for (int i = 0; i < 4; ++i) {
            float lo, hi;
            arc_part(phip, al[i >> 1], ah[i >> 1], i & 1, lo, hi);
            if (lo <= hi && sp >= lo && sp <= hi) ++n;
          }
        }
      if (n == 0) ++missed;
      if (n > 1) ++twice;
    }
  }
  printf("%ld %ld %ld %ld %ld %ld\n", missed, twice, inside, all, given, nones);
  return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("reach")
    (d / "reach.hip").write_text(PROGRAM)
    out = d / "reach"
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), str(d / "reach.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


@pytest.mark.parametrize("nz,radius", [(16, 16.0), (16, 68.0), (1, 20.0), (64, 40.0), (5, 128.0)])
def test_no_hit_within_the_bound_is_missed(exe, nz, radius):
    r = subprocess.run([exe, str(nz), str(radius)], check=True, capture_output=True, text=True).stdout.split()
    missed, twice, inside, seen, given, nones = (int(v) for v in r)
    assert missed == 0 and twice == 0, r
    assert inside > 10000 and inside < seen and given > 400 and nones > 20, r  # (the bounds bite, and are given)
