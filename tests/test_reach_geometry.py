"""The check of test_reach.py (no hit within the bound is missed, none is
counted twice) over barrels of other half-lengths and radii, from small ones
to some ten metres, where the row edges and the angles are formed in FP32 from
larger numbers; and with hits on the very edges of the rows whose chi2 is just
within the bound."""
import os
import shutil
import subprocess

import pytest

from test_reach import HIPCC, PROGRAM, ROOT


EDGES = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include "kfreach.h"
using namespace kfreach;
int main(int argc, char** argv) {
  const int nz = atoi(argv[1]); const float radius = atof(argv[2]), zh = atof(argv[3]);
  std::mt19937_64 g(7); auto U = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(g); };
  long missed = 0, twice = 0, inside = 0;
  for (int c = 0; c < 500000; ++c) {
    const float sz = 0.1f, sig = 0.01f;
    const float sw = std::exp(U(std::log(0.02), std::log(10.))), su = std::exp(U(std::log(0.02), std::log(10.)));
    const float suu = su * su, sww = sw * sw, suw = (c & 1) ? (float)(U(-1, 1) * su * sw * 0.99) : 0.f;
    Reach q; q.v = bound_word(sig * sig * 1.00001f, sz * sz);
    q.rad = (f_bits(radius * 0.98f) & 0xFFFF0000u) | bound_word(0.f, radius * 1.02f);
    const float bound = std::exp(U(std::log(0.1), std::log(30.)));
    q.set(bound, suu, suw, sww);
    const int edge = g() % (nz + 1);
    float hz = (float)(-(double)zh + 2.0 * (double)zh * edge / nz);
    if (c & 2) hz = std::nextafterf(hz, c & 4 ? 1e9f : -1e9f);
    const double V5 = sz * sz, lim = std::sqrt((double)bound * (sww + V5));
    const float fz = hz + (c & 8 ? -1 : 1) * (float)(lim * (1 - std::exp(U(-18, -1))));
    const float r1 = hz - fz;
    // best r0 for this r1, and near the ends of its range
    const double s00 = suu + (double)sig * sig, s11 = sww + V5, D = s00 * s11 - (double)suw * suw;
    const double k = suw / s11, room = (bound - (double)r1 * r1 / s11) * D / s11;
    if (room < 0) continue;
    const double r0w = k * r1 + U(-1, 1) * std::sqrt(room) * (c & 16 ? 1 : 0.999999);
    const double ph = U(0, 2 * M_PI);
    if (std::fabs(r0w) > radius) continue;
    const float fx = radius * std::cos(ph), fy = radius * std::sin(ph), irr = 1.f / sqrtf(fx * fx + fy * fy);
    const double an = std::asin(r0w / radius);
    const float hx = radius * std::cos(ph + an), hy = radius * std::sin(ph + an);
    const float ctx = -fy * irr, cty = fx * irr, r0 = ctx * (hx - fx) + cty * (hy - fy);
    const float f00 = suu + sig * sig, f11 = sww + sz * sz, det = f00 * f11 - suw * suw;
    const float c2 = (f11 * r0 * r0 - 2.f * suw * r0 * r1 + f00 * r1 * r1) * (1.f / det);
    if (!(det > 0) || !(c2 <= bound)) continue;
    double p64 = std::atan2((double)hy, (double)hx); if (p64 < 0) p64 += 2 * M_PI;
    const float sp = (float)p64; float phip = atan2f(fy, fx); if (phip < 0) phip += kTwoPiF;
    const float dz = 100.f * sqrtf(sww + sz * sz), hw = 4.f;
    const Rows rw = rows_of(fz, fminf(dz + kEpsZ, q.dz(sww)), zh, nz);
    double fr = std::floor(((double)hz + (double)zh) * nz / (2.0 * (double)zh));
    const int row = fr < 0 ? 0 : (fr > nz - 1 ? nz - 1 : (int)fr);
    ++inside; int n = 0;
    if (row >= rw.lo && row <= rw.hi) {
      float al[2], ah[2]; reach_arcs(q, suu, suw, sww, sqrtf(fx * fx + fy * fy), fz, hw, dz + kEpsZ, row, nz, zh, al, ah);
      for (int i = 0; i < 4; ++i) { float lo, hi; arc_part(phip, al[i >> 1], ah[i >> 1], i & 1, lo, hi); if (lo <= hi && sp >= lo && sp <= hi) ++n; }
    }
    missed += n == 0; twice += n > 1;
  }
  printf("%ld %ld %ld\n", missed, twice, inside);
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("reach_geometry")
    src = PROGRAM.replace("zh = 100.f;", "zh = atof(argv[3]), zs = zh / 100.f;")
    src = src.replace("fz = U(-130, 130);", "fz = U(-130, 130) * zs;").replace("(float)U(-120, 120);", "(float)U(-120, 120) * zs;")
    # hits close to the edges of the rows too
    src = src.replace("double ph64 = std::atan2",
                      "if (k % 5 == 0) hz = std::nextafterf(-zh + 2.f * zh * (float)(g() % (nz + 1)) / nz, k % 10 ? 1e9f : -1e9f);\n"
                      "      double ph64 = std::atan2")
    assert src.count("zs") >= 3 and "nextafterf" in src
    (d / "reach.hip").write_text(src)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), str(d / "reach.hip"), "-o", str(d / "reach")],
                   check=True, capture_output=True)
    return str(d / "reach")


@pytest.mark.parametrize("nz,radius,zh", [(16, 4.0, 1.0), (16, 68.0, 30.0), (33, 40.0, 270.0), (64, 110.0, 1000.0),
                                          (16, 700.0, 1000.0), (16, 1000.0, 3000.0), (128, 60.0, 3000.0),
                                          (7, 3000.0, 100.0)])
def test_no_hit_within_the_bound_is_missed(exe, nz, radius, zh):
    r = subprocess.run([exe, str(nz), str(radius), str(zh)], check=True, capture_output=True, text=True).stdout.split()
    missed, twice, inside, seen, given, nones = (int(v) for v in r)
    assert missed == 0 and twice == 0, r
    assert inside > 1000 and inside < seen and given > 400, r


@pytest.mark.parametrize("nz,radius,zh", [(16, 68.0, 100.0), (16, 4.0, 1.0), (64, 110.0, 1000.0), (16, 1000.0, 3000.0),
                                          (128, 60.0, 3000.0), (64, 100.0, 30000.0)])
def test_hits_on_row_edges_at_the_bound(tmp_path, nz, radius, zh):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    (tmp_path / "edges.hip").write_text(EDGES)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), str(tmp_path / "edges.hip"), "-o",
                    str(tmp_path / "edges")], check=True, capture_output=True)
    r = subprocess.run([str(tmp_path / "edges"), str(nz), str(radius), str(zh)], check=True, capture_output=True,
                       text=True).stdout.split()
    missed, twice, inside = (int(v) for v in r)
    assert missed == 0 and twice == 0 and inside > 100000, r
