"""Range starts of grouped binning (csrc/kfranges.h) on the CPU: whatever the
event offsets (not ascending, negative, past the end, not covering the hits)
and whatever the layers, either a block is flagged or every range start is
written, ascending, and holds exactly its hits.  The blocks of the pass are
those of bin_kernel: runs of consecutive hits, each with its own bracket of
events."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "kfranges.h"
using namespace kfranges;
// returns whether a block is flagged; seg starts at -7
static bool pass(const std::vector<int32_t>& eoff, int E, int L, const std::vector<int>& layer, int per, bool check,
                 std::vector<int32_t>& seg) {
  const int n = (int)layer.size();
  bool ok = true;
  seg.assign(E * L + 1, -7);
  if (n == 0) seg.assign(E * L + 1, 0);
  if (check)
    for (int e = 0; e < E; ++e) ok = tiles(eoff.data(), E, n, e) && ok;
  for (int i0 = 0; i0 < n; i0 += per) {
    const int i1 = i0 + per < n ? i0 + per : n;
    const int elo = event_of(eoff.data(), 0, E, i0), ehi = event_of(eoff.data(), elo, E, i1 - 1) + 1;
    for (int i = i0; i < i1; ++i) {
      const int l = layer[i], lp = i > 0 ? layer[i - 1] : -1, e = event_of(eoff.data(), elo, ehi, i);
      if (e < 0 || e >= E) { printf("event out of range\n"); return false; }
      if (l < 0 || l >= L) { ok = false; continue; }
      ok = range_starts(eoff.data(), E, L, n, i, e, l, lp, seg.data()) && ok;
    }
  }
  return !ok;
}
static bool sound(const std::vector<int32_t>& eoff, int E, int L, const std::vector<int>& layer,
                  const std::vector<int32_t>& seg) {
  const int n = (int)layer.size();
  if (seg[0] != 0 || seg[E * L] != n) return false;
  for (int s = 0; s < E * L; ++s) {
    if (seg[s + 1] < seg[s]) return false;
    for (int i = seg[s]; i < seg[s + 1]; ++i)
      if (layer[i] != s % L || i < eoff[s / L] || i >= eoff[s / L + 1]) return false;
  }
  return true;
}
int main() {
  std::mt19937 g(3);
  long unsound = 0, unflagged = 0, flagged = 0, missed_without = 0, refused = 0;
  std::vector<int32_t> seg;
  auto one = [&](const std::vector<int32_t>& eoff, int E, int L, const std::vector<int>& layer, int per, bool good) {
    const bool f = pass(eoff, E, L, layer, per, true, seg);
    if (f) ++flagged; else { ++unflagged; unsound += !sound(eoff, E, L, layer, seg); }
    refused += f && good;
    const bool f0 = pass(eoff, E, L, layer, per, false, seg);
    if (!f0) missed_without += !sound(eoff, E, L, layer, seg);
  };
  // offsets that descend, all hits on one layer
  one({0, 60, 20, 100}, 3, 2, std::vector<int>(100, 0), 256, false);
  // every offset vector of up to three events over up to five hits
  for (int n = 0; n <= 5; ++n)
    for (int E = 1; E <= 3; ++E)
      for (int L = 1; L <= 2; ++L) {
        std::vector<int32_t> eoff(E + 1, -1);
        for (;;) {
          for (int m = 0; m < (1 << n); ++m) {
            std::vector<int> layer(n);
            bool valid = true;
            for (int i = 0; i < n; ++i) { layer[i] = (m >> i) & 1; valid = valid && layer[i] < L; }
            for (int per = 1; per <= n + 1; per += 2) one(eoff, E, L, layer, per, false);
          }
          int k = 0;
          while (k <= E && ++eoff[k] > n + 1) eoff[k++] = -1;
          if (k > E) break;
        }
      }
  // larger ones: ordered input, then one offset or one layer changed
  for (int c = 0; c < 20000; ++c) {
    const int E = 1 + g() % 12, L = 1 + g() % 6;
    std::vector<int32_t> eoff{0};
    std::vector<int> layer;
    for (int e = 0; e < E; ++e) {
      for (int l = 0; l < L; ++l) layer.insert(layer.end(), g() % 3 ? g() % 9 : 0, l);
      eoff.push_back((int)layer.size());
    }
    const int per = 1 + g() % 40;
    one(eoff, E, L, layer, per, true);
    const int n = (int)layer.size();
    auto off = eoff;
    off[g() % (E + 1)] = (int)(g() % (n + 20)) - 10;
    one(off, E, L, layer, per, false);
    if (n) {
      layer[g() % n] = (int)(g() % (L + 2)) - 1;
      one(eoff, E, L, layer, per, false);
    }
  }
  printf("%ld %ld %ld %ld %ld\n", unsound, refused, unflagged, flagged, missed_without);
  return 0;
}
"""


def test_no_unflagged_input_leaves_a_range_start_unwritten(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    (tmp_path / "r.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), str(tmp_path / "r.hip"), "-o",
                    str(tmp_path / "r")], check=True, capture_output=True)
    r = subprocess.run([str(tmp_path / "r")], check=True, capture_output=True, text=True).stdout.split()
    unsound, refused, unflagged, flagged, missed_without = (int(v) for v in r)
    assert unsound == 0 and refused == 0, r
    assert unflagged > 20000 and flagged > 20000, r
    assert missed_without > 0, r  # (the hits' order alone does not tell)


def test_grid_of_a_grouped_sort_stays_in_bounds(tmp_path):
    """part_blocks: the blocks of every call whose launch stays below 2^32
    threads, -1 at and above (a product in 32 bits would wrap there)."""
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    (tmp_path / "g.hip").write_text(r"""
#include <cstdio>
#include "kfranges.h"
int main() {
  const long long R[] = {1, 17, 4194302, 4194303, 4194304, 4250000, 8388607, 1ll << 30, (1ll << 31) - 2};
  const int N[] = {0, 1023, 1024, 2147483647};
  for (long long r : R) for (int n : N) for (int t : {256, 1024})
    printf("%lld %d %d %lld\n", r, n, t, (long long)kfranges::part_blocks(n, 1024, r, t));
}
""")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), str(tmp_path / "g.hip"), "-o",
                    str(tmp_path / "g")], check=True, capture_output=True)
    lines = subprocess.run([str(tmp_path / "g")], check=True, capture_output=True, text=True).stdout.splitlines()
    refused = 0
    for line in lines:
        r, n, t, got = map(int, line.split())
        blocks = n // 1024 + r
        assert got == (blocks if blocks * t < 2 ** 32 else -1), line
        refused += got < 0
    assert 0 < refused < len(lines)
