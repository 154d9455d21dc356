"""Waves per CU of the build kernel (csrc/kfplan.h), on the CPU: eight (what
its registers allow) wherever a candidate cap of 4 and more leaves the LDS for
it, in every arithmetic, state and window; seven or six at the caps below whose
records or pools do not fit; and the block width that gives them."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CU_LDS = 160 * 1024

PROGRAM = r"""
#include <cstdio>
#include "kfplan.h"
int main() {
  for (int t : {4, 8}) for (int l = 0; l < 2; ++l) for (int h = 0; h < 2; ++h) for (int cap = 1; cap <= 8; ++cap) {
    printf("%d %d %d %d %d", t, l, h, cap, plan_lanes(14, cap, t, l, h, 163840));
    for (int lanes : {256, 128, 64}) printf(" %zu", lds_plan(14, lanes / 64, cap, t, l, h).total);
    printf("\n");
  }
  printf("%d\n", plan_lanes(14, 6, 8, false, true, 1024));
}
"""


def test_waves_per_cu(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    (tmp_path / "w.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-w", "-I",
                    os.path.join(ROOT, "paper_1711_06571_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(tmp_path / "w.hip"), "-o", str(tmp_path / "w")], check=True, capture_output=True)
    lines = subprocess.run([str(tmp_path / "w")], check=True, capture_output=True, text=True).stdout.splitlines()
    assert int(lines.pop()) == 0  # no width fits
    assert len(lines) == 64
    for line in lines:
        t, learned, hyb, cap, lanes, *total = map(int, line.split())
        waves = {w: min(8, CU_LDS // b * (w // 64)) for w, b in zip((256, 128, 64), total)}
        least = 8 if cap >= 4 or (t == 4 and not learned) else 6 if cap == 1 else 7
        assert waves[lanes] == max(waves.values()) >= least, line
        assert lanes == max(w for w in waves if waves[w] == waves[lanes]), line
