"""How a run of steps on LDS tiles is cut into launches (no GPU).

The launches alternate between the handle's own planes and the second set.  Each takes
an even number of steps, at most m, they add up to the run, and at every moment
the time level is the one whose state the own planes hold, also when a launch
fails: a host copy of the two planes is followed through every run and every failure.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "lbm_axi_tile.h"
#include <cstdio>
int main() {
  long long runs = 0;
  for (int m = 4; m <= 8; m += 2)  // what the plan chooses
    for (int n = 4; n <= 200; n += 2) {
      const int pairs = (n + 2 * m - 1) / (2 * m);
      for (int bad = 0; bad <= 2 * pairs; ++bad) {  // the launch that fails; the last: none
        long long t = 40, level[2] = {40, -1};      // level held by the own planes and the second ones
        int calls = 0, err = 0;
        const int rc = lbmaxi::tile_pairs(t, n, m, [&](int i, int steps, long long at) {
          if (i != calls++ || steps < 2 || steps > m || (steps & 1)) err = 1;
          if (level[i & 1] != at) err = 2;
          if (i == bad) return -3;
          level[(i & 1) ^ 1] = at + steps;
          return 0;
        });
        if (err) return std::printf("n %d m %d: launch error %d\n", n, m, err), 1;
        if (t != level[0]) return std::printf("n %d m %d, launch %d fails: level %lld, planes at %lld\n", n, m, bad, t, level[0]), 1;
        if (bad == 2 * pairs ? (rc != 0 || t != 40 + n || calls != 2 * pairs) : rc != -3) return std::printf("result\n"), 1;
        ++runs;
      }
    }
  std::printf("%lld runs\n", runs);
  return 0;
}
"""


def test_level_and_planes_agree_in_every_run_and_failure(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "pairs.hip", tmp_path / "pairs"
    src.write_text(SOURCE)
    subprocess.check_call([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_1409_5929_amd", "csrc"), "-o", str(exe), str(src)],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "runs" in r.stdout, r.stdout
