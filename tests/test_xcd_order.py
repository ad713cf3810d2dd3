"""How the units of a persistent kernel are dealt to XCDs and workgroups, compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r'''
#include <cstdio>
#include <vector>
#include "f8_device.h"
// Every unit once, in order along an XCD; the k-th eighth on XCD k; the XCDs' shares differ by one unit at most, and so do the runs on one XCD.
static bool check(int n, unsigned grid) {
  std::vector<char> seen(n, 0);
  int total[8] = {}, least[8], most[8] = {};
  for (int k = 0; k < 8; ++k) least[k] = 1 << 30;
  for (unsigned b = 0; b < grid; ++b) {
    const f8::XcdRange r = f8::xcd_run(b, grid, n);
    const int k = b & 7, len = r.end - r.first;
    if (len < 1 || r.step != 1 || r.first < 0 || r.end > n) return false;
    if (r.first != (b < 8 ? (int)((long long)n / 8 * k + (k < n % 8 ? k : n % 8)) : f8::xcd_run(b - 8, grid, n).end)) return false;
    for (int t = r.first; t < r.end; ++t) if (seen[t]++) return false;
    total[k] += len;
    if (len < least[k]) least[k] = len;
    if (len > most[k]) most[k] = len;
  }
  for (int t = 0; t < n; ++t) if (!seen[t]) return false;
  for (int k = 0; k < 8 && k < (int)grid; ++k)
    if (total[k] < n / 8 || total[k] > n / 8 + 1 || most[k] > least[k] + 1) return false;
  return true;
}
int main() {
  for (int n = 1; n < 2100; ++n) if (!check(n, n < 512 ? n : 512)) { std::printf("%d\n", n); return 1; }
  for (int n = 1 << 20; n < (1 << 20) + 600; n += 37) if (!check(n, 512)) { std::printf("%d\n", n); return 1; }
  std::puts("ok");
  return 0;
}
'''


def test_runs_of_neighbouring_units(tmp_path):
    src, exe = tmp_path / "run.hip", tmp_path / "run"
    src.write_text(SOURCE)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    subprocess.run([hipcc, "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2202_05239_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
