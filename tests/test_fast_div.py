"""Division by run-time constants (FastDiv), the arithmetic under every kernel's addresses, compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r'''
#include <cstdio>
#include "f8_device.h"
// For a divisor d: around every multiple-of-d boundary that a scan of quotients meets, at both ends of the range, and on random numerators.
static unsigned long long seed = 88172645463325252ull;
static unsigned rnd() { seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17; return (unsigned)(seed >> 33); }
static bool check(unsigned d) {
  const f8::FastDiv f(d);
  auto ok = [&](unsigned n) { return f.div(n) == n / d; };
  const unsigned top = 0x7fffffffu;
  for (unsigned k = 0; k < 40; ++k) {
    if (!ok(k) || !ok(top - k) || !ok(rnd() & top)) return false;
    const unsigned m = rnd() % (top / d + 1) * d;                     // a multiple of d
    if (!ok(m) || (m && !ok(m - 1)) || (m < top && !ok(m + 1))) return false;
  }
  const unsigned last = top / d * d;
  return ok(last) && (!last || ok(last - 1));
}
int main() {
  if (f8::FastDiv().d != 1 || f8::FastDiv().div(12345) != 12345) return 2;
  for (unsigned d = 1; d <= 70000; ++d) if (!check(d)) { std::printf("%u\n", d); return 1; }
  for (int i = 0; i < 200000; ++i) { const unsigned d = rnd() | 1u; if (d <= 0x7fffffffu && !check(d)) { std::printf("%u\n", d); return 1; } }
  for (int s = 1; s < 31; ++s) for (int e = -1; e <= 1; ++e) if (!check((1u << s) + e)) { std::printf("%u\n", (1u << s) + e); return 1; }
  if (!check(0x7fffffffu)) return 1;
  std::puts("ok");
  return 0;
}
'''


def test_fast_div_is_exact_below_2_to_the_31(tmp_path):
    src, exe = tmp_path / "div.hip", tmp_path / "div"
    src.write_text(SOURCE)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    subprocess.run([hipcc, "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2202_05239_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
