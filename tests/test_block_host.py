"""Host checks of what the LDS-resident sweeps compute with (no GPU needed):
the sponge's quotient compiled for the host against the division."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1406_1864_amd", "csrc")

QUOTIENT = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include "fwi_quotient.h"
static uint64_t bits(double x) { uint64_t b; std::memcpy(&b, &x, 8); return b; }
int main() {
  const double inf = INFINITY;
  const double special[] = {inf, -inf, NAN, 0.0, -0.0, 1e-90, -1e-90, 1.1e77, -1.1e77, 1.0, -3.0};
  std::mt19937_64 rng(7);
  std::normal_distribution<double> mant(0.0, 1.0);
  std::uniform_int_distribution<int> expo(-120, 120);
  int bad = 0;
  auto check = [&](double x, double plus) {
    const double got = fwi::quotient(x, plus, 1.0 / plus), want = x / plus;
    if (std::isnan(want) ? !std::isnan(got) : bits(got) != bits(want))
      if (bad++ < 10) std::printf("%a / %a: %a, not %a\n", x, plus, got, want);
  };
  // 1 + g over the depths of sponges 4 to 128 cells wide; x as the sweeps form
  // it, sums of float products
  for (int N : {4, 8, 20, 50, 128}) {
    const double a = 0.5 * 1e-3 * 3.0 * 2500.0 * std::log(1e3) / (2.0 * N * 10.0) / ((double)N * N);
    for (int k = 1; k <= N; ++k) {
      const double plus = 1.0 + a * (double)(k * k);
      for (double x : special) check(x, plus);
      for (int i = 0; i < 2000; ++i) {
        const float u = (float)std::ldexp(mant(rng), expo(rng)), w = (float)mant(rng), l = (float)mant(rng);
        check((2.0 - plus) * (double)u + (double)w * (double)l * (double)u, plus);
      }
    }
  }
  return bad != 0;
}
"""


def compiled(tmp_path, name, source):
    src = tmp_path / (name + ".cpp")
    src.write_text(source)
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I" + CSRC, "-pthread", str(src), "-o", exe],
                   check=True)
    return exe


def test_sponge_quotient_is_the_division(tmp_path):
    """Finite quotients, infinities, NaN and signed zeros, bit for bit."""
    r = subprocess.run([compiled(tmp_path, "quotient", QUOTIENT)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
