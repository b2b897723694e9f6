"""Host checks of the runtime's parts that need no GPU, compiled for the host:
the sponge's quotient against the division, the pool of side streams."""
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
  const double exact[] = {1.0, 2.0, 1.5, 1.25, 4.0};
  std::mt19937_64 rng(7);
  std::normal_distribution<double> mant(0.0, 1.0);
  std::uniform_int_distribution<int> expo(-120, 120);
  int bad = 0;
  auto check = [&](double x, double plus) {
    const double got = fwi::quotient(x, fwi::reciprocal(plus)), want = x / plus;
    if (std::isnan(want) ? !std::isnan(got) : bits(got) != bits(want))
      if (bad++ < 10) std::printf("%a / %a: %a, not %a\n", x, plus, got, want);
  };
  for (double plus : exact)
    for (double x : special) check(x, plus);
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


CHAINS = r"""
#include <atomic>
#include <cstdio>
#include <set>
#include <thread>
#include "fwi_chains.h"
static std::atomic<int> made{0};
static std::atomic<bool> finished[256];  // by event
struct Api {
  using Stream = int;
  using Event = int;
  using Error = int;
  static constexpr int kOk = 0;
  static int make_stream(int* s) { *s = 1000 + made++; return 0; }
  static int make_event(int* e) { *e = made++; finished[*e] = true; return 0; }
  static bool done(int e) { return finished[e]; }
  static bool shared(int s) { return s != 2; }
};
using Pool = fwi::ChainPool<Api>;
static int failures = 0;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); ++failures; } } while (0)
// a call of n chains: takes a set, records its joins and gives it back
static Pool::Set* call(Pool& p, int dev, int user, int n, bool done) {
  Pool::Set* s = nullptr;
  CHECK(p.take(dev, user, n, &s) == 0);
  if (!s) return s;
  CHECK(s->streams >= n);
  for (int i = 1; i < n; ++i) finished[s->join[i]] = done;
  p.give(s);
  return s;
}
int main() {
  {
    Pool p;
    Pool::Set* a = call(p, 0, 10, 2, false);
    CHECK(call(p, 0, 10, 3, false) == a);          // its own stream's next call
    Pool::Set* b = call(p, 0, 11, 2, false);       // another stream, a's work still running
    CHECK(b && b != a);
    for (int i = 1; i < 3; ++i) CHECK(b->stream[1] != a->stream[i]);
    CHECK(call(p, 1, 12, 2, true)->device == 1);   // another device
    finished[a->join[1]] = true;
    Pool::Set* c = call(p, 0, 13, 2, false);       // one of a's two chains still runs
    CHECK(c != a && c != b);
    finished[a->join[1]] = finished[a->join[2]] = true;
    CHECK(call(p, 0, 14, 2, true) == a);           // done: anyone's
    CHECK(call(p, 0, 11, 2, false) == b);
  }
  {
    Pool p;                                        // a handle that names a stream per thread
    Pool::Set* a = call(p, 0, 2, 2, false);
    CHECK(call(p, 0, 2, 2, false) != a);
  }
  {
    Pool p;                                        // bounded: then one chain
    std::set<Pool::Set*> seen;
    for (int u = 0; u < fwi::kMaxChainSets; ++u) seen.insert(call(p, 0, 100 + u, 2, false));
    CHECK((int)seen.size() == fwi::kMaxChainSets && !seen.count(nullptr));
    CHECK(call(p, 0, 99, 2, false) == nullptr);
    CHECK(call(p, 0, 100, 2, false) != nullptr);
    CHECK(call(p, 1, 99, 2, true) != nullptr);
  }
  {
    Pool p;                                        // no set is two calls' at once
    std::atomic<int> held[2 * fwi::kMaxChainSets + 1] = {};
    std::atomic<int> shared{0}, none{0};
    std::vector<std::thread> t;
    for (int u = 0; u < 6; ++u)
      t.emplace_back([&, u] {
        for (int i = 0; i < 2000; ++i) {
          Pool::Set* s = nullptr;
          p.take(0, 10 + u % 3, 2, &s);
          if (!s) { ++none; continue; }
          const int id = s->join[1] % (2 * fwi::kMaxChainSets + 1);
          if (held[id]++) ++shared;
          held[id]--;
          p.give(s);
        }
      });
    for (auto& x : t) x.join();
    CHECK(shared == 0 && none == 0);
  }
  return failures != 0;
}
"""


def test_side_streams_of_busy_calls_are_not_shared(tmp_path):
    """A set of side streams goes to another stream's call only when its work
    is done; there is a bound on the sets of a device."""
    r = subprocess.run([compiled(tmp_path, "chains", CHAINS)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
