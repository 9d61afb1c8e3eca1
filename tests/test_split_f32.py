"""The cut of a float32 operand into three bf16 terms (split_f32.h), compiled for the host (no GPU)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_04865_amd", "csrc")
PROGRAM = r"""
#include "split_f32.h"
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
using namespace sl;
static float term(const Split& s, int i, int e) {
  const __bf16 v = s.t[i][e];
  unsigned short u;
  memcpy(&u, &v, 2);
  return __builtin_bit_cast(float, (unsigned)u << 16);
}
int main() {
  std::mt19937_64 r(1);
  std::normal_distribution<float> normal;
  long long inexact = 0, n = 0;
  double worst = 0, sum = 0;
  float x[8], y[8];
  auto look = [&](bool products) {
    const Split a = split8(x), b = split8(y);
    for (int e = 0; e < 8; ++e) {
      inexact += ((double)term(a, 0, e) + term(a, 1, e)) + term(a, 2, e) != x[e];
      double taken = 0;   // every term of it is exact in 64 bits, and so nearly is the sum
      for (int t = 0; t < 6; ++t) taken += (double)term(a, TERM_A[t], e) * term(b, TERM_B[t], e);
      const double off = taken / ((double)x[e] * y[e]) - 1.0;
      if (!products) continue;
      worst = std::fmax(worst, std::fabs(off));
      sum += off;
      ++n;
    }
  };
  const float edge[8] = {0x1.01fffep0f, 0x1.00fffep0f, 0x1.017f7ep0f, 0x1.fffffep0f, 1.f, 0x1.810102p0f, -0x1.01fffep0f, 0x1.03fffep0f};
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 8; ++j) {
      for (int e = 0; e < 8; ++e) { x[e] = edge[i] * std::ldexp(1.f, 3 * e - 12); y[e] = edge[j]; }
      look(true);
    }
  n = 0; sum = 0;   // (the edges are no sample)
  for (int i = 0; i < 1 << 18; ++i) {
    for (int e = 0; e < 8; ++e) { x[e] = normal(r); y[e] = normal(r); }
    look(true);
  }
  for (int i = 0; i < 1 << 16; ++i) {   // any bits: from 2^-110 up to what rounds to an infinite leading term
    for (int e = 0; e < 8; ++e) {
      do x[e] = __builtin_bit_cast(float, (unsigned)r()); while (!(std::fabs(x[e]) >= 0x1p-110f && std::fabs(x[e]) < 0x1.ffp127f));
      y[e] = 1.f;
    }
    look(false);
  }
  for (int i = 0; i < 1 << 16; ++i) {   // scaled: down to the smallest float
    for (int e = 0; e < 8; ++e)
      do x[e] = __builtin_bit_cast(float, (unsigned)r()); while (!(std::fabs(x[e]) < 0x1p79f));
    const Split a = split8(x, -SPLIT_UP);
    for (int e = 0; e < 8; ++e) inexact += ((double)term(a, 0, e) + term(a, 1, e)) + term(a, 2, e) != x[e] * -(double)SPLIT_UP;
  }
  std::printf("%lld %.17g %.17g\n", inexact, worst, sum / n);
}
"""


# Terms are rests rounded to nearest: the middle one is at most 2^-8 of the leading unit, the trailing one 2^-17.  The three products that
# are not taken are at most 2 * 2^-25 + 2^-34 of a product of two numbers in [1, 2), and their signs are even: two million of them average to
# 2^-24 / sqrt(2e6) or less.
def test_terms_and_the_products_taken(tmp_path):
    from paper_2403_04865_amd.build import _hipcc
    (tmp_path / "split.hip").write_text(PROGRAM)
    subprocess.run([_hipcc(), "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "split.hip"), "-o", str(tmp_path / "split")],
                   check=True, capture_output=True)
    inexact, worst, mean = subprocess.run([str(tmp_path / "split")], check=True, capture_output=True, text=True).stdout.split()
    print(inexact, worst, mean)
    assert int(inexact) == 0
    assert float(worst) < 2 ** -24 * 1.002
    assert abs(float(mean)) < 3 * 2 ** -24 / 2e6 ** 0.5
