"""Host arithmetic of what the head's gradients are dealt to (no GPU): every element once, none outside, for launches of up to 2^41 threads."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_04865_amd", "csrc")

# rows, features and classes; workgroups per row block and per features as the kernels that write the feature gradients launch them:
# 32 x 32 (float32) and 8 x 256 (wide rows).  2^33 features, in either, and one more block of rows; 8.4 million rows of 2048
CASES = [(1, 64, 1), (37, 384, 4), (45056, 768, 3), (5592405, 1536, 1), (5592405 + 32, 1536, 2), (1 << 23, 2048, 4), (8400000, 2048, 4),
         (1 << 30, 64, 1)]
PROGRAM = r"""
#include "slide_internal.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
int main(int argc, char** argv) {
  const long long rows = atoll(argv[1]);
  const int D = atoi(argv[2]), len = atoi(argv[3]) * (D + 1), rb = atoi(argv[4]), db = atoi(argv[5]);
  const unsigned gx = (unsigned)((rows + rb - 1) / rb), gy = (D + db - 1) / db;
  const long long wgs = (long long)gx * gy;
  std::vector<int> seen(len, 0);
  long long outside = 0;
  // every workgroup of a small launch; the first and the last few hundred thousand of a large one, and some in between
  auto look = [&](long long w) {
    for (unsigned t = 0; t < 256; ++t) {
      const sl::Share s = sl::wg_share((unsigned)(w / gy), (unsigned)(w % gy), gx, gy, t);
      if (s.first < 0 || s.step != wgs * 256) ++outside;
      for (long long i = s.first; i < len && s.step > 0; i += s.step)
        if (i < 0) ++outside; else ++seen[i];
    }
  };
  const long long ends = wgs < 1 << 19 ? wgs : 1 << 18;
  for (long long w = 0; w < ends; ++w) look(w);
  for (long long w = ends; w < wgs - ends; w += (wgs - 2 * ends) / 65536 + 1) look(w);
  for (long long w = wgs - ends > ends ? wgs - ends : ends; w < wgs; ++w) look(w);
  int once = 0;
  for (int v : seen) once += v == 1;
  std::printf("%lld %d %d\n", outside, once, len);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2403_04865_amd.build import _hipcc
    d = tmp_path_factory.mktemp("shares")
    (d / "shares.hip").write_text(PROGRAM)
    subprocess.run([_hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(d / "shares.hip"), "-o", str(d / "shares")],
                   check=True, capture_output=True)
    return str(d / "shares")


@pytest.mark.parametrize("rows,D,C", CASES)
@pytest.mark.parametrize("rb,db", [(32, 32), (8, 256)])
def test_every_element_once(program, rows, D, C, rb, db):
    out = subprocess.run([program, str(rows), str(D), str(C), str(rb), str(db)], check=True, capture_output=True, text=True).stdout
    outside, once, n = map(int, out.split())
    assert outside == 0 and once == n == C * (D + 1)
