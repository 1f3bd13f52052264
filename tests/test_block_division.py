"""The multiplication that stands for position / block_size in the attention kernels, on the host: every block size at the edges of its
quotients and of the 31 bits of a position."""
import os
import subprocess

import pytest

from paper_2603_13289_amd import build

PROGRAM = r"""
#include <cstdio>
#include "common.h"
int main() {
  long bad = 0, seen = 0;
  const long top = (1l << 31) - 1;
  auto check = [&](rc::KvGeom& g, long n) {
    if (n < 0 || n > top) return;
    ++seen;
    if (rc::block_of(g, (int)n) != (int)(n / g.block_size)) { if (bad++ < 5) printf("%ld / %d\n", n, g.block_size); }
  };
  auto size = [&](long d) {
    if (d < 1 || d > top) return;
    rc::KvGeom g = {};
    g.block_size = (int)d;
    rc::set_block_division(&g);
    for (long q : {0l, 1l, 2l, 3l, 1000l, top / d - 1, top / d, top / d + 1})
      for (long e = -2; e <= 2; ++e) check(g, q * d + e);
    for (long n = top - 3; n <= top; ++n) check(g, n);
  };
  for (long d = 1; d <= 70000; ++d) size(d);
  for (int s = 16; s < 32; ++s)
    for (long e = -40; e <= 40; ++e) size((1l << s) + e);
  for (long d = 99991; d < top; d += 1000003) size(d);
  printf("%ld of %ld wrong\n", bad, seen);
  return bad != 0;
}
"""


def test_quotients(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "division.hip", str(tmp_path / "division")
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(src), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
