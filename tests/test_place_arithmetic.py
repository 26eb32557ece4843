"""Places at the end of the largest plan (2^31 - 2 particles): the strided walks of
the moments and the 64-probe search of the leaf offsets stay inside their ranges.
The headers' own arithmetic, compiled for the host."""
import os
import subprocess

import pytest

from paper_2009_00767_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstdint>
#include <type_traits>
#include "device_common.h"
using namespace sffmm;

// places a group's lanes visit of slice j of [s0, s1), with the types the kernels use
template <class P>
static long walk(void (*slice)(const P2mPlan&, int, int, int32_t, int32_t, P&, P&),
                 const P2mPlan& pl, int j, int32_t s0, int32_t s1) {
  P lo, hi;
  slice(pl, 2, j, s0, s1, lo, hi);
  long seen = 0;
  for (int r = 0; r < 64; ++r)
    for (P i = lo + r; i < hi; i += 64) {
      if (++seen > 1 << 16 || (int64_t)i < s0 || (int64_t)i >= s1) return -1;
    }
  return seen;
}

int main() {
  const int32_t n = 0x7FFFFFFF - 1;
  int bad = 0;
  for (int ls : {0, 3})
    for (int32_t s0 : {n - 1, n - 63, n - 64, n - 65, n - 5000}) {
      P2mPlan pl{};
      pl.lgS[2] = ls;
      long all = 0;
      for (int j = 0; j < 1 << ls; ++j) {
        const long w = walk(p2m_slice, pl, j, s0, n);
        if (w < 0) { all = -1; break; }
        all += w;
      }
      if (all != n - s0) { printf("slices %d of [%d, %d): %ld\n", ls, s0, n, all); bad = 1; }
    }
  for (int32_t m : {1, 63, 64, 65, 1 << 20, n - 64, n - 63, n})
    if (probe_step(m) != ((int64_t)m + 63) / 64) { printf("step of %d: %d\n", m, probe_step(m)); bad = 1; }
  return bad;
}
"""


def test_places_near_the_largest_plan(tmp_path):
    src, exe = tmp_path / "places.hip", tmp_path / "places"
    src.write_text(PROGRAM)
    # -fwrapv: a signed overflow shows as the wrapped value
    subprocess.run([build.HIPCC] + build.COMMON + ["-fwrapv", "-O0", "-I", build.CSRC, str(src),
                                                   "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
