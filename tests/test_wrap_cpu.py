"""Wrapped tap arithmetic of the kernels, compiled for the host: every index
that a sampling position can give lies inside its level."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_06040_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include "ntc_device.hpp"
using namespace ntc;

static long bad = 0;
static void check(int i, int n, float rn) {
  const int want = (int)((((long long)i % n) + n) % n);
  if (wrap_near(i, n, rn) != want && bad++ < 10) printf("i %d n %d rn %a: %d, not %d\n", i, n, rn, wrap_near(i, n, rn), want);
}

int main() {
  unsigned seed = 1;
  auto rnd = [&] { return (int)((seed = seed * 1664525u + 1013904223u) >> 8); };  // 24 bits
  for (int n = 1; n <= 16384; ++n) {
    // the two FP32 numbers around 1 / n (that number itself for powers of two)
    const float r0 = 1.0f / (float)n, r1 = std::nextafter(r0, (double)r0 * n < 1.0 ? 1.0f : 0.0f);
    const int far = n < 4 ? 1 << 22 : (1 << 24) + 2 * n;
    for (float rn : {r0, (n & (n - 1)) ? r1 : r0}) {
      for (int d = 0; d <= 4; ++d)
        for (int s : {-1, 1}) {
          check(s * (far - d), n, rn);
          check(s * d, n, rn);
          const int q = far / n * n;
          for (int m : {q, q - n, q / 2 / n * n, n})
            if (std::abs(m) + d <= far) {
              check(s * (m + d), n, rn);
              check(s * (m - d), n, rn);
            }
        }
      for (int k = 0; k < 64; ++k) {
        const int i = rnd() % (far + 1);
        check(i, n, rn);
        check(-i, n, rn);
      }
    }
  }
  // levels past n_levels: sides of level 0, zero scales, position 0 for finite
  // coordinates and the lower limit for others
  for (int w = 4; w <= 16384; ++w) {
    LevelArgs A;
    std::memset(&A, 0, sizeof A);
    A.w = w;
    A.h = 16388 - w;
    A.sx = A.sy = 0.5f;
    for (bool used : {false, true}) {
      A.fw = used ? (float)A.w : 0.0f;
      A.fh = used ? (float)A.h : 0.0f;
      const LevelSel L = level_sel(A);
      for (float u : {0.3f, -1e30f, 3e38f, INFINITY, -INFINITY, NAN}) {
        float x = std::fma(u, L.fw, -0.5f) + L.sx, y = std::fma(u, L.fh, -0.5f) + L.sy;
        x = std::fmin(std::fmax(x, -16777216.0f), 16777216.0f);
        y = std::fmin(std::fmax(y, -16777216.0f), 16777216.0f);
        check((int)std::floor(x), L.w, L.rw);
        check((int)std::floor(y), L.h, L.rh);
      }
    }
  }
  printf("%ld wrong\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_wrapped_indices_stay_inside(tmp_path):
    src = tmp_path / "wrap.hip"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "wrap")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-ffp-contract=off", "-I" + CSRC,
                    "-o", exe, str(src)], check=True)
    p = subprocess.run([exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout
