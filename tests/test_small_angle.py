"""The short arctangents of the direct-sum kernels against the full one (no
GPU needed).

The kernels take atan(t) = t q(t^2) by the full polynomial's Horner chain
started at a lower coefficient when t is below a limit, and rely on the rounded
q being the full chain's.  The test evaluates both chains with the C library's
fused multiply-adds, on a grid of random t below each limit and at the limit's
neighbours, with the limits and degrees read from the kernel source.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2106_12655_amd import build

SRC = """
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#define constexpr const
#include "atan_poly.h"
static uint64_t s0 = 88172645463325252ull;
static double rnd(void) {
  s0 ^= s0 << 13; s0 ^= s0 >> 7; s0 ^= s0 << 17;
  return (double)(s0 >> 11) * 0x1p-53;
}
static float hf(float t, int d) {
  const float s = t * t;
  float q = kAtanQ[d];
  for (int k = d - 1; k >= 0; --k) q = fmaf(q, s, kAtanQ[k]);
  return q;
}
static double hd(double t, int d) {
  const double s = t * t;
  double q = kAtanQ64[d];
  for (int k = d - 1; k >= 0; --k) q = fma(q, s, kAtanQ64[k]);
  return q;
}
int main(int c, char** v) {  /* f32 or f64, degree, limit, count */
  const int d = atoi(v[2]);
  const double lim = atof(v[3]);
  const long n = atol(v[4]);
  long bad = 0;
  for (long i = 0; i < n; ++i) {
    /* the first ones just below the limit, then uniform and log-uniform */
    const double u = i < 1000 ? 1.0 - (double)(i + 1) * 0x1p-24 : rnd();
    double t = lim * (i & 1 ? u : exp2(-24.0 * (1.0 - u)));
    if (v[1][1] == '3') {
      const float f = (float)t;
      if (!((double)f < lim)) continue;
      bad += hf(f, d) != hf(f, LK_ATAN_DEG);
    } else {
      bad += hd(t, d) != hd(t, LK_ATAN_DEG64);
    }
  }
  printf("%ld\\n", bad);
  return 0;
}
"""


def _tiers():
    s = open(os.path.join(build.CSRC, "lk_ds.hip")).read()
    f32 = s[s.index("struct SmallAngle<float>"):s.index("struct SmallAngle<double>")]
    f64 = s[s.index("struct SmallAngle<double>"):]
    nums = lambda t, pat: [x.strip() for x in re.search(pat, t).group(1).split(",")]
    d32 = nums(f32, r"int D\[2\] = \{([^}]*)\}")
    l32 = [float(x.rstrip("f")) for x in nums(f32, r"lim\[2\] = \{([^}]*)\}")]
    d64 = nums(f64, r"int D\[2\] = \{([^}]*)\}")
    words = [int(x.rstrip("u"), 16) for x in nums(f64, r"lim\[2\] = \{([^}]*)\}")]
    import struct
    l64 = [struct.unpack("<d", struct.pack("<Q", w << 32))[0] for w in words]
    return [("f32", int(d), l) for d, l in zip(d32, l32)] + \
           [("f64", int(d), l) for d, l in zip(d64, l64)]


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")
@pytest.mark.parametrize("tier", range(4))
def test_short_chain_gives_the_full_chains_bits(tier, tmp_path):
    kind, degree, limit = _tiers()[tier]
    src, exe = tmp_path / "c.c", str(tmp_path / "c")
    src.write_text(SRC)
    r = subprocess.run(["gcc", "-O2", "-mfma", "-ffp-contract=off", "-I" + build.CSRC, str(src),
                        "-o", exe, "-lm"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe, kind, str(degree), "%.17g" % limit, "4000000"],
                         capture_output=True, text=True)
    assert out.stdout.strip() == "0", (kind, degree, limit, out.stdout)
