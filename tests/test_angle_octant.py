"""The direct-sum kernels' arctangent without octant reduction (no GPU needed).

Where every tangent t = |Y| / X of a wave is below a limit near 1, the kernels
leave the octant reduction out; both forms give the same bits only if
|Y| <= X.  t comes from a hardware reciprocal that may be one unit in the last
place off (FP64: an estimate refined by two Newton steps and a residual), so |Y|
just above X must not give a t below the limit.  The test evaluates t for Y at X
and the next values above it, over random X and every reciprocal within that
error, with the limits read from the kernel source."""
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
#include <string.h>
static uint64_t s0 = 88172645463325252ull;
static uint64_t rnd(void) { s0 ^= s0 << 13; s0 ^= s0 >> 7; s0 ^= s0 << 17; return s0; }
int main(int c, char** v) {  /* f32 or f64, limit (FP64: upper word), count */
  const long n = atol(v[3]);
  long bad = 0, low = 0;  /* low: below 1 with |Y| > X */
  if (v[1][1] == '3') {
    const float lim = (float)atof(v[2]);
    for (long k = 0; k < n; ++k) {
      const uint32_t b = 0x3f800000u | (uint32_t)(rnd() & 0x7fffff);
      float x, y;
      memcpy(&x, &b, 4);
      y = x;
      const double r = 1.0 / (double)x;
      for (int up = 0; up < 4; ++up) {
        float i = (float)r;
        for (int d = -1; d <= 1; ++d) {
          const float j = d < 0 ? nextafterf(i, 0.0f) : d ? nextafterf(i, 2.0f) : i;
          const double ulp = (double)nextafterf((float)r, 2.0f) - (double)(float)r;
          if (fabs((double)j - r) > ulp) continue;  /* within one place of 1 / x */
          const float t = y * j;
          if (y > x) { low += t < 1.0f; bad += t < lim; }
        }
        y = nextafterf(y, 4.0f);
      }
    }
  } else {
    const uint32_t lim = (uint32_t)strtoul(v[2], 0, 16);
    for (long k = 0; k < n; ++k) {
      const uint64_t b = 0x3ff0000000000000ull | (rnd() & 0xfffffffffffffull);
      double x, y;
      memcpy(&x, &b, 8);
      y = x;
      for (int up = 0; up < 4; ++up) {
        double i = 1.0 / x * (1.0 + 0x1p-23 * ((double)(rnd() >> 11) * 0x1p-52 - 1.0));
        i = fma(i, fma(-x, i, 1.0), i);
        i = fma(i, fma(-x, i, 1.0), i);
        const double q = y * i, t = fma(fma(-x, q, y), i, q);
        uint64_t w;
        memcpy(&w, &t, 8);
        if (y > x) { low += t < 1.0; bad += (uint32_t)(w >> 32) < lim; }
        y = nextafter(y, 4.0);
      }
    }
  }
  printf("%ld %ld\\n", bad, low);
  return 0;
}
"""


def _limits():
    s = open(os.path.join(build.CSRC, "lk_ds.hip")).read()
    f32 = s[s.index("struct SmallAngle<float>"):s.index("struct SmallAngle<double>")]
    f64 = s[s.index("struct SmallAngle<double>"):]
    return {"f32": re.search(r"\boctant = ([0-9.]+)f;", f32).group(1),
            "f64": re.search(r"\boctant = (0x\w+?)u;", f64).group(1)}


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")
@pytest.mark.parametrize("kind", ["f32", "f64"])
def test_no_tangent_above_one_passes_the_limit(kind, tmp_path):
    src, exe = tmp_path / "c.c", str(tmp_path / "c")
    src.write_text(SRC)
    r = subprocess.run(["gcc", "-O2", "-mfma", "-ffp-contract=off", str(src), "-o", exe, "-lm"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    limit = _limits()[kind]
    out = subprocess.run([exe, kind, limit, "3000000"], capture_output=True, text=True).stdout
    bad, low = map(int, out.split())
    print("%s: limit %s, %d tangents of |Y| > X below 1, %d below the limit" % (kind, limit, low, bad))
    assert bad == 0
