"""The ticket of the preparation in pieces (no GPU needed).

The workgroup that takes the last ticket joins the pieces; the ticket lives in
memory that later calls use again, so it has to be 0 after every whole number of
launches, whatever order their workgroups came in.  An atomic increment that
wraps at the last workgroup is; a count that the last workgroup stores back to 0
is not if two launches (of calls that overlap against the rules) mix: their
increments pass the last workgroup's number, and every later call joins too
early.  The check compiles the kernel and looks for the wrapping atomic."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2106_12655_amd import build

HIPCC = build._hipcc()


def test_a_wrapping_ticket_ends_at_zero_after_mixed_launches():
    groups = 128
    wrap = lambda t: 0 if t >= groups - 1 else t + 1
    for launches in (1, 2, 3):
        t, last = 0, 0
        for _ in range(launches * groups):
            last += t == groups - 1
            t = wrap(t)
        assert t == 0 and last == launches


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC),
                    reason="hipcc not available")
def test_the_kernel_takes_a_wrapping_ticket(tmp_path):
    out = str(tmp_path / "lk_aux.s")
    r = subprocess.run([HIPCC, *build.HIPFLAGS, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "lk_aux.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    bodies = re.findall(r"^(_Z\w*prep_plan_k\w*):(.*?)^\.Lfunc_end", open(out).read(), re.S | re.M)
    assert len(bodies) == 2, [n for n, _ in bodies]
    for name, body in bodies:
        assert len(re.findall(r"global_atomic_inc\b", body)) == 1, name
