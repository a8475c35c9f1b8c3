"""Properties of the compiled device code that the solvers rely on, checked on
the host: wait states around wave masks in hand-written instructions."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MASK_KERNEL = r"""
#include <hip/hip_runtime.h>
#include "lupp_segments.h"
extern "C" __global__ void mask_reader(const double *a, int *o, double *q)
{
    const int i = threadIdx.x;
    double x = a[i], z = a[i + 64];
    int p = o[i];
    const double xs = a[i + 128], zs = a[i + 192];
    lupp::mask_select(__ballot(a[i + 256] > 0.5), x, xs, z, zs, p, i);
    q[i] = x;
    q[i + 64] = z;
    o[i] = p;
}
"""


def test_selects_wait_for_the_mask(tmp_path):
    """gfx950 needs two wait states between a vector compare that writes a
    mask and a vector instruction that reads it; inside asm nothing but the
    asm itself keeps them."""
    from paper_2609_15217_amd import build
    if not os.path.exists(build.HIPCC) and shutil.which(build.HIPCC) is None:
        pytest.skip("hipcc not found")
    src = tmp_path / "mask.hip"
    src.write_text(MASK_KERNEL)
    asm = subprocess.run([build.HIPCC, *build.CXXFLAGS, "--cuda-device-only", "-S", str(src), "-o", "-"],
                         capture_output=True, text=True, check=True).stdout
    body = [l.split(";")[0].strip() for l in asm.split("mask_reader:")[1].split("s_endpgm")[0].splitlines()]
    body = [l for l in body if l and not l.startswith(".") and not l.endswith(":")]
    selects = 0
    for at, line in enumerate(body):
        m = re.match(r"v_cndmask_b32_e64 .*, (s\[\d+:\d+\]|vcc)$", line)
        if m is None:
            continue
        selects += 1
        states = 0
        for prev in reversed(body[:at]):
            if prev.startswith("v_cmp") and prev.split()[1].rstrip(",") == m.group(1):
                break
            nop = re.match(r"s_nop (\d+)$", prev)
            # s_waitcnt may pass at once: not counted
            states += int(nop.group(1)) + 1 if nop else (0 if prev.startswith("s_waitcnt") else 1)
        else:
            pytest.fail(f"no writer of the mask of: {line}")
        assert states >= 2, (line, states)
    assert selects == 5
