"""Properties of the compiled device code that the solvers rely on, checked on
the host: wait states around wave masks in hand-written instructions, and
kernels free of scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import msgpack
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


def _sections(elf):
    """(name, type, file offset, size) of the sections of a 64-bit ELF image."""
    shoff = struct.unpack_from("<Q", elf, 0x28)[0]
    size, count, names = struct.unpack_from("<HHH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQ", elf, shoff + i * size) for i in range(count)]
    strings = heads[names][4]
    return [(elf[strings + h[0]:elf.index(b"\0", strings + h[0])].decode(), h[1], h[4], h[5])
            for h in heads]


def _kernels(lib):
    """The compiler's records of the gfx950 kernels in a built library: the
    AMDGPU metadata notes of the code objects in its offload bundles."""
    fat = next(lib[o:o + n] for name, _, o, n in _sections(lib) if name == ".hip_fatbin")
    kernels, at = {}, 0
    while (at := fat.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", fat, at + 24)[0]):
            off, size, length = struct.unpack_from("<QQQ", fat, entry)
            triple = fat[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" not in triple or size == 0:
                continue
            code = fat[at + off:at + off + size]
            for _, kind, pos, n in _sections(code):
                end = pos + n
                while kind == 7 and pos < end:  # SHT_NOTE
                    namesz, descsz, note = struct.unpack_from("<III", code, pos)
                    desc = pos + 12 + (namesz + 3 & ~3)
                    pos = desc + (descsz + 3 & ~3)
                    if note == 32:  # NT_AMDGPU_METADATA
                        for k in msgpack.unpackb(code[desc:desc + descsz])["amdhsa.kernels"]:
                            kernels[k[".name"]] = k
        at += 24
    return kernels


def test_solver_kernels_have_no_scratch():
    """No kernel uses scratch memory: a spilling build of the sizes 1..16
    ragged kernel returned wrong, varying solutions, and any spill costs up to
    half the speed. The 8-lane Newton form, which no table chooses, is known
    to spill."""
    from paper_2609_15217_amd import build
    if not os.path.exists(build.LIB):
        build.build(verbose=False)
    kernels = _kernels(open(build.LIB, "rb").read())
    names = " ".join(kernels)
    for must in ("k_threadILi13E", "k_segILi32ELi16E", "k_seg_soaILi24ELi8E", "k_lanesILi32E",
                 "k_lanes_soaILi32E", "k_ragged_c0", "k_ragged_c1", "k_ragged_c2", "k_ragged_oneILi16E",
                 "k_grouped_c0", "k_grouped_c1", "k_grouped_c2", "k_newtonILi13E"):
        assert must in names, must
    scratch = {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
               if k[".private_segment_fixed_size"] or k[".uses_dynamic_stack"]}
    assert all("k_newton_lanesILi13ELi8E" in n for n in scratch), scratch
