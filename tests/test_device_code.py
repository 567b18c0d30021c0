"""What the compiled device code of this library must not contain, read from the assembly that hipcc writes for its sources
(cross-compiled, no GPU).  A load into LDS takes its LDS address from M0 and may issue one wait state after a scalar write of
M0 at the earliest; the compiler inserts that state between its own instructions but never inside an asm statement."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_26444_amd import build as hipbuild

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def instructions(asm):
    for line in asm.splitlines():
        line = line.split(";")[0].split("//")[0].strip()
        if line and not line.startswith(".") and not line.endswith(":"):
            yield line


def loads_into_lds(asm):
    """(number of loads into LDS, those right behind a scalar write of M0)"""
    loads, early, before = 0, [], ""
    for ins in instructions(asm):
        op = ins.split()[0]
        if re.match(r"(global|buffer|scratch)_load_.*lds", op) or (op.startswith("buffer_load") and ins.endswith(" lds")):
            loads += 1
            if re.match(r"s_\w+\s+m0\b", before):
                early.append((before, ins))
        before = ins
    return loads, early


def assembly(source):
    flags = [f for f in hipbuild.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [HIPCC, *flags, "-I", os.path.join(hipbuild.ROOT, "include"), "-I", hipbuild.CSRC, "--cuda-device-only", "-S", "-o", "-", source]
    return subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300).stdout


def test_the_check_sees_a_missing_wait_state():
    good = "\ts_mov_b32 m0, s5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[2:3]\n"
    assert loads_into_lds(good) == (1, [])
    assert len(loads_into_lds(good.replace("\ts_nop 0\n", "\t;;#ASMSTART\n"))[1]) == 1


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_every_load_into_lds_keeps_its_distance_from_the_write_of_m0():
    total = 0
    for source in sorted(glob.glob(os.path.join(hipbuild.CSRC, "*.hip"))):
        with open(source) as f:
            if "load_lds" not in f.read():
                continue
        loads, early = loads_into_lds(assembly(source))
        assert not early, (os.path.basename(source), len(early), early[:3])
        total += loads
    assert total > 0
