"""Wait states around the inline asm that rescales gradient accumulators (block_kernel.hpp, fp32 passes of one wave per SIMD): the compiler
counts none for it, so those that the matrix instructions need have to stand in the code."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2211_12281_amd import build

TRIPLE = [r"v_accvgpr_read_b32 (v\d+), (a\d+)", r"v_mul_f32(?:_e32|_e64)? (v\d+), (v\d+), v\d+", r"v_accvgpr_write_b32 (a\d+), (v\d+)"]


def _instructions(source):
    r = subprocess.run(["hipcc", *(f for f in build.FLAGS if f != "-fPIC"), "--cuda-device-only", "-S", source, "-o", "-"], cwd=build.CSRC,
                       capture_output=True, text=True, check=True)
    lines = (l.split(";")[0].strip() for l in r.stdout.splitlines())
    return [l for l in lines if l and not l.startswith(".")]


def _rescaling(ins, i):
    m = [re.match(p, t) for p, t in zip(TRIPLE, ins[i:i + 3])]
    return all(m) and m[0][1] == m[1][1] == m[1][2] == m[2][2] and m[0][2] == m[2][1]


def _waits(ins, at, step):
    """Wait states between an instruction and the nearest matrix instruction or end of its straight line of code, in one direction."""
    states = 0
    at += step
    while 0 <= at < len(ins) and not re.match(r"v_mfma|s_c?branch|s_endpgm|.*:$", ins[at]):
        m = re.match(r"s_nop (\d+)", ins[at])
        states += int(m[1]) + 1 if m else 0
        at += step
    return states


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source", ["block_f32_fwd_ls.hip", "block_f32_gradt_ls.hip"])
def test_rescaled_accumulators_have_settled(source):
    ins = _instructions(source)
    at = [i for i in range(len(ins) - 2) if _rescaling(ins, i)]
    assert at                                              # (the kernels are in these files)
    for i in at:
        assert _waits(ins, i, -1) >= 20, ins[i - 4:i + 3]
        assert _waits(ins, i + 2, 1) >= 2, ins[i:i + 6]
