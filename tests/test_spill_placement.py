"""The compiler's register spills in the FP64 tile kernels.  hipcc has stored vector registers to
scratch at the head of a block, before the instruction that brings back the lanes a branch had
masked off: the masked lanes' values were lost, and a store went to the address one of them held.
The kernels are written so that no such place exists; this reads the assembly of each build for one."""
import os
import re
import subprocess

import pytest

from paper_2411_04703_amd import build


def misplaced(asm):
    found, kernel, head, pending = [], "", False, []
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            kernel = m.group(1)
        if line.startswith(".LBB"):
            head, pending = True, []
            continue
        s = line.split(";")[0].strip()
        if not head or not s or s.startswith("."):
            continue
        if s.startswith("s_or_b64 exec, exec"):
            found += [(kernel, p) for p in pending]
            head = False
        elif re.match(r"s_\w+_saveexec|s_mov_b64 exec|s_andn2_b64 exec|s_and_b64 exec|s_cbranch|s_branch", s):
            head = False
        elif s.startswith("scratch_"):
            pending.append(s)
    return found


def test_the_reader_finds_a_misplaced_spill():
    bad = "_Z1k:\n.LBB0_1:\n\tscratch_store_dwordx2 off, v[0:1], off offset:8\n\ts_or_b64 exec, exec, s[8:9]\n"
    good = "_Z1k:\n.LBB0_1:\n\ts_or_b64 exec, exec, s[8:9]\n\tscratch_store_dwordx2 off, v[0:1], off offset:8\n"
    assert len(misplaced(bad)) == 1 and not misplaced(good)


@pytest.mark.parametrize("src", ["k_tiles64.hip", "k_adjoint.hip"])
def test_no_spill_under_a_partial_mask(src, tmp_path):
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, *build.PER_FILE.get(src, []), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        assert not misplaced(f.read())
