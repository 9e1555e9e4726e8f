"""The check of test_spill_placement on every other source of the library: its kernels are built under
register caps too."""
import os
import subprocess

import pytest

from paper_2411_04703_amd import build
from test_spill_placement import misplaced


@pytest.mark.parametrize("src", [s for s in build.SOURCES if s not in ("k_tiles64.hip", "k_adjoint.hip")])
def test_no_spill_under_a_partial_mask(src, tmp_path):
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, *build.PER_FILE.get(src, []), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        assert not misplaced(f.read())
