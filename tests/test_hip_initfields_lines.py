"""GPU test of the initial beam field on line lengths at the edges of the line transform's dispatch:
several lines a thread group (short lines, an odd number of them left over), one group of four lines
(more points than a workgroup has threads), one line a thread (more than 819 points), and a single
point along y; and on numbers of planes that are no multiple of the eight the solve along z loads
ahead.  Against the oracle with the bar of the initial field's parity test: 1e-11 of the field's norm
(two exact FP64 solvers that sum in different orders)."""
import numpy as np
import pytest

import picinputs as pin
from oracle import pyoracle as po
from test_hip_fp64 import FIELDS, _pair

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_built")]


@pytest.mark.parametrize("nx, ny, nz", [(9, 11, 33), (300, 9, 16), (832, 1, 23), (31, 257, 17)])
def test_line_lengths(nx, ny, nz):
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=400, sigma=(1, 1, 1.5))
    w["plasma"]["n0_lab_cm3"] = 0.0
    w["plasma"]["ions"] = 0
    w["beam"]["charge_C"] = 1e-9
    ref, gpu = _pair(w, init_fields=1)
    po.init_beam_fields(ref)
    assert np.linalg.norm(ref.field("Ex")) > 0
    for f in FIELDS:
        a, b = gpu.field(f), ref.field(f)
        nb = np.linalg.norm(b)
        assert np.linalg.norm(a - b) <= (1e-11 * nb if nb > 0 else 0.0), f
