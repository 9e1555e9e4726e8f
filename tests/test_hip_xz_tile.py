"""GPU tests of the FP32 step on an x-z tile, where its boxes hold the grid's one row along y:
grids one tile wide, whose halo columns are the tile's own cells, one tile long, and with an odd
number of tiles.

The current is a sum of integers, so the deposit that adds a window's rows up first gives the
bits of the one that adds each node (variant 1).  Against FP64 the bar is that of the FP32 path:
1e-4 of the whole field's magnitude (FP32 rounding of the update, 2^-f quantisation of the current)."""
import math

import numpy as np
import pytest

import picinputs as pin

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz")


@pytest.mark.parametrize("nx, nz, steps", [(16, 16, 4), (16, 48, 9), (48, 80, 12)])
def test_one_row_boxes(nx, nz, steps):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=nx, ny=1, nz=nz, n_beam=3001, sigma=(2, 1, 2))
    w["beam"]["charge_C"] = 3e-10
    nrm = pin.beam_normals(w["beam"]["n_macro"], 3)
    runs = []
    for variant in (0, 1):
        s = Sim(w, nrm, precision=1, variant=variant)
        s.step(steps)
        runs.append({f: s.field(f) for f in FIELDS})
    s = Sim(w, nrm, precision=0)
    s.step(steps)
    want = {f: s.field(f) for f in FIELDS}
    total = math.sqrt(sum(np.linalg.norm(v) ** 2 for v in want.values()))
    assert total > 0
    for f in FIELDS:
        assert np.array_equal(runs[0][f], runs[1][f]), f
        assert np.linalg.norm(runs[0][f] - want[f]) <= 1e-4 * total, f
