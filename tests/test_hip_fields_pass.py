"""GPU tests of the FP32 field update in one pass (B, E, Mur faces and shift from one set of fields
into the other) on grids whose planes are not whole workgroups, on one row along y, and where a
plane is less than one workgroup.

Against the oracle, without particles: each step rounds every updated value a few times (at most 8
FP32 operations per Yee component, relative error 2^-24 each, on values whose size the update keeps
to the field's scale), so after n steps the bar is n x 16 x 2^-24 of the array's norm."""
import numpy as np
import pytest

import picinputs as pin
from oracle import pyoracle as po

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_built")]

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz")


@pytest.mark.parametrize("beta", [0.98, 0.0])
@pytest.mark.parametrize("nx, ny, nz, steps", [(24, 40, 32, 21), (8, 16, 48, 12), (48, 1, 112, 17), (56, 24, 36, 5)])
def test_one_pass_matches_oracle(nx, ny, nz, steps, beta):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=0)
    w["plasma"]["n0_lab_cm3"] = 0.0
    w["plasma"]["ions"] = 0
    w["frame"]["window_beta"] = beta
    nrm = np.zeros((6, 0))
    ref, gpu = po.Sim(w, nrm), Sim(w, nrm, precision=1)
    rng = np.random.default_rng(12)
    for f in FIELDS:
        a = rng.standard_normal((nz, ny, nx)).astype(np.float32).astype(np.float64)
        ref.field(f)[...] = a
        gpu.write(f, a)
    ref.step(steps)
    gpu.step(steps)
    assert gpu.diag()["k0"] == ref.info().k0 > (0 if beta > 0 else -1)
    for f in FIELDS:
        a, b = gpu.field(f), ref.field(f)
        assert np.linalg.norm(a - b) <= steps * 16 * 2.0 ** -24 * np.linalg.norm(b), f
