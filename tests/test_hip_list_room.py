"""FP64 particle lists in each place that may hold them: the buffer of the next compaction (which moves with
every compaction), the staging of the beam's normals, and room of their own.  Against the oracle at the
FP64 path's bar, with reports (which list the particles too) between the steps."""
import pytest

import picinputs as pin
from paper_2411_04703_amd import abi
from test_hip_fp64 import _compare, _pair

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_built")]


@pytest.mark.parametrize("n_beam,n0,opts", [
    (3001, 1e16, {"check_every": 2}),            # compaction's buffer, swapped every other step
    (0, 1e16, {"check_every": 3}),
    (5, 0.0, {}),                                # five particles: the staging is too small for their lists
    (3001, 0.0, {"check_every": 2}),             # staging
    (60001, 1e16, {"record": 1}),                # staging, a beam of more particles than the plasma
    (3001, 1e16, {"record": 1}),                 # their own
], ids=lambda v: str(v).replace(" ", ""))
def test_lists_in_every_place(n_beam, n0, opts):
    w = pin.scaled(pin.workload(1), nx=9, ny=12, nz=40, n_beam=n_beam, sigma=(1, 1.5, 4))
    w["plasma"]["n0_lab_cm3"] = n0
    w["beam"]["charge_C"] = 3e-10
    if not n_beam:
        w["frame"]["window_beta"] = 0.9
    ref, gpu = _pair(w, max_steps=16, **opts)
    for n in range(1, 8):
        ref.step(1)
        gpu.step(1)
        gpu.diag(abi.PIC_DIAG_GAUSS)
        _compare(ref, gpu, 1e-12 * n, f"step {n}")
