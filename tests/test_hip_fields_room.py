"""The FP32 mode's second set of fields in each place that may hold it: room of its own (a small beam), the
staging of the beam's normals, and the adjoint's scratch of a recorded run.  Runs of one beam are equal
bit for bit wherever it lies, after odd and even numbers of steps, a report and a restore."""
import pytest
import torch

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz")


@pytest.mark.parametrize("n_beam", [4095, 4096])  # 16 x 16 x 32 cells: staging from 4096 particles on
def test_runs_are_equal(n_beam):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=16, ny=16, nz=32, n_beam=n_beam, sigma=(2, 2, 3))
    w["beam"]["charge_C"] = 3e-10
    w["frame"]["window_beta"] = 0.9
    out = []
    for opts in ({}, {"record": 1, "max_steps": 40}):
        s = Sim(w, pin.beam_normals(n_beam, 2), precision=1, **opts)
        got = []
        for n in (1, 2, 3, 1):
            s.step(n)
            s.diag(abi.PIC_DIAG_GAUSS)
            got += [s.read(f) for f in FIELDS]
        snap = s.get_state()
        s.step(2)
        late = [s.read(f) for f in FIELDS]
        s.set_state(snap)
        s.step(2)
        for x, y in zip(late, [s.read(f) for f in FIELDS]):
            assert torch.equal(x, y)
        out.append(got + late)
    for x, y in zip(*out):
        assert torch.equal(x, y)
    assert float(out[0][-1].abs().max()) > 0
