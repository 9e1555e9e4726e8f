"""FP64 runs with particles that a caller wrote outside the window: a report and a reverse step leave
every particle as it is, a step takes those out."""
import numpy as np
import pytest
import torch

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [16, 1])  # tiles of both kinds
def test_only_a_step_takes_particles_out(ny):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=16, ny=ny, nz=48, n_beam=501, sigma=(2, 2, 5))
    w["frame"]["window_beta"] = 0.9
    s = Sim(w, pin.beam_normals(501, 6), precision=0, record=1, max_steps=8)
    s.step(1)
    kept = s.diag(abi.PIC_DIAG_GAUSS)["n_beam"]
    p = s.read(abi.PIC_A_BEAM).cpu().numpy()
    live = np.flatnonzero(s.read(abi.PIC_A_BEAM_ALIVE).cpu().numpy())
    p[2, live[3]], p[2, live[7]] = -40.0, 1e4  # below and above every plane of the window
    s.write(abi.PIC_A_BEAM, p)
    before = [s.read(k) for k in (abi.PIC_A_BEAM, abi.PIC_A_BEAM_ALIVE, abi.PIC_A_PLASMA_ALIVE)]
    s.diag(abi.PIC_DIAG_MOMENTS | abi.PIC_DIAG_GAUSS)
    lam = torch.zeros(s.lambda_len(), dtype=torch.float64, device="cuda")
    lam[:6 * 501] = 1.0
    s.adjoint_step(lam, np.zeros(2))
    after = [s.read(k) for k in (abi.PIC_A_BEAM, abi.PIC_A_BEAM_ALIVE, abi.PIC_A_PLASMA_ALIVE)]
    for x, y in zip(before, after):
        assert torch.equal(x, y)
    assert s.diag(0)["n_beam"] == kept
    out = lam[:6 * 501].view(6, 501)
    assert not bool(out[:, [live[3], live[7]]].any()) and bool(out[:, live[5]].any())  # no adjoint through the step
    s.step(1)
    s.sync()  # no error flag
    assert not bool(s.read(abi.PIC_A_BEAM_ALIVE)[[live[3], live[7]]].any())
    assert s.diag(0)["n_beam"] <= kept - 2
