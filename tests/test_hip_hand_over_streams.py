"""The FP32 to FP64 hand-over between contexts of different streams waits for the source's steps."""
import pytest
import torch

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu


def test_steps_in_flight_are_in_the_hand_over():
    """FP32 runs are bitwise reproducible, so the state handed over while steps are in flight equals
    the one handed over after a wait."""
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=64, ny=64, nz=128, n_beam=200001, sigma=(4, 4, 12))
    nrm = pin.beam_normals(200001, 9)
    out = []
    for wait in (True, False):
        a = Sim(w, nrm, precision=1, record=1, max_steps=34, stream=torch.cuda.Stream())
        b = Sim(w, nrm, precision=0, record=1, max_steps=34, stream=torch.cuda.Stream())
        torch.cuda.synchronize()
        a.step(32)
        if wait:
            a.sync()
        a.export_to(b)
        out.append([b.read(k) for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz")] + [
            b.read(alive) for alive in (abi.PIC_A_BEAM_ALIVE, abi.PIC_A_PLASMA_ALIVE)] + [
            b.read(p) * (b.read(alive) == 1) for p, alive in ((abi.PIC_A_BEAM, abi.PIC_A_BEAM_ALIVE),
                                                              (abi.PIC_A_PLASMA, abi.PIC_A_PLASMA_ALIVE))])
        a.close()
        b.close()
    for x, y in zip(*out):
        assert torch.equal(x, y)
    assert float(out[0][0].abs().max()) > 0
