"""GPU test of snapshots: saved into buffers on 16 bytes (one launch) and off them (piece by piece),
in both precisions, with and without particle ids, on sizes whose pieces are not whole 16-byte words;
both give the same bytes of state and restore to the same run, bit for bit in FP32."""
import numpy as np
import pytest
import torch

import picinputs as pin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision, record, grid", [(1, 0, (24, 40, 32)), (1, 1, (16, 16, 40)), (0, 1, (9, 11, 37)),
                                                     (0, 0, (8, 8, 32))])
def test_snapshot_on_any_alignment(precision, record, grid):
    from paper_2411_04703_amd.sim import Sim
    nx, ny, nz = grid
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=1003, sigma=(1, 1, 3))
    opts = {"record": 1, "max_steps": 16} if record else {}
    s = Sim(w, pin.beam_normals(1003, 1), precision=precision, **opts)
    s.step(3)
    a = s.get_state()
    n = a.numel()
    raw = torch.zeros(n + 16, dtype=torch.uint8, device="cuda")
    b = raw[4:4 + n]
    s.get_state(b)
    outs = []
    for st in (a, b):
        s.set_state(st)
        again = s.get_state(torch.zeros_like(a))
        s.set_state(st)
        s.step(4)
        outs.append((again, [s.read(f) for f in ("Ex", "Ez", "By")]))
    # the header is followed by what nobody writes, up to 256 bytes
    assert torch.equal(outs[0][0][:96], a[:96])
    for x, y in zip(outs[0][1], outs[1][1]):
        if precision == 1:
            assert torch.equal(x, y)
        else:  # FP64 sums are taken in any order
            assert float((x - y).norm()) <= 1e-9 * float(y.norm())
    assert np.isfinite(float(outs[0][1][0].abs().max()))
    assert torch.equal(outs[0][0], outs[1][0])
