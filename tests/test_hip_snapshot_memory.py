"""Snapshots in memory that the copy kernel of the context's GPU does not reach by itself (host memory here,
pinned and not; another GPU's memory takes the same way): the same bytes, and they restore."""
import pytest
import torch

import picinputs as pin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_host_memory_holds_a_snapshot(precision, pinned):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=8, ny=16, nz=32, n_beam=507, sigma=(1, 2, 3))
    s = Sim(w, pin.beam_normals(507, 8), precision=precision)
    s.step(2)
    n = int(s.layout.state_bytes)
    dev = s.get_state(torch.zeros(n, dtype=torch.uint8, device="cuda"))
    host = s.get_state(torch.zeros(n, dtype=torch.uint8, pin_memory=pinned))
    assert torch.equal(host, dev.cpu())
    want = s.read("Ex")
    s.step(2)
    assert not torch.equal(s.read("Ex"), want)
    s.set_state(host)
    assert torch.equal(s.read("Ex"), want)
    assert torch.equal(s.get_state(torch.zeros_like(dev)), dev)
