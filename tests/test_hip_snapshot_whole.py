"""A snapshot holds the whole state: saved into a buffer on 16 bytes (one launch) and off them (piece by
piece) it is the same bytes, and either restores every field and particle of a run that has gone on,
or of another run of the same configuration, as they were, bit for bit."""
import numpy as np
import pytest
import torch

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz")
PARTICLES = (abi.PIC_A_BEAM, abi.PIC_A_BEAM_ALIVE, abi.PIC_A_PLASMA, abi.PIC_A_PLASMA_ALIVE)


def _run(grid, precision, record, seed):
    """A run three steps after random fields on every plane, so that any cell differs between steps."""
    from paper_2411_04703_amd.sim import Sim
    nx, ny, nz = grid
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=1003, sigma=(1, 1, 3))
    w["frame"]["window_beta"] = 0.9
    s = Sim(w, pin.beam_normals(1003, seed), precision=precision, **({"record": 1, "max_steps": 16} if record else {}))
    r = np.random.default_rng(seed)
    for f in FIELDS:
        s.write(f, 1e-3 * r.standard_normal(nx * ny * nz))
    s.step(3)
    return s


def _all(s):
    return [s.read(k) for k in FIELDS + PARTICLES]


# cell counts that are multiples of 32 and not: 15 over, and 27 (there a block of E and B takes the room of its six arrays)
@pytest.mark.parametrize("precision, record, grid", [(0, 1, (9, 11, 37)), (0, 0, (9, 11, 41)), (0, 0, (8, 8, 32)),
                                                     (1, 0, (24, 40, 32)), (1, 1, (16, 16, 40))])
def test_both_ways_hold_and_restore_everything(precision, record, grid):
    s = _run(grid, precision, record, 1)
    n = int(s.layout.state_bytes)
    a = torch.full((n,), 0x55, dtype=torch.uint8, device="cuda")
    b = torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda")[4:4 + n]
    s.get_state(a)
    s.get_state(b)
    gap = (a == 0x55) & (b == 0xAA)  # what neither wrote: the ends of the 256-byte blocks
    assert torch.equal(a[~gap], b[~gap])
    assert int(gap.sum()) < 256 * 11 and not bool(gap[:96].any())
    want = _all(s)
    other = _run(grid, precision, record, 2)
    for run in (s, other):
        for snap in (a, b):
            run.step(2)
            now = _all(run)
            assert not any(torch.equal(x, y) for x, y in zip(now[:6], want[:6]))
            run.set_state(snap)
            for k, x, y in zip(FIELDS + PARTICLES, _all(run), want):
                assert torch.equal(x, y), k
            again = run.get_state(torch.full_like(a, 0x55))
            assert torch.equal(again, a)


def test_earlier_layout_is_refused():
    s = _run((9, 11, 41), 0, 0, 1)
    a = s.get_state()
    a[0] -= 1
    with pytest.raises(abi.PicError) as e:
        s.set_state(a)
    assert e.value.status == abi.PIC_ESTATE


@pytest.mark.usefixtures("oracle_built")
def test_gradient_over_checkpoints_on_a_ragged_grid():
    """bunching_grad, whose backward pass restores checkpoints, against the oracle's adjoint, at the bar
    of the reverse steps by themselves (1e-9)."""
    from oracle import pyoracle as po
    from paper_2411_04703_amd.autograd import bunching_grad
    w = pin.scaled(pin.adjoint_subcase(), nx=9, ny=11, nz=37, n_beam=700, sigma=(1, 1.5, 4))
    w["beam"]["charge_C"] = 3e-9
    w["undulator"]["z_start_lab_m"] = w["frame"]["gamma_boost"] * 10 * w["grid"]["dx_m"]
    w["undulator"]["entrance_ramp_periods"] = 0.5
    nrm = pin.beam_normals(700, 2)
    w["frame"]["window_beta"] = po.Sim(w, nrm).info().bw
    L, gK, gn = po.grad_bunching(w, nrm, 12, 2 * np.pi / 20.0)
    loss, hK, hn = bunching_grad(w, nrm, 12, every=5)
    assert loss == pytest.approx(L, rel=1e-11)
    assert hK == pytest.approx(gK, rel=1e-9)
    assert hn == pytest.approx(gn, rel=1e-9)
