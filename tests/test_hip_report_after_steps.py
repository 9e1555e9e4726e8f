"""The Gauss residual of an FP32 run after odd and even numbers of steps, in an arena that holds what an
earlier owner of its memory left there: the ion profiles alternate from step to step, also in runs
without immobile ions, where no kernel writes them."""
import pytest
import torch

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu


def _empty_of(pattern):
    """torch.empty whose byte tensors (the arena) hold `pattern`."""
    empty = torch.empty

    def filled(*a, **k):
        t = empty(*a, **k)
        return t.fill_(pattern) if t.dtype == torch.uint8 else t
    return filled


@pytest.mark.parametrize("pattern", [0xFF, 0x40])  # as a double: NaN, 32.5
@pytest.mark.parametrize("n0, ions", [(0.0, 0), (1e16, 0), (1e16, 1), (1e16, 2)])
def test_residual_in_a_used_arena(n0, ions, pattern, monkeypatch):
    """Against the same run in an arena of zeros: FP32 states are equal bit for bit, and the charge is
    summed with FP64 atomics in any order, which moves it by round-off of the gross charge (1e-12 of it
    is the bar of the allocation-free reports' test too)."""
    from paper_2411_04703_amd.sim import Sim, derive
    w = pin.scaled(pin.workload(1), nx=16, ny=24, nz=64, n_beam=2003, sigma=(2, 2, 6))
    w["plasma"].update(n0_lab_cm3=n0, ions=ions)
    gross = derive(w)["gamma_R"] * derive(w)["n0_norm"]
    sims = []
    for fill in (0, pattern):
        with monkeypatch.context() as m:
            m.setattr(torch, "empty", _empty_of(fill))
            sims.append(Sim(w, pin.beam_normals(2003, 4), precision=1))
    for n in (1, 2, 1):
        a, b = ([s.step(n), s.diag(abi.PIC_DIAG_GAUSS)][1] for s in sims)
        assert a["rho_max"] > 0
        for k in ("rho_max", "gauss_max", "gauss_drift"):
            assert abs(a[k] - b[k]) <= 1e-12 * max(a["rho_max"], gross), (k, a[k], b[k])
