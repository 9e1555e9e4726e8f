"""FP64 runs on grids of more tiles than one block of the list's scan goes through: a step from zero fields
moves every particle once, straight on, and deposits each one's whole current."""
import numpy as np
import pytest

import picinputs as pin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,n_beam,sigma", [
    (130, 131, 260, 20011, (40, 40, 60)),    # 17 x 17 x 65 tiles: the last block is not full
    (130, 131, 260, 20011, (.5, .5, .7)),    # nearly all in one tile
    (2000, 1, 1100, 5003, (400, 1, 200)),    # two-dimensional tiles
    (64, 64, 1025, 3001, (20, 20, 300)),     # one tile layer past a whole block
], ids=lambda v: str(v).replace(" ", ""))
def test_every_particle_is_listed_once(nx, ny, nz, n_beam, sigma):
    """A straight move rounds by two units in the last place of the coordinate.  With E = 0 before, the sum
    of E_c over the grid afterwards is that of w dX_c (Esirkepov's currents add up to the move): off per
    particle by the rounding of its coordinate (2^-52 of at most 2048 cells: 4.6e-13) and of at most 144
    contributions (1e-14), so 1e-12 w; a particle lost or listed twice changes E_z's sum by some 0.4 w."""
    from paper_2411_04703_amd.sim import Sim, derive
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=n_beam, sigma=sigma)
    w["plasma"]["n0_lab_cm3"] = 0.0
    w["frame"]["window_beta"] = 0.9
    d = derive(w)
    s = Sim(w, pin.beam_normals(n_beam, 3), precision=0)
    a = s.particles(0)
    s.step(1)
    b = s.particles(0)
    live = a["alive"] == 1
    assert live.sum() > 0.5 * n_beam
    g = np.sqrt(1.0 + a["ux"] ** 2 + a["uy"] ** 2 + a["uz"] ** 2)
    for k, n, f in (("x", nx, "Ex"), ("y", ny, "Ey"), ("z", 0, "Ez")):
        move = d["dt"] * a["u" + k] / g
        to = a[k] + move
        if n:
            to = np.where(to < 0, to + n, np.where(to >= n, to - n, to))
        assert np.all(np.abs(b[k] - to)[live] <= 2.0 ** -51 * np.maximum(np.abs(a[k]), max(n, 1))[live])
        total = float(np.sum(move[live]) * d["w_beam"])
        assert abs(float(s.field(f).sum()) - total) <= 1e-12 * n_beam * d["w_beam"], k
    assert abs(np.sum(move[live])) > 0.3 * live.sum()
