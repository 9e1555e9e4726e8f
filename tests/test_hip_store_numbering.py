"""The FP32 store read, summed and grouped on both sides of the rules that number it: bins that one block
goes through and more, beams that are grouped without numbering and one particle past that."""
import numpy as np
import pytest

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,tile,n_beam,sigma", [
    ((64, 64, 1056), (8, 8, 4), 9001, (9, 9, 200)),     # 16896 bins, a block past one's share: a wide beam
    ((64, 64, 1056), (8, 8, 4), 40009, (.4, .4, .6)),   # a crowded one
    ((64, 64, 1024), (8, 8, 4), 5003, (9, 9, 200)),     # 16384 bins: one block's share
    ((32, 32, 64), (16, 8, 8), 8192, (3, 3, 8)),        # the largest beam that is not numbered for its groups
    ((32, 32, 64), (16, 8, 8), 8193, (3, 3, 8)),
    ((16, 1, 64), (16, 1, 16), 3, (1, 1, 4)),           # most waves without a particle
], ids=lambda v: str(v).replace(" ", ""))
def test_store_read_and_grouped(grid, tile, n_beam, sigma):
    """At the start both modes hold the same particles, the FP32 one's offsets rounded by 2^-25 of a cell and
    its momenta by 2^-24 of themselves: in the order of z (bins have their own), z to 1e-6 and the sums of
    the groups, taken from the same store in another order, to 1e-12 of their terms' magnitudes."""
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=grid[0], ny=grid[1], nz=grid[2], n_beam=n_beam, sigma=sigma)
    w["plasma"]["n0_lab_cm3"] = 0.0
    nrm = pin.beam_normals(n_beam, 5)
    s, ref = Sim(w, nrm, precision=1, tile=tile), Sim(w, nrm, precision=0)
    p, q, L = s.particles(0), ref.particles(0), s.beam_lab()
    live = q["alive"] == 1
    assert len(p["z"]) == live.sum() == s.diag(abi.PIC_DIAG_MOMENTS)["n_beam"]
    np.testing.assert_allclose(np.sort(p["z"]), np.sort(q["z"][live]), rtol=0, atol=1e-6)
    np.testing.assert_allclose(s.diag(abi.PIC_DIAG_MOMENTS)["mean"], ref.diag(abi.PIC_DIAG_MOMENTS)["mean"], rtol=0, atol=1e-6)
    for nz, nu in ((64, 1), (5, 3)):
        z, u = p["z"], p["uz"]
        z0, dz = z.min() - 1e-3, (z.max() - z.min() + 2e-3) / nz
        u0, du = u.min() - 1e-6, (u.max() - u.min() + 2e-6) / nu
        got = s.lab_groups(z0, dz, nz, u0, du, nu)
        g = (np.floor((z - z0) / dz) * nu + np.floor((u - u0) / du)).astype(int)
        for k, v in ((0, np.ones_like(z)), (1, p["w"]), (5, p["w"] * L["z"]), (8, p["w"] * L["x"] ** 2),
                     (15, p["w"] * L["gamma"])):
            want, scale = (np.bincount(g, x, minlength=nz * nu) for x in (v, np.abs(v)))
            assert np.all(np.abs(got[:, k] - want) <= 1e-12 * scale), k
        for k in range(nz * nu):
            t = L["t"][g == k]
            np.testing.assert_allclose(got[k, 3:5], (t.min(), t.max()) if len(t) else (np.inf, -np.inf), rtol=1e-13)
