"""Report kernels where their work is split: lab-frame groups with many and with few particles a wave,
a bin of the FP32 store that several workgroups share, and the numbering of its particles."""
import numpy as np
import pytest

import picinputs as pin
from paper_2411_04703_amd import abi

pytestmark = pytest.mark.gpu


def _sim(precision, n_beam, sigma, grid=(32, 32, 64), **plasma):
    from paper_2411_04703_amd.sim import Sim
    w = pin.scaled(pin.workload(1), nx=grid[0], ny=grid[1], nz=grid[2], n_beam=n_beam, sigma=sigma)
    w["plasma"].update(plasma)
    return Sim(w, pin.beam_normals(n_beam, 5), precision=precision, **({} if precision else {"max_steps": 8}))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nz,nu", [(1, 1), (64, 1), (16, 16), (1, 256)])
def test_lab_groups_against_the_beam_read_back(precision, nz, nu):
    """FP64 sums of the same particles in another order: 1e-12 of the sum of magnitudes."""
    s = _sim(precision, 5003, (3, 3, 8))
    s.step(2)
    p, L = s.particles(0), s.beam_lab()
    live = p["alive"] == 1
    z, u = p["z"][live], p["uz"][live]
    z0, dz = z.min() - 1e-3, (z.max() - z.min() + 2e-3) / nz
    u0, du = u.min() - 1e-6, (u.max() - u.min() + 2e-6) / nu
    got = s.lab_groups(z0, dz, nz, u0, du, nu)
    g = (np.floor((z - z0) / dz) * nu + np.floor((u - u0) / du)).astype(int)
    w = p["w"][live]
    q = {k: L[k][live] for k in ("x", "y", "z", "t", "ux", "uy", "gamma")}
    terms = [np.ones_like(w), w, w * q["t"], None, None, w * q["z"], w * q["z"] ** 2, w * q["x"], w * q["x"] ** 2,
             w * q["y"], w * q["y"] ** 2, w * q["ux"], w * q["ux"] ** 2, w * q["uy"], w * q["uy"] ** 2, w * q["gamma"]]
    for k, v in enumerate(terms):
        if v is not None:
            want = np.bincount(g, v, minlength=nz * nu)
            scale = np.bincount(g, np.abs(v), minlength=nz * nu)
            assert np.all(np.abs(got[:, k] - want) <= 1e-12 * scale), k
    for k in range(nz * nu):
        t = q["t"][g == k]
        want = (t.min(), t.max()) if len(t) else (np.inf, -np.inf)
        np.testing.assert_allclose(got[k, 3:5], want, rtol=1e-13)


@pytest.mark.parametrize("n_beam,sigma", [(70001, (.4, .4, .6)), (257, (.4, .4, .6)), (20011, (4, 4, 9)), (0, (1, 1, 1))])
def test_fp32_report_follows_the_fp64_one(n_beam, sigma):
    """At the start both stores hold the same particles, the FP32 one's offsets rounded by 2^-25 of a cell
    and its momenta and weights by 2^-24: the charge's maximum to 1e-6, moments and energies to 1e-6."""
    d = []
    for precision in (0, 1):
        s = _sim(precision, n_beam, sigma)
        d.append(s.diag(abi.PIC_DIAG_MOMENTS | abi.PIC_DIAG_ENERGY | abi.PIC_DIAG_GAUSS))
    a, b = d
    assert a["n_beam"] == b["n_beam"] and a["n_plasma"] == b["n_plasma"]
    for k in ("rho_max", "gauss_max", "kin_beam", "kin_plasma", "wsum"):
        assert b[k] == pytest.approx(a[k], rel=1e-6, abs=1e-7), k
    if n_beam:
        np.testing.assert_allclose(b["sigma"], a["sigma"], rtol=1e-6)
        np.testing.assert_allclose(b["mean"], a["mean"], rtol=1e-6)
