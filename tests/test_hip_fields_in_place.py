"""GPU test of the FP32 field update in place (grids of more than 2^27 cells, which hold one set of
fields): B, E with the Mur faces, and the plane that enters when the window shifts, against the FP64
path of the same grid from the same fields (exact in FP32), without particles.

Each step rounds every updated value a few times (at most 8 FP32 operations per Yee component,
relative error 2^-24 each), so after n steps the bar is n x 16 x 2^-24 of the array's norm; the two
planes at each face are held to it by themselves."""
import numpy as np
import pytest
import torch

import picinputs as pin

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz")
STEPS = 5


@pytest.mark.parametrize("beta", [0.98, 0.0])
def test_large_grid_matches_fp64(beta):
    from paper_2411_04703_amd.sim import Sim
    nx, ny, nz = 512, 512, 520
    assert nx * ny * nz > 1 << 27
    w = pin.scaled(pin.workload(1), nx=nx, ny=ny, nz=nz, n_beam=0)
    w["plasma"]["n0_lab_cm3"] = 0.0
    w["plasma"]["ions"] = 0
    w["frame"]["window_beta"] = beta
    block = np.random.default_rng(5).standard_normal((1 << 20) + 7).astype(np.float32).astype(np.float64)
    out = {}
    for precision in (0, 1):
        s = Sim(w, np.zeros((6, 0)), precision=precision, **({"max_steps": 8} if precision == 0 else {}))
        for k, f in enumerate(FIELDS):
            s.write(f, np.resize(np.roll(block, 1000 * k), nx * ny * nz))
        s.step(STEPS)
        out[precision] = [s.read(f).view(nz, ny, nx).to(torch.float32 if precision else torch.float64).cpu()
                          for f in FIELDS]
        del s
        torch.cuda.empty_cache()
    for k, f in enumerate(FIELDS):
        a, b = out[1][k].double(), out[0][k]
        tol = STEPS * 16 * 2.0 ** -24
        assert float((a - b).norm()) <= tol * float(b.norm()), f
        for p in (slice(0, 2), slice(nz - 2, nz)):
            assert float((a[p] - b[p]).norm()) <= tol * max(float(b[p].norm()), float(b[2:4].norm())), (f, p)
