"""Work items of the FP32 step by the workgroups that take them: with one workgroup a CU an x-z run gets
items for 256 of them, not for 512 (fewer, larger items: a smaller arena)."""
import picinputs as pin
from paper_2411_04703_amd import abi
from paper_2411_04703_amd.sim import query_layout


def _arena(w, wg):
    return query_layout(w, precision=abi.PIC_FP32_SPLIT, wg_per_cu=wg).arena_bytes


def test_items_follow_the_grid_of_the_step():
    xz = pin.scaled(pin.workload(1), nx=256, ny=1, nz=512, n_beam=1000000, sigma=(4, 1, 16))
    xz["plasma"]["n0_lab_cm3"] = 0.0
    assert _arena(xz, 1) < _arena(xz, 0)
    assert _arena(xz, 2) == _arena(xz, 8) == _arena(xz, 0)
    box = pin.scaled(pin.workload(1), nx=64, ny=64, nz=128, n_beam=1000000, sigma=(4, 4, 16))
    assert _arena(box, 1) == _arena(box, 2) == _arena(box, 0)
