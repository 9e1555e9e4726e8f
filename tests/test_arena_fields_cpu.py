"""What the FP32 mode's second set of fields (24 bytes a cell) adds to the arena: nothing in a recorded run,
whose adjoint scratch (48 bytes a cell) the FP64 mode alone uses, nor where the staging of the beam's
normals (48 bytes a particle) holds it."""
import picinputs as pin
from paper_2411_04703_amd import abi
from paper_2411_04703_amd.sim import query_layout


def _arena(nz, n_beam, **opts):
    w = pin.scaled(pin.workload(1), nx=32, ny=32, nz=nz, n_beam=n_beam, sigma=(2, 2, 8))
    w["plasma"]["n0_lab_cm3"] = 0.0
    return query_layout(w, precision=abi.PIC_FP32_SPLIT, **opts).arena_bytes


def test_fields_of_the_next_step():
    """Per cell: E and B 24 bytes, the currents 24, the previous residual 8, 32 slots of slack in each of four
    buffers a bin of 1024 cells 4, partial sums 1 where the cells are the most: 61, and 24 for the second set;
    a recorded run has 48 for the adjoint and half a byte of ids."""
    cells = 32 * 32 * 256
    own, record, staging = [(_arena(512, n, **o) - _arena(256, n, **o)) / cells
                            for n, o in ((1000, {}), (1000, {"record": 1}), (1 << 20, {}))]
    assert 84 < own < 87
    assert 108 < record < 111
    assert 59 < staging < 62
