"""16-bit formats at the smallest subnormal: a uniform field of one unit in E_z, B_x
and B_y, with rest weight 1/2 (eps = 2, w0_vac = 0), is an equilibrium whose
populations are whole units (2 at rest; 1, 0, 1, 0 moving), so every step keeps it
exactly.  Halves of the moments themselves would not be whole units."""
import os

import numpy as np
import pytest

from gpu_util import announce
from paper_1108_2651_amd import lbem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f16dev", "bf16dev", "f16ghost", "bf16ghost"])
@pytest.mark.parametrize("fuse", ["1", "4"])
def test_uniform_unit_field_stays(prec, fuse):
    announce(f"subnormal moments {prec} steps per launch {fuse}")
    u = float(np.float32(1e-45))
    nx, ny = 60, 9
    E, B = np.zeros((3, nx * ny)), np.zeros((3, nx * ny))
    E[2], B[0], B[1] = u, u, u
    os.environ["LBEM_FUSE"] = fuse
    try:
        s = lbem.Solver(2, (nx, ny, 1), prec, w0_vac=0.0)
    finally:
        os.environ.pop("LBEM_FUSE")
    s.set_medium(np.full(nx * ny, 2.0))
    s.init_fields(E, B)
    assert s.steps_per_launch == int(fuse)
    for n in (1, 4, 7):
        s.step(n)
        Eg, Bg = s.moments()
        assert np.array_equal(Eg, E) and np.array_equal(Bg, B), (n, Eg[2, :3] / u, Bg[:2, 0] / u)
    s.close()
