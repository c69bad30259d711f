"""Device memory of a dispersion pole in 3D FP32: coefficients (12 B per cell), P and J
(24 B) and, where launches of two steps use it, a second P and J.  With walls every
launch is a single step and the second copy is not held."""
import numpy as np
import pytest

from gpu_util import announce
from paper_1108_2651_amd import lbem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls,per_cell", [(True, 36), (False, 60)])
def test_second_copy_only_where_it_is_used(walls, per_cell):
    import torch
    shape = (128, 128, 128)
    s = lbem.Solver(3, shape, "f32", streaming="pull")
    if walls:
        s.set_boundary(2, "pec")
    s.set_medium(np.ones(s.n))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    s.set_dispersion(0.01, 0.02, 0.001)
    used = before - torch.cuda.mem_get_info()[0]
    announce(f"3D f32 pole, walls={walls}: {used / s.n:.1f} B per cell")
    # each of the two or three allocations is rounded up to at most 4 MiB more
    assert per_cell * s.n <= used <= per_cell * s.n + 3 * (4 << 20)
    s.close()
