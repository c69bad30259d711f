"""Two steps per launch of 3D FP32 at the borders of its tiles of 64 x 13 stored cells:
a last tile of one column, full neighbouring tiles, an interior tile between two
others, one tile that wraps onto itself, whole rows of tiles, with scattered sources
and the mu term across the borders.  Bit for bit equal to single steps."""
import numpy as np
import pytest

from gpu_util import announce, random_problem
from test_gpu_pair3f import solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(65, 13, 8), (128, 26, 5), (129, 27, 9), (193, 39, 3), (64, 14, 4), (192, 12, 4)])
@pytest.mark.parametrize("mu", [False, True])
def test_tile_borders(shape, mu):
    p = random_problem(3, shape, seed=sum(shape) + 5 * mu, mu=mu, nsteps=9)
    for pole, damp, steps, tau in ((True, True, 5, None), (False, False, 8, 0.8), (False, False, 5, None)):
        ref = solver(p, {"LBEM_FUSE3": "1"}, pole, damp, tau)
        ref.step(steps, p.amp[:steps])
        want = ref.get_state()
        ref.close()
        for lz in ("", "1", "2"):               # "": the default chunk
            announce(f"pair f32 borders {shape} mu={mu} pole={pole} steps={steps} tau={tau} planes={lz}")
            env = dict(LBEM_FUSE3="2", LBEM_PAIR3F="1", **({"LBEM_FUSE3_LZ": lz} if lz else {}))
            got = solver(p, env, pole, damp, tau)
            assert got.steps_per_launch == 2
            got.step(steps, p.amp[:steps])
            assert np.array_equal(got.get_state(), want), (shape, pole, steps, lz)
            got.close()


@pytest.mark.parametrize("shape", [(66, 130, 124), (124, 126, 70), (250, 80, 60), (256, 64, 64)])
def test_default_of_either_tiling(shape):
    """Boxes on both sides of the rule that chooses between the two kinds of tiles."""
    p = random_problem(3, shape, seed=sum(shape), nsteps=5)
    announce(f"3D f32 default {shape}")
    a, b = solver(p, {}, False, False, None), solver(p, {"LBEM_FUSE3": "1"}, False, False, None)
    for s in (a, b):
        s.step(5, p.amp[:5])
    assert a.steps_per_launch == 2 and np.array_equal(a.get_state(), b.get_state())
    a.close()
    b.close()
