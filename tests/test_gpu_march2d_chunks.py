"""2D launches of several steps on boxes of middle size, where the rows of a chunk are
chosen by the waves that share a SIMD, and on one wider than 256 strips, whose source
mask holds one bit for strips 256 apart: bit for bit equal to single steps."""
import numpy as np
import pytest

from gpu_util import announce, gpu_run, random_problem

pytestmark = pytest.mark.gpu


def equal(p, steps, prec):
    ref = gpu_run(p, steps, prec, "pull", env={"LBEM_FUSE": 1})
    got = gpu_run(p, steps, prec, "pull")
    assert got.steps_per_launch == 4
    ok = np.array_equal(got.get_state(), ref.get_state())
    ref.close()
    got.close()
    return ok


@pytest.mark.parametrize("prec", ["f32", "f64", "f16dev"])
@pytest.mark.parametrize("shape", [(350, 351, 1), (500, 500, 1), (700, 690, 1), (1201, 400, 1), (3000, 80, 1), (80, 3001, 1)])
def test_chunks_of_middle_sizes(prec, shape):
    announce(f"march chunks {prec} {shape}")
    p = random_problem(2, shape, seed=sum(shape), mu=shape[0] == 700, nsteps=10)
    assert equal(p, 10, prec), (prec, shape)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("cells", [[(60, 3)], [(14395, 1)], [(60, 3), (14395, 1)]])
def test_strips_that_share_a_mask_bit(prec, cells):
    announce(f"march mask {prec} {cells}")
    p = random_problem(2, (14400, 6, 1), seed=7, nsteps=9)
    p.src_cells = np.array([x + 14400 * y for x, y in cells])
    p.src_weights = np.linspace(1.0, 2.0, len(cells))
    assert equal(p, 9, prec), cells
