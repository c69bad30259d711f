"""2D multi-step launches (register march over column strips and row chunks):
two, three and four steps per launch equal single steps bit for bit, in every
format that has them, fields and stored state, at the
edges of the strips (56 stored columns of 64, or 120 of 128 for large FP32
lattices with rows of even length) and of the chunks, with sources whose
periodic images fall into several strips, the mu term, general tau, and call
lengths that leave every remainder.  Both sides run the same arithmetic, so
the tolerance is zero."""
import numpy as np
import pytest

from gpu_util import announce, gpu_run, random_problem

pytestmark = pytest.mark.gpu


def same(a, b):
    x, y = a.moments(), b.moments()
    ok = np.array_equal(x[0], y[0]) and np.array_equal(x[1], y[1])
    a.close()
    b.close()
    return ok


@pytest.mark.parametrize("prec", ["f32", "f64", "f16dev", "bf16dev", "f16ghost", "bf16ghost"])
@pytest.mark.parametrize("shape", [(55, 9, 1), (56, 1, 1), (57, 3, 1), (64, 25, 1), (113, 48, 1), (3, 70, 1)])
@pytest.mark.parametrize("mu", [False, True])
def test_strip_and_chunk_edges(prec, shape, mu):
    p = random_problem(2, shape, seed=sum(shape) + 3 * mu, mu=mu, nsteps=12)
    for steps in (3, 4, 5, 11, 12):          # after the first single step: 2, 3, 4, 4+4+2, 4+4+3
        for tau in (None, 0.8):
            announce(f"march {prec} {shape} mu={mu} steps={steps} tau={tau}")
            ref = gpu_run(p, steps, prec, "pull", tau=tau, env={"LBEM_FUSE": 1})
            got = gpu_run(p, steps, prec, "pull", tau=tau)
            assert ref.steps_per_launch == 1 and got.steps_per_launch == 4
            assert np.array_equal(got.get_state(), ref.get_state()), (prec, shape, steps, tau)
            assert same(got, ref), (prec, shape, steps, tau)


@pytest.mark.parametrize("shape", [(4096, 1960, 1), (4095, 1961, 1)])
def test_large_lattices(shape):
    """From 8e6 cells on, FP32 rows of even length take two cells per lane."""
    p = random_problem(2, shape, seed=5, nsteps=6)
    announce(f"march f32 {shape}")
    assert same(gpu_run(p, 6, "f32", "pull"), gpu_run(p, 6, "f32", "pull", env={"LBEM_FUSE": 1}))
