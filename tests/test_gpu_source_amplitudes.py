"""A source amplitude that is not finite reaches the source cells alone in its own
step, however many steps the launch takes: the same fields as single steps, cell by
cell (NaN and infinity in the same places)."""
import os

import numpy as np
import pytest

from gpu_util import announce, random_problem
from paper_1108_2651_amd import lbem

pytestmark = pytest.mark.gpu


def run(p, prec, env, amp, steps):
    os.environ.update(env)
    try:
        s = lbem.Solver(p.dim, p.shape, prec, streaming="pull")
    finally:
        for k in env:
            os.environ.pop(k)
    s.set_medium(p.eps_r)
    s.init_fields(p.E0, p.B0)
    s.set_source(p.src_comp, p.src_cells[:3], p.src_weights[:3])
    spl = s.steps_per_launch
    s.step(steps, amp)
    out = s.moments()
    s.close()
    return out, spl


@pytest.mark.parametrize("dim,shape,prec,single,several", [
    (2, (150, 21, 1), "f32", {"LBEM_FUSE": "1"}, {}), (2, (150, 21, 1), "f64", {"LBEM_FUSE": "1"}, {}),
    (2, (150, 21, 1), "f16dev", {"LBEM_FUSE": "1"}, {}), (2, (150, 21, 1), "f16ghost", {"LBEM_FUSE": "1"}, {}),
    (3, (140, 30, 9), "f32", {"LBEM_FUSE3": "1"}, {"LBEM_FUSE3": "2", "LBEM_PAIR3F": "1"}),
    (3, (140, 30, 9), "f16dev", {"LBEM_DEV3F": "0"}, {"LBEM_DEV3F": "1"}),
    (3, (140, 30, 9), "f16ghost", {"LBEM_DEV3F": "0"}, {"LBEM_DEV3F": "1"})])
def test_amplitude_that_is_not_finite(dim, shape, prec, single, several):
    p = random_problem(dim, shape, seed=sum(shape), nsteps=5)
    for steps, at in ((5, 4), (5, 3), (3, 2)):
        for bad in (np.inf, np.nan):
            announce(f"amplitude {bad} in step {at} of {steps}: {dim}D {prec} {several}")
            amp = np.array(p.amp[:steps])
            amp[at] = bad
            (Ea, Ba), one = run(p, prec, single, amp, steps)
            (Eb, Bb), more = run(p, prec, several, amp, steps)
            assert one == 1 and more > 1
            assert np.array_equal(Ea, Eb, equal_nan=True) and np.array_equal(Ba, Bb, equal_nan=True), (steps, at, bad)
            assert 0 < np.count_nonzero(~np.isfinite(Ea)) < p.n // 2
