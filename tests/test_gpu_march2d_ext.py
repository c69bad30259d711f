"""Several steps per launch of 2D FP32 and FP64 with walls, an absorbing layer
and a dispersion pole: bit for bit equal to single steps for every kind of wall,
at the edges of strips (56 columns, 120 with two cells per lane) and chunks of
rows, on boxes narrower than a strip and lower than a chunk, with scattered
sources, the mu term, general tau and step counts that leave one, two and three.
Both sides run the same arithmetic, so the tolerance is zero."""
import os

import numpy as np
import pytest

from gpu_util import announce, random_problem
from paper_1108_2651_amd import lbem

pytestmark = pytest.mark.gpu


def run(p, prec, env, walls, pole, damp, tau, steps):
    os.environ.update(env)
    try:
        s = lbem.Solver(2, p.shape, prec, tau=p.tau if tau is None else tau, streaming="pull",
                        mu_varies=p.mu_r is not None)
    finally:
        for k in env:
            os.environ.pop(k)
    rng = np.random.default_rng(5)
    for a, kind in walls:
        s.set_boundary(a, kind)
    s.set_medium(p.eps_r, p.mu_r)
    if pole:
        s.set_dispersion(rng.uniform(0, 0.02, p.n), rng.uniform(0, 0.03, p.n), rng.uniform(0, 0.01, p.n))
    if damp:
        s.set_absorber(rng.uniform(0, 0.1, p.n))
    s.init_fields(p.E0, p.B0)
    if len(p.src_cells):
        s.set_source(p.src_comp, p.src_cells, p.src_weights)
    spl = s.steps_per_launch
    for n, k in zip(steps, np.cumsum([0] + steps)):
        s.step(n, p.amp[k:k + n] if len(p.src_cells) else None)
    out = s.get_state()
    s.close()
    return out, spl


WALLS = [[], [(0, "pec")], [(1, "pec")], [(0, "pmc"), (1, "pmc")], [(0, "pmc"), (1, "pec")], [(0, "pec"), (1, "pec")]]


@pytest.mark.parametrize("shape", [(56, 74, 1), (57, 75, 1), (113, 41, 1), (1, 4096, 1), (2049, 2, 1), (65, 200, 1)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("mu,src", [(False, True), (True, False)])
def test_walls_and_extras(shape, prec, mu, src):
    p = random_problem(2, shape, seed=sum(shape) + 3 * mu, mu=mu, src=src, nsteps=32)
    for walls in WALLS:
        for pole, damp, tau in ((False, False, None), (True, False, 0.8), (False, True, None), (True, True, None)):
            if not (walls or pole or damp):
                continue
            steps = [9, 3, 8, 4]
            announce(f"march ext {prec} {shape} mu={mu} walls={walls} pole={pole} damp={damp} tau={tau}")
            want, one = run(p, prec, {"LBEM_FUSE": "1"}, walls, pole, damp, tau, steps)
            got, four = run(p, prec, {}, walls, pole, damp, tau, steps)
            assert (one, four) == (1, 4)
            assert np.array_equal(got, want), (shape, walls, pole, damp)
            got, two = run(p, prec, {"LBEM_FUSE": "2"}, walls, pole, damp, tau, steps)
            assert two == 2 and np.array_equal(got, want), (shape, walls, pole, damp)


def test_two_cells_per_lane():
    p = random_problem(2, (3602, 2222, 1), seed=4, nsteps=8)
    for walls, pole, damp in (([(0, "pec"), (1, "pmc")], False, True), ([(1, "pec")], True, False)):
        announce(f"march ext two cells per lane walls={walls} pole={pole} damp={damp}")
        want, _ = run(p, "f32", {"LBEM_FUSE": "1"}, walls, pole, damp, None, [8])
        got, spl = run(p, "f32", {}, walls, pole, damp, None, [8])
        assert spl == 4 and np.array_equal(got, want)
