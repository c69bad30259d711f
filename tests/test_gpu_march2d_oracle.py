"""2D FP32 and FP64 with walls, an absorbing layer or a dispersion pole in launches of
four steps (boxes of 4096 cells and more) against the oracle, with every other term
present (heterogeneous eps and mu, a scattered source).  The bars are those of every
parity test of these formats."""
import numpy as np
import pytest

from gpu_util import announce, random_problem, rel
from oracle import oracle as O
from paper_1108_2651_amd import lbem
from test_gpu_boundaries import layer
from test_gpu_dispersion import poles
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

#        shape           walls                        mu     absorber  pole
CASES = [((70, 61, 1), [(0, "pec")], False, True, False), ((57, 80, 1), [(0, "pmc"), (1, "pec")], True, False, False),
         ((120, 40, 1), [(0, "pec"), (1, "pec")], False, True, False), ((113, 41, 1), [(1, "pmc")], True, True, False),
         ((90, 61, 1), [], True, False, True), ((64, 66, 1), [(0, "pec"), (1, "pmc")], False, True, True),
         ((2050, 2, 1), [(0, "pmc")], False, False, True), ((3, 1400, 1), [(1, "pec")], True, True, True)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape,walls,mu,absorb,pole", CASES)
def test_extras_in_launches_of_four_match_the_oracle(shape, walls, mu, absorb, pole, prec):
    steps = 58                                  # a single step, fourteen launches of four, one single
    p = random_problem(2, shape, seed=sum(shape) + len(walls), mu=mu, nsteps=steps)
    s = lbem.Solver(2, shape, prec, w0_vac=p.w0_vac, mu_varies=mu, streaming="pull")
    o = O.Oracle(2, shape, p.tau, p.w0_vac)
    for h in (s, o):
        for a, k in walls:
            h.set_boundary(a, k)
        h.set_medium(p.eps_r, p.mu_r)
        if absorb:
            h.set_absorber(layer(shape, 4, 0.08, [a for a, _ in walls] or [0, 1]))
        if pole:
            h.set_dispersion(*poles(p.n, sum(shape)))
        h.init_fields(p.E0, p.B0)
        h.set_source(p.src_comp, p.src_cells, p.src_weights)
    assert s.steps_per_launch == 4
    s.step(steps, p.amp[:steps])
    o.step(steps, p.amp[:steps])
    (Eg, Bg), (Eo, Bo) = s.moments(), o.fields()
    eE, eB = rel(Eg, Eo), rel(Bg, Bo)
    announce(f"march extras {shape} {walls} mu={mu} absorber={absorb} pole={pole} {prec}: E {eE:.2e} B {eB:.2e}")
    assert eE <= TOL[prec] and eB <= TOL[prec], (eE, eB)
    s.close()
