"""Two steps per launch of 3D FP32 on tiles of 62 x 14 stored cells, with an
absorbing layer, a dispersion pole, both or neither: bit for bit equal to single
steps at the edges of the tiles and chunks, on boxes smaller than a tile's
frame, with scattered sources, the mu term, general tau, and odd step counts.
Both sides run the same arithmetic, so the tolerance is zero."""
import os

import numpy as np
import pytest

from gpu_util import announce, random_problem
from paper_1108_2651_amd import lbem

pytestmark = pytest.mark.gpu


def solver(p, env, pole, damp, tau):
    os.environ.update(env)
    try:
        s = lbem.Solver(3, p.shape, "f32", tau=p.tau if tau is None else tau, streaming="pull",
                        mu_varies=p.mu_r is not None)
    finally:
        for k in env:
            os.environ.pop(k)
    rng = np.random.default_rng(5)
    s.set_medium(p.eps_r, p.mu_r)
    if pole:
        s.set_dispersion(rng.uniform(0, 0.02, p.n), rng.uniform(0, 0.03, p.n), rng.uniform(0, 0.01, p.n))
    if damp:
        s.set_absorber(rng.uniform(0, 0.1, p.n))
    s.init_fields(p.E0, p.B0)
    s.set_source(p.src_comp, p.src_cells, p.src_weights)
    return s


@pytest.mark.parametrize("shape", [(62, 14, 8), (63, 15, 9), (61, 13, 3), (125, 29, 5), (3, 4, 5), (64, 30, 1)])
@pytest.mark.parametrize("mu", [False, True])
def test_tile_and_chunk_edges(shape, mu):
    p = random_problem(3, shape, seed=sum(shape) + 3 * mu, mu=mu, nsteps=9)
    for pole, damp in ((True, False), (False, True), (True, True), (False, False)):
        for steps, tau in ((5, None), (8, 0.8)):
            ref = solver(p, {"LBEM_FUSE3": "1"}, pole, damp, tau)
            assert ref.steps_per_launch == 1
            ref.step(steps, p.amp[:steps])
            want = ref.get_state()
            ref.close()
            for lz in ("", "1", "3", "8"):             # "": the default chunk
                announce(f"pair f32 {shape} mu={mu} pole={pole} damp={damp} steps={steps} tau={tau} planes={lz}")
                env = dict(LBEM_FUSE3="2", LBEM_PAIR3F="1", **({"LBEM_FUSE3_LZ": lz} if lz else {}))
                got = solver(p, env, pole, damp, tau)
                assert got.steps_per_launch == 2
                got.step(steps, p.amp[:steps])
                assert np.array_equal(got.get_state(), want), (shape, pole, damp, steps, lz)
                got.close()


def test_extras_come_and_go():
    """A pole and an absorber added and taken away between calls, a blob
    saved between pairs, and the default choice: the same as single steps."""
    p = random_problem(3, (101, 96, 90), seed=3, nsteps=32)
    out = []
    for env in ({}, {"LBEM_FUSE3": "1"}):
        s = solver(p, env, True, False, None)
        spl = s.steps_per_launch
        s.step(5, p.amp[:5])
        blob = s.get_state()
        s.step(4, p.amp[5:9])
        s.set_state(blob)
        s.step(3, p.amp[5:8])
        a = s.get_state()
        s.set_absorber(np.full(p.n, 0.01))
        s.step(6, p.amp[8:14])
        s.set_dispersion(None)
        s.step(7, p.amp[14:21])
        s.set_absorber(None)
        s.step(4, p.amp[21:25])
        out.append((a, s.get_state()))
        announce(f"extras come and go: steps per launch {spl}")
        assert spl == (1 if env else 2)
        s.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("dim,shape,prec,env", [(2, (130, 40, 1), "f32", {}), (2, (130, 40, 1), "f16ghost", {}),
                                                (3, (40, 30, 20), "f16dev", {"LBEM_DEV3F": "1"}),
                                                (3, (40, 30, 20), "f32", {"LBEM_FUSE3": "2"})])
def test_captured_steps_replay(dim, shape, prec, env):
    """A graph of an even number of steps replays: it ends in the buffer it
    began in, also where eager calls take several steps per launch."""
    import torch
    announce(f"captured steps {dim}D {shape} {prec}")
    p = random_problem(dim, shape, seed=sum(shape), nsteps=4, src=False)
    st = torch.cuda.Stream()
    os.environ.update(env)
    try:
        a, b = (lbem.Solver(dim, shape, prec, streaming="pull", stream=st) for _ in range(2))
    finally:
        for k in env:
            os.environ.pop(k)
    for s in (a, b):
        s.set_medium(p.eps_r)
        if env.get("LBEM_FUSE3"):
            s.set_dispersion(0.01, 0.02, 0.001)
        s.init_fields(p.E0, p.B0)
        s.step(3)
    assert a.steps_per_launch > 1
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        a.step(18)
    x = torch.zeros(1000, device="cuda")
    for k in range(3):
        with torch.cuda.stream(st):
            g.replay()
        torch.cuda.synchronize()
        x += 1
        torch.cuda.synchronize()
        b.step(18)
        (Ea, Ba), (Eb, Bb) = a.moments(), b.moments()
        assert np.array_equal(Ea, Eb) and np.array_equal(Ba, Bb), k
    assert float(x[0]) == 3.0
    a.close()
    b.close()
