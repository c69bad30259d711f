"""A captured lbem_step replayed with eager calls and batch ticks of even numbers of
steps between the replays: every replay advances the handle as the same eager call
does, bit for bit (the reference handle takes every step eagerly)."""
import os

import numpy as np
import pytest

from gpu_util import announce, random_problem
from paper_1108_2651_amd import lbem, serve

pytestmark = pytest.mark.gpu

#        dim  shape          format     environment           pole
CASES = [(2, (130, 40, 1), "f16ghost", {}, False), (2, (130, 40, 1), "f32", {}, False),
         (2, (130, 40, 1), "f64", {}, True), (3, (40, 30, 20), "f16dev", {"LBEM_DEV3F": "1"}, False),
         (3, (40, 30, 20), "f32", {"LBEM_FUSE3": "2"}, True), (3, (104, 100, 100), "f32", {}, False)]


def handles(dim, shape, prec, env, pole, stream, nsteps=4):
    p = random_problem(dim, shape, seed=sum(shape), nsteps=nsteps, src=False)
    os.environ.update(env)
    try:
        out = [lbem.Solver(dim, shape, prec, streaming="pull", stream=stream) for _ in range(2)]
    finally:
        for k in env:
            os.environ.pop(k)
    for s in out:
        s.set_medium(p.eps_r)
        if pole:
            s.set_dispersion(0.01, 0.02, 0.001)
        s.init_fields(p.E0, p.B0)
        s.step(3)
        assert s.steps_per_launch > 1
    stream.synchronize()
    return out


def capture(s, stream, n):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        s.step(n)
    return g


def replay(g, stream):
    import torch
    with torch.cuda.stream(stream):
        g.replay()
    torch.cuda.synchronize()


def same(a, b):
    (Ea, Ba), (Eb, Bb) = a.moments(), b.moments()
    return np.array_equal(Ea, Eb) and np.array_equal(Ba, Bb)


@pytest.mark.parametrize("dim,shape,prec,env,pole", CASES)
def test_even_calls_between_replays(dim, shape, prec, env, pole):
    import torch
    st = torch.cuda.Stream()
    a, b = handles(dim, shape, prec, env, pole, st)
    g = capture(a, st, 10)
    for eager in (0, 4, 2, 6, 12):
        announce(f"replay {dim}D {shape} {prec} pole={pole}: after {eager} eager steps")
        a.step(eager)
        replay(g, st)
        b.step(eager)
        b.step(10)
        assert same(a, b), eager
    if not pole:
        os.environ["LBEM_BATCH_MULTI"] = "2"      # also where the members are too small for it to pay
        try:
            batch = serve.Batch(2, 6, st)
        finally:
            os.environ.pop("LBEM_BATCH_MULTI")
        for tick in (6, 4):
            announce(f"replay {dim}D {shape} {prec}: after a batch tick of {tick} steps")
            batch.run([a], [tick])
            replay(g, st)
            b.step(tick)
            b.step(10)
            assert same(a, b), tick
        batch.close()
    a.close()
    b.close()


@pytest.mark.parametrize("dim,shape,prec,n", [(2, (130, 40, 1), "f32", 5), (2, (130, 40, 1), "f32", 7),
                                              (2, (60, 50, 1), "f64", 3), (3, (104, 100, 100), "f32", 3),
                                              (3, (104, 100, 100), "f32", 7)])
def test_odd_captures_of_plain_formats(dim, shape, prec, n):
    """An odd number of steps, more than one, of FP32 and FP64 without extras replays
    as well."""
    import torch
    st = torch.cuda.Stream()
    a, b = handles(dim, shape, prec, {}, False, st)
    g = capture(a, st, n)
    for k in range(3):
        announce(f"replay {dim}D {shape} {prec}: {n} steps, {k}")
        replay(g, st)
        b.step(n)
        assert same(a, b), k
        a.step(4)
        b.step(4)
    a.close()
    b.close()
