"""Several steps per launch for the batched 16-bit classes (four in 2D, two in
3D): every member equals the same lattice stepped alone, bit for bit, for step
counts that leave every remainder (members that skip launches beside members
that take them), with sources and their amplitudes, and with a varying mu in
every member of a class.  Both sides run the same arithmetic: tolerance zero."""
import os

import numpy as np
import pytest

from gpu_util import announce, gpu_run, random_problem
from paper_1108_2651_amd import lbem, serve

pytestmark = pytest.mark.gpu

SHAPES = {2: [(70, 33, 1), (56, 24, 1), (130, 5, 1), (57, 64, 1)], 3: [(20, 16, 12), (61, 13, 9), (60, 24, 5), (9, 30, 17)]}


@pytest.mark.parametrize("prec", ["f16dev", "bf16dev", "f16ghost", "bf16ghost"])
@pytest.mark.parametrize("dim,mu", [(2, False), (2, True), (3, False), (3, True)])
def test_members_equal_solo_runs(dim, mu, prec):
    import torch
    st = torch.cuda.Stream()
    os.environ["LBEM_BATCH_MULTI"] = "2"       # also where the 3D members are too small for it to pay
    try:
        batch = serve.Batch(8, 11, st)
    finally:
        os.environ.pop("LBEM_BATCH_MULTI", None)
    plan = [[11, 8, 1, 6], [4, 0, 5, 2], [7, 3, 11, 10]]
    total = np.sum(plan, axis=0)
    probs, members = [], []
    for k, shape in enumerate(SHAPES[dim]):
        p = random_problem(dim, shape, seed=40 + k, mu=mu, src=k != 1, nsteps=int(total[k]))
        os.environ["LBEM_DEV3F"] = "1"         # 3D members carry the source segments
        try:
            s = lbem.Solver(dim, shape, prec, mu_varies=mu, streaming="pull", stream=st)
        finally:
            os.environ.pop("LBEM_DEV3F", None)
        s.setup(p)
        probs.append(p)
        members.append(s)
    done = np.zeros(4, int)
    for ns in plan:
        amps = [p.amp[d:d + n] if p.amp is not None else None for p, d, n in zip(probs, done, ns)]
        batch.run(members, ns, amps)
        done += np.asarray(ns)
    for k, p in enumerate(probs):
        announce(f"batch multi {dim}D {p.shape} {prec} mu={mu} steps={total[k]}")
        want = gpu_run(p, int(total[k]), prec, "pull", env={"LBEM_FUSE": 1, "LBEM_DEV3F": 0})
        assert members[k].t == total[k]
        a, b = members[k].moments(), want.moments()
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (p.shape, prec)
        assert np.array_equal(members[k].get_state(), want.get_state())
        want.close()
        members[k].close()
    batch.close()
