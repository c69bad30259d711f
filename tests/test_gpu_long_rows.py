"""Rows of more than 2^29 columns, whose byte offsets of doubles need 64 bits.  2D
FP64: two steps per launch against the FP64 oracle on windows around pulses and
source cells on both sides of column 2^29, and no field elsewhere.  3D 16-bit: the
fields as the per-cell reader gives them, also where the tiled reader is asked for."""
import os

import numpy as np
import pytest

from gpu_util import announce
from oracle import oracle as O
from paper_1108_2651_amd import lbem
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

NX, STEPS = 2 ** 29 + 192, 5
H = STEPS + 2                           # half width of a window: the light cone and one cell for grad ln mu


@pytest.mark.parametrize("mu", [False, True])
def test_long_rows(mu):
    import torch
    torch.cuda.empty_cache()            # arenas of earlier tests, cached by torch
    announce(f"2D f64 {NX}x1 mu={mu}: set-up")
    rng = np.random.default_rng(3)
    eps = np.resize(rng.uniform(1.0, 4.0, 1000003), NX)
    mur = np.resize(rng.uniform(1.0, 1.5, 1000033), NX) if mu else None
    centres = [0, 40, 2 ** 28, 2 ** 29 - 20, 2 ** 29, 2 ** 29 + 20, NX - 40]
    E, B = np.zeros((3, NX)), np.zeros((3, NX))
    cells = []
    for k, c in enumerate(centres):
        if k % 2:
            cells.append(c)
        else:
            E[2, c] = 1.0 + k
            B[0, c], B[1, c] = 0.5, -0.25 * k
    weights = np.linspace(1.0, 2.0, len(cells))
    amp = rng.standard_normal(STEPS)
    s = lbem.Solver(2, (NX, 1, 1), "f64", mu_varies=mu)
    s.set_medium(eps, mur)
    s.init_fields(E, B)
    s.set_source(2, np.array(cells), weights)
    assert s.steps_per_launch == 2
    announce("  steps")
    s.step(STEPS, amp)
    Eg = torch.zeros((3, NX), dtype=torch.float64, device="cuda")
    Bg = torch.zeros_like(Eg)
    s.moments_device(Eg, Bg)
    seen = 0
    for c in centres:
        idx = (np.arange(c - H, c + H + 1)) % NX
        o = O.Oracle(2, (2 * H + 1, 1, 1))
        o.set_medium(eps[idx], None if mur is None else mur[idx])
        o.init_fields(E[:, idx], B[:, idx])
        here = [(int(np.where(idx == x)[0][0]), w) for x, w in zip(cells, weights) if x in idx]
        if here:
            o.set_source(2, np.array([x for x, _ in here]), np.array([w for _, w in here]))
        o.step(STEPS, amp if here else None)
        Eo, Bo = o.fields()
        at = torch.from_numpy(idx).cuda()
        inner = slice(1, 2 * H)         # the window's outermost cells see its own edge through grad ln mu
        for got, want in ((Eg[2][at].cpu().numpy(), Eo[2]), (Bg[1][at].cpu().numpy(), Bo[1])):
            assert np.abs(got - want)[inner].max() <= TOL["f64"] * max(np.abs(want).max(), 1.0), c
        seen += int(torch.count_nonzero(Eg[2][at]))
        assert int(torch.count_nonzero(Eg[2][at])) > 0, c
    assert int(torch.count_nonzero(Eg[2])) == seen
    s.close()
    del s, Eg, Bg
    torch.cuda.empty_cache()


def test_fields_of_long_rows():
    import torch
    torch.cuda.empty_cache()
    n = 2 ** 29 + 192
    E, B = np.zeros((3, n)), np.zeros((3, n))
    centres = [0, 40, 2 ** 28, 2 ** 29 - 20, 2 ** 29, 2 ** 29 + 20, n - 40]
    for k, c in enumerate(centres):
        E[:, c], B[:, c] = (1.0, -0.5, 0.25 + k), (0.5, 0.125, -k)
    os.environ["LBEM_FIELDS3"] = "1"
    try:
        s = lbem.Solver(3, (n, 1, 1), "f16ghost")
    finally:
        os.environ.pop("LBEM_FIELDS3", None)
    announce(f"fields 3d f16ghost {n}x1x1: set-up")
    s.set_medium(np.full(n, 1.0))
    s.init_fields(E, B)
    announce("  step")
    s.step(1)
    Eg = torch.zeros((3, n), dtype=torch.float64, device="cuda")
    Bg = torch.zeros_like(Eg)
    s.moments_device(Eg, Bg)
    seen = [0] * 6
    for c in centres:
        idx = np.arange(c - H, c + H + 1) % n
        o = O.Oracle(3, (2 * H + 1, 1, 1))
        o.set_medium(np.full(2 * H + 1, 1.0))
        o.init_fields(E[:, idx], B[:, idx])
        o.step(1)
        at = torch.from_numpy(idx).cuda()
        for k, (got, want) in enumerate(zip((*Eg, *Bg), (*o.fields()[0], *o.fields()[1]))):
            got = got[at].cpu().numpy()
            assert np.abs(got - want).max() <= TOL["f16ghost"] * np.abs(o.fields()).max(), (c, k)
            seen[k] += np.count_nonzero(got)
    assert [int(torch.count_nonzero(f)) for f in (*Eg, *Bg)] == seen
    s.close()
    del s, Eg, Bg
    torch.cuda.empty_cache()
