"""Two steps per launch of the 3D 16-bit formats (tiles of 60 x 12 stored cells,
chunks of planes): bit for bit equal to single steps at the edges of the tiles
and chunks, on boxes smaller than a tile's frame, with sources whose periodic
images fall into several tiles, the mu term, general tau, and odd step counts.
Both sides run the same arithmetic, so the tolerance is zero."""
import numpy as np
import pytest

from gpu_util import announce, gpu_run, random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(60, 12, 8), (61, 13, 9), (59, 11, 3), (121, 25, 5), (4, 4, 4), (64, 30, 1)])
@pytest.mark.parametrize("mu", [False, True])
def test_tile_and_chunk_edges(shape, mu):
    p = random_problem(3, shape, seed=sum(shape) + 3 * mu, mu=mu, nsteps=8)
    for prec in ("f16dev", "f16ghost", "bf16dev", "bf16ghost"):
        for steps, tau in ((5, None), (8, 0.8)):
            ref = gpu_run(p, steps, prec, "pull", tau=tau, env={"LBEM_DEV3F": 0})
            want = ref.get_state()
            ref.close()
            for lz in (0, 1, 3, 8):             # 0: the default chunk
                announce(f"pair {prec} {shape} mu={mu} steps={steps} tau={tau} planes={lz}")
                env = dict(LBEM_DEV3F=1, **({"LBEM_FUSE3_LZ": lz} if lz else {}))
                got = gpu_run(p, steps, prec, "pull", tau=tau, env=env)
                assert got.steps_per_launch == 2
                assert np.array_equal(got.get_state(), want), (prec, shape, steps, lz)
                got.close()


@pytest.mark.parametrize("shape", [(62, 14, 6), (63, 15, 7), (61, 13, 5), (3, 4, 5), (130, 30, 1)])
def test_fields_on_tiles(shape):
    """E and B read on tiles (62 x 14 cells, each stored cell decoded once)
    equal the per-cell reader's, both fields together and each alone."""
    import torch
    p = random_problem(3, shape, seed=sum(shape), nsteps=3)
    for prec in ("f16dev", "f16ghost", "bf16dev", "bf16ghost"):
        announce(f"fields on tiles {prec} {shape}")
        a = gpu_run(p, 3, prec, "pull", env={"LBEM_FIELDS3": 0})
        b = gpu_run(p, 3, prec, "pull", env={"LBEM_FIELDS3": 1})
        (Ea, Ba), (Eb, Bb) = a.moments(), b.moments()
        assert np.array_equal(Ea, Eb) and np.array_equal(Ba, Bb), (prec, shape)
        E = torch.zeros((3, p.n), dtype=torch.float64, device="cuda")
        B = torch.zeros_like(E)
        b.moments_device(E, B)
        assert np.array_equal(E.cpu().numpy(), Ea) and np.array_equal(B.cpu().numpy(), Ba)
        a.close()
        b.close()


def test_default_takes_the_pair_on_large_boxes():
    """From about 88^3 on; the default equals single steps."""
    p = random_problem(3, (101, 96, 90), seed=3, nsteps=5)
    a = gpu_run(p, 5, "f16ghost")
    b = gpu_run(p, 5, "f16ghost", env={"LBEM_DEV3F": 0})
    announce("pair default 101x96x90 f16ghost")
    assert a.steps_per_launch == 2 and b.steps_per_launch == 1
    assert np.array_equal(a.get_state(), b.get_state())
    a.close()
    b.close()
