"""Batch members with the default tiles may share one launch and chunk length,
members whose tile was set keep it; either way each member's state is that of
the mesh stepped alone, bit for bit."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

# rows of half a wave to two tiles, with ragged ends of tile and chunk
SIZES_2D = [(32, 7), (64, 64), (129, 33), (192, 65), (257, 16), (512, 5)]
SIZES_3D = [(32, 16, 5), (48, 48, 9), (33, 17, 16)]


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


@pytest.mark.parametrize("sizes,tiles", [(SIZES_2D, None), (SIZES_2D, [(64, 1, 0), (128, 1, 2), (256, 1, 0)]),
                                         (SIZES_3D, None), (SIZES_3D, [(16, 16, 0), (32, 8, 3), (32, 16, 0)])])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("integrator", [0, 1])
def test_members_equal_alone(H, sizes, tiles, precision, integrator):
    import torch
    s = torch.cuda.Stream()
    cases = [wl.turbulence_3d(n=n, mach=0.6, seed=30 + i) for i, n in enumerate(sizes)]

    def mesh(c, i):
        h = H.Hydro(c.n, c.gamma, c.cfl, precision=precision, stream=s, integrator=integrator)
        if tiles:
            h.set_tile(*tiles[i % len(tiles)])
        h.set_primitive(c.W)
        return h

    say("batch tiles", len(sizes[0]), tiles, precision, integrator)
    ms = [mesh(c, i) for i, c in enumerate(cases)]
    b = H.Batch(ms, use_graph=False)
    if tiles:
        assert b.info()["groups"] == len(tiles)
    b.step(4)
    s.synchronize()
    got = [(h.get_state(), h.time()) for h in ms]
    b.close()
    for i, c in enumerate(cases):
        h = mesh(c, i)
        h.step_auto(4)
        assert np.array_equal(h.get_state(), got[i][0]) and h.time() == got[i][1], c.n
        h.close()
        ms[i].close()
