"""The FP64 3-D Heun stage 2 has a form for launches of few work-groups: the
same states bit for bit as the other form on either side of the line between
them (two work-groups of four waves on each of 256 CUs), alone, on block
streams and in batches."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


def _run(H, c, tile, bc=None, blocks=None, streams=False):
    h = H.Hydro(c.n, c.gamma, c.cfl, precision=H.FP64, bc=bc, blocks=blocks)
    h.set_tile(*tile)
    if streams:
        h.set_block_streams(True)
    h.set_primitive(c.W)
    h.step_auto(3)
    out = h.get_state(), h.time()
    h.close()
    return out


# 512 work-groups of 32 x 8, 516 of them, and ragged ends of tile and chunk
@pytest.mark.parametrize("n", [(128, 128, 8), (129, 64, 13), (96, 88, 86), (33, 17, 37)])
@pytest.mark.parametrize("bc", [0, 2, 3])
def test_forms_agree(H, n, bc):
    c = wl.turbulence_3d(n=n, mach=0.6, seed=31)
    bc = ((bc, bc),) * 3
    say("few waves", n, bc)
    ref = _run(H, c, (16, 16, n[2]), bc)
    for tile in [(32, 8, 1), (32, 8, 7), (16, 16, 1), (16, 16, 5), (32, 16, 1), (64, 8, 3), (32, 8, 0)]:
        got = _run(H, c, tile, bc)
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1], tile


def test_forms_agree_on_block_streams_and_in_batches(H):
    import torch
    c = wl.turbulence_3d(n=(64, 64, 48), mach=0.6, seed=32)
    say("few waves, block streams")
    ref = _run(H, c, (16, 16, 48))
    for tile in [(16, 16, 1), (16, 16, 12), (32, 16, 4)]:
        got = _run(H, c, tile, blocks=(2, 2, 2), streams=True)
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1], tile
    for tile in [(16, 16, 1), (16, 16, 24), (64, 8, 12)]:
        say("few waves, batch", tile)
        s = torch.cuda.Stream()
        ms = []
        for _ in range(2):
            h = H.Hydro(c.n, c.gamma, c.cfl, precision=H.FP64, stream=s)
            h.set_tile(*tile)
            h.set_primitive(c.W)
            ms.append(h)
        b = H.Batch(ms, use_graph=False)
        b.step(3)
        s.synchronize()
        for h in ms:
            assert np.array_equal(h.get_state(), ref[0]) and h.time() == ref[1], tile
        b.close()
