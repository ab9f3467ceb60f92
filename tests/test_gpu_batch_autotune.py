"""The batch autotuner on requests of two and three dimensions whose 3-D
members share a tile: what it leaves steps every member as if alone, bit for
bit, and it refuses a plan that the workspace cannot hold."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

# 48 and 80 default to 16 x 16, the others to 32 x 16 (mixed)
SIZES = [(48,) * 3, (64,) * 3, (80,) * 3, (32,) * 3, (224,) * 2, (96,) * 2, (352, 128), (64, 64)]


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


def _mesh(H, i, stream, precision):
    c = wl.turbulence_3d(n=SIZES[i], mach=0.6, seed=50 + i)
    h = H.Hydro(c.n, c.gamma, c.cfl, precision=precision, stream=stream)
    h.set_primitive(c.W)
    return h


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("graph", [False, True])
def test_autotuned_mix_equals_alone(H, precision, graph):
    import torch
    s = torch.cuda.Stream()
    say("batch autotune 2-D and 3-D", precision, graph)
    ms = [_mesh(H, i, s, precision) for i in range(len(SIZES))]
    b = H.Batch(ms, use_graph=graph)
    # members of the default tiles share launches
    assert b.info()["groups"] < len({(h.ndim, h.get_tile(1)[:2]) for h in ms})
    b.autotune(steps_per_rule=1)
    done, steps, flags = b.status()
    assert steps == [13] * len(ms) and not any(flags)
    b.step(3)
    b.status()
    b.step(3)
    s.synchronize()
    for i, h in enumerate(ms):
        a = _mesh(H, i, s, precision)
        a.step_auto(19)
        assert np.array_equal(a.get_state(), h.get_state()) and a.time() == h.time(), SIZES[i]
        a.close()
    b.close()


def test_refuses_tables_larger_than_the_workspace(H):
    import torch
    s = torch.cuda.Stream()
    say("batch autotune, a tile set after the workspace was sized")
    case = wl.turbulence_3d(n=(1024, 1024), mach=0.6, seed=70)

    def mesh():
        h = H.Hydro(case.n, case.gamma, case.cfl, precision=1, stream=s)
        h.set_primitive(case.W)
        return h

    h, alone = mesh(), mesh()
    b = H.Batch([h], use_graph=False)
    # a work-group per 64 x 1 cells: 16384 of them, where the default lengths
    # give the chip a round or two of them
    assert b.info()["workgroups"] * 2 < 16384
    h.set_tile(64, 1, 1)
    with pytest.raises(H.HydroError) as e:
        b.autotune(steps_per_rule=1)
    assert e.value.status == H.E_INVAL and h.steps_done() == 0
    b.step(2)
    alone.step_auto(2)
    s.synchronize()
    assert b.status()[1] == [2]
    assert np.array_equal(alone.get_state(), h.get_state())
    b.close()
