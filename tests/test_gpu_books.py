"""The time step's books where a call hands them over: from replays of a
captured graph to eager calls, and from one launch of a 1-D run to the next.
Everything against the same steps launched eagerly, bit for bit."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


def _mesh(H, n, stream, precision=0, blocks=None, integrator=0):
    c = wl.turbulence_3d(n=n, mach=0.6, seed=21)
    h = H.Hydro(c.n, c.gamma, c.cfl, precision=precision, stream=stream, blocks=blocks, integrator=integrator)
    h.set_primitive(c.W)
    return h


def _same(a, b):
    return a.time() == b.time() and a.steps_done() == b.steps_done() and np.array_equal(a.get_state(), b.get_state())


def _busy():
    import torch
    torch.ones(1 << 20, device="cuda").mul_(2.0)
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,blocks", [((200,), None), ((70, 44), None), ((16, 16, 16), (2, 1, 2))])
@pytest.mark.parametrize("ask", [False, True])
def test_host_step_replayed_then_eager(H, n, blocks, ask):
    """ask: the captured step is one that leaves its state's rate pending."""
    import torch
    say("host step replayed", n, blocks, ask)
    s = torch.cuda.Stream()
    h, ref = _mesh(H, n, s, blocks=blocks), _mesh(H, n, s, blocks=blocks)
    dt = 0.3 * ref.cfl_dt()
    if ask:
        h.cfl_dt()
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        h.step(dt)
    for r in range(3):
        for _ in range(r + 1):
            g.replay()
            ref.step(dt)
        _busy()
        assert h.cfl_dt() == ref.cfl_dt(), r
    g.replay()
    ref.step(dt)
    h.step_auto(3)
    ref.step_auto(3)
    assert _same(h, ref)
    if blocks:
        g.replay()
        ref.step(dt)
        h.set_block_streams(True)
        h.step_auto(3)
        ref.step_auto(3)
        assert _same(h, ref)
    g.replay()
    ref.step(dt)
    if not blocks:
        b = H.Batch([h], use_graph=False)
        b.step(2)
        s.synchronize()
        b.close()
        ref.step_auto(2)
    assert h.cfl_dt() == ref.cfl_dt() and _same(h, ref)
    del g
    h.close()
    ref.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("integrator", [0, 1])
def test_1d_run_replayed(H, precision, integrator):
    import torch
    say("1-D run replayed", precision, integrator)
    s = torch.cuda.Stream()
    h = _mesh(H, (300,), s, precision, integrator=integrator)
    ref = _mesh(H, (300,), s, precision, integrator=integrator)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        h.step_auto(5)
    for _ in range(3):
        g.replay()
        _busy()
        ref.step_auto(5)
        assert _same(h, ref)
    h.step_auto(2)
    ref.step_auto(2)
    assert _same(h, ref)
    del g
    h.close()
    ref.close()


def test_1d_run_of_more_steps_than_a_launch(H):
    """4097 steps in one call: two launches; the reference launches stages
    (stage timing is on)."""
    import torch
    say("1-D run of 4097 steps")
    s = torch.cuda.Stream()
    h, ref = _mesh(H, (64,), s), _mesh(H, (64,), s)
    ref.profile(1)
    h.step_auto(4097)
    ref.step_auto(4097)
    assert _same(h, ref) and h.steps_done() == 4097
    h.close()
    ref.close()
