"""The marching stage kernels in chunks of every length down to one plane, and
in the automatic length, give the same state bit for bit."""
import numpy as np
import pytest

from paper_2501_02317_amd import workloads as wl

from gpu_util import say

pytestmark = pytest.mark.gpu

PER, FREE, OUT, REF = 0, 1, 2, 3
CASES = [  # n, boundaries, blocks: extents at, just past and below tiles, chunks and two planes
    ((96, 5), ((REF, REF), (PER, PER)), None),
    ((257, 63), ((PER, PER), (OUT, REF)), None),
    ((33, 17, 21), ((PER, PER), (FREE, OUT), (REF, OUT)), None),
    ((48, 48, 7), ((PER, PER),) * 3, None),
    ((32, 16, 24), ((PER, PER), (OUT, FREE), (PER, PER)), (2, 1, 4)),
]


@pytest.fixture(scope="module")
def H():
    from paper_2501_02317_amd import hydro
    return hydro


@pytest.mark.parametrize("n,bc,blocks", CASES)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("integrator", [0, 1])
def test_results_independent_of_chunk_length(H, n, bc, blocks, precision, integrator):
    c = wl.turbulence_3d(n=n, mach=0.7, seed=5)
    ref = None
    for kz in (16, 0, 1, 2, 3, 5):
        say("chunk", n, precision, integrator, kz)
        h = H.Hydro(n, 1.4, 0.3, precision=precision, bc=bc, integrator=integrator, blocks=blocks)
        for stage in (1, 2):
            tx, ty, _ = h.get_tile(stage)
            h.set_tile(tx, ty, kz, stage=stage)
        h.set_primitive(c.W)
        h.step_auto(3)
        U = h.get_state()
        t = h.time()
        h.close()
        if ref is None:
            ref = (U, t)
        assert np.isfinite(U).all() and np.array_equal(U, ref[0]) and t == ref[1], kz
