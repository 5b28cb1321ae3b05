"""Network inputs of 4^3 blocks, whose patches are single cells (four blocks a
work-group): list lengths around the group's, against the oracle."""
import numpy as np
import pytest

from oracle import mlp
from synthetic import as_dict, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [(1, 1, 1), (3, 1, 1), (4, 1, 1), (5, 1, 1), (7, 3, 3)])
@pytest.mark.parametrize("tracer", [False, True])
def test_features(blocks, tracer):
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=tuple(4 * b for b in blocks), block=(4, 4, 4))
    sim = ic.Sim(grid, as_dict(w.wind), [], tracer=tracer)
    bl, U = sim.state()
    U = U * np.random.default_rng(len(bl)).uniform(0.9999, 1.0001, U.shape)
    sim.set_state(bl, U)
    ref = np.stack([mlp.features(u[:8], grid["gamma"]) for u in U])
    np.testing.assert_allclose(sim.features(), ref, rtol=3e-7, atol=1e-12)      # one float32 rounding
    sim.close()
