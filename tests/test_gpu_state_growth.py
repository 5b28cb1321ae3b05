"""States in and out of a sim whose forest grows and shrinks between the
exchanges: a pinned area smaller than the state (several parts), then larger
ones; every exchange exact."""
import numpy as np
import pytest

from synthetic import as_dict, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,n,tracer", [((4, 4, 4), (8, 4, 8), False), ((12, 12, 12), (12, 12, 12), True),
                                            ((8, 8, 8), (16, 8, 16), False)])
def test_growing_forest(block, n, tracer):
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=n, block=block, max_level=4)
    sim = ic.Sim(grid, as_dict(w.wind), [], dict(regrid_every=0, buffer_blocks=0), max_blocks=4096, tracer=tracer)
    g = np.random.default_rng(3)

    def exchange():
        b, U = sim.state()
        V = U * g.uniform(0.9999, 1.0001, U.shape)
        order = g.permutation(len(b))
        sim.set_state([b[q] for q in order], V[order])
        b2, V2 = sim.state()
        assert b2 == b and np.array_equal(V, V2)

    def refine(share):
        """User flags for a share of the leaves (the 2:1 rule adds more)."""
        f = np.where(np.arange(len(sim.blocks())) < share * len(sim.blocks()), 1, 0).astype(np.int8)
        sim.regrid([f])

    sizes = []
    for share in (0, 0, 0, 0.5, 0.2, 1.0, 0.1, 0.3, 1.0):
        if share:
            refine(share)
        sizes.append(len(sim.blocks()))
        exchange()
    assert sizes[-1] > 30 * sizes[0]
    for _ in range(3):
        sim.regrid([np.full(len(sim.blocks()), -1, np.int8)])
        exchange()
    sim.close()
