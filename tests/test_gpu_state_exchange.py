"""States in and out of the pool, which pass in parts of up to 8 MB staged in
turn: one block, one part, several with a ragged last one, blocks given in any
order, an exchange that outgrows the one before; and the sample ring read after
it wrapped."""
import numpy as np
import pytest

from synthetic import as_dict, workload

pytestmark = pytest.mark.gpu


def _sim(n, block, tracer=False):
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=n, block=block)
    return ic.Sim(grid, as_dict(w.wind), [], tracer=tracer)


@pytest.mark.parametrize("n,block,tracer", [
    ((4, 4, 4), (4, 4, 4), False),               # one block of 4 KB
    ((12, 12, 12), (12, 12, 12), True),
    ((48, 36, 48), (12, 12, 12), False),         # 48 blocks: one part
    ((72, 48, 72), (12, 12, 12), False),         # 144 of 111 KB, 75 a part: two, the second ragged
    ((96, 48, 96), (16, 12, 12), True),          # 192 of 166 KB, 50 a part: four
    ((96, 64, 96), (4, 4, 4), False),            # 9,216 of 4 KB, 2,048 a part
])
def test_round_trip(n, block, tracer):
    sim = _sim(n, block, tracer)
    b0, U0 = sim.state()                         # the first exchange
    g = np.random.default_rng(len(b0))
    U = U0 * g.uniform(0.999, 1.001, U0.shape)
    order = g.permutation(len(b0))
    sim.set_state([b0[q] for q in order], U[order])
    b1, U1 = sim.state()
    assert b1 == b0 and np.array_equal(U1, U)
    sim.set_state(b0, U0)
    assert np.array_equal(sim.state()[1], U0)
    sim.close()


def test_small_then_large():
    """A refining sim whose later state needs a larger staging area than its first."""
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=(24, 12, 24), block=(4, 4, 4), max_level=2)
    sim = ic.Sim(grid, as_dict(w.wind), [], dict(regrid_every=10, buffer_blocks=0), max_blocks=4096)
    b0, U0 = sim.state()
    sim.regrid([np.ones(len(b0), np.int8)])
    b1, U1 = sim.state()
    assert len(b1) == 8 * len(b0)
    sim.set_state(b1, 1.0001 * U1)
    assert np.array_equal(sim.state()[1], 1.0001 * U1)
    sim.close()


def test_ring_wraps():
    """The sample ring holds 65,536 records; later ones replace the oldest."""
    sim = _sim((8, 4, 8), (4, 4, 4))
    sim.advance(1e12, max_steps=65500)
    a = sim.timeseries()
    sim.advance(1e12, max_steps=100)
    b = sim.timeseries()
    assert len(a) == 65500 and len(b) == 65536
    assert np.array_equal(b[:-100], a[64:])      # 65,600 records: the first 64 are gone
    assert np.all(np.diff(b[:, 0]) > 0.0)
    assert np.array_equal(sim.timeseries(cap=70), b[-70:])     # the wrap (record 65,536) inside: 64 after it
    sim.close()
