"""Steps enqueued together (the next step's dt set by the launch that ends a
step) and one by one give the same bits: states, clocks, dt and samples, with
members that reach their end time between them, a point outside the domain, a
fixed dt, and a box without any ghost slab."""
import numpy as np
import pytest

from synthetic import as_dict, workload

pytestmark = pytest.mark.gpu


def _wedge(members, **opt):
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=(24, 8, 16), block=(8, 8, 8))
    cme = as_dict(w.cmes[0])
    return ic.Sim(grid, as_dict(w.wind), [dict(cme, v_kms=700.0 + 300.0 * m) for m in range(members)], **opt)


@pytest.mark.parametrize("members,outside,opt", [(1, False, {}), (3, False, dict(scheme="hancock")),
                                                 (2, True, dict(divb_cd=0.1)), (1, False, dict(tracer=True))])
def test_together_and_one_by_one(members, outside, opt):
    out = []
    for together in (True, False):
        sim = _wedge(members, **opt)
        if outside:
            sim.set_sample_point(50.0, 90.0, 0.0)
        if together:
            sim.advance(1e9, max_steps=13)        # two replays of five steps, three of one
        else:
            for _ in range(13):
                sim.step()
        out.append(([sim.state(m)[1] for m in range(members)], [sim.time(m) for m in range(members)],
                    [sim.timeseries(m) for m in range(members)]))
        sim.close()
    (Ua, ta, sa), (Ub, tb, sb) = out
    assert ta == tb
    for a, b in zip(Ua + sa, Ub + sb):
        assert np.isfinite(a).all() and np.array_equal(a, b)
    assert len(sa[0]) == (0 if outside else 13)


def test_members_end_between_steps():
    """An end time that the members reach in the middle of a replay: each member's samples end there, as in
    a sim of its own that is advanced by what is left, a step a call."""
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    grid = dict(as_dict(w.grid), n=(24, 8, 16), block=(8, 8, 8))
    a = _wedge(2)
    end = 7.5 * a.step()["dt_s"]
    start = [a.time(m)[0] for m in range(2)]
    a.advance(end)
    for m in range(2):
        b = ic.Sim(grid, as_dict(w.wind), [dict(as_dict(w.cmes[0]), v_kms=700.0 + 300.0 * m)])
        b.step()
        while start[m] + end - b.time()[0] > 1e-9 * end:
            b.advance(start[m] + end - b.time()[0], max_steps=1)
        np.testing.assert_allclose(a.timeseries(m), b.timeseries(), rtol=1e-9, atol=1e-12)
        np.testing.assert_allclose(a.state(m)[1], b.state()[1], rtol=1e-9, atol=1e-12)
        b.close()
    a.close()


def test_fixed_dt_and_no_slabs():
    import paper_2211_12867_amd as ic
    grid = dict(geometry="cartesian", x0=(0.0, 0.0, 0.0), x1=(1.0, 1.0, 1.0), n=(8, 8, 16), block=(8, 8, 8),
                stretched_r=False, max_level=1, periodic=(True, True, True), gamma=1.5, cfl=0.4)
    w = workload("tiny_wedge")
    sims = [ic.Sim(grid, as_dict(w.wind), []) for _ in range(2)]
    g = np.random.default_rng(2)
    b, U = sims[0].state()
    U = np.ones_like(U)
    U[:, 1:4] = 0.1 * g.standard_normal(U[:, 1:4].shape)
    U[:, 4] = 5.0
    U[:, 5:8] = 0.05
    for s in sims:
        s.set_state(b, U)
    sims[0].advance(1e9, max_steps=6)
    for _ in range(6):
        sims[1].step()
    assert np.array_equal(sims[0].state()[1], sims[1].state()[1]) and sims[0].time() == sims[1].time()
    t0 = sims[0].time()[0]
    sims[0].step(12.0)
    assert abs(sims[0].time()[0] - t0 - 12.0) < 1e-6
    for s in sims:
        s.close()
