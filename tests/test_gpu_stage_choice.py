"""Which stage kernel the steps launch (Sim.stage_planes): the rule at its lines
on the device of the test (256 compute units), a set schedule, and a schedule
that ic_autotune measured or read from its cache -- the one it reports is the
one that runs, and entries without the short-list kernel's mark name the
marching kernel."""
import numpy as np
import pytest

from synthetic import as_dict, workload
from test_gpu_short_lists import SHAPES

pytestmark = pytest.mark.gpu


def _sim(block, n):
    import paper_2211_12867_amd as ic
    w = workload("tiny_wedge")
    return ic.Sim(dict(as_dict(w.grid), n=n, block=block), as_dict(w.wind), [as_dict(w.cmes[0])])


def _planes(block, n):
    sim = _sim(block, n)
    got = sim.stage_planes()
    sim.set_tuning(2, 0, 0, 1)
    assert sim.stage_planes() == 0
    sim.close()
    return got


@pytest.fixture
def cu256():
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lists are sized for 256 compute units")


def test_lists_of_the_bit_comparison(cu256):
    assert [_planes(*c) for c in SHAPES] == [1, 2, 4, 1, 2, 4, 1, 2, 4, 1, 2, 4, 1, 2]


@pytest.mark.parametrize("block,blocks,planes", [
    ((12, 12, 12), (7, 3, 1), 1), ((12, 12, 12), (11, 2, 1), 2),          # 21 blocks x 12 planes, 22
    ((12, 12, 12), (7, 6, 1), 2), ((12, 12, 12), (43, 1, 1), 4),          # 42 x 6, 43
    ((12, 12, 12), (31, 11, 1), 4), ((12, 12, 12), (19, 18, 1), 0),       # 341 x 3, 342
    ((12, 8, 12), (31, 11, 1), 4), ((12, 8, 12), (19, 18, 1), 0),
    ((8, 8, 8), (32, 16, 1), 4), ((8, 8, 8), (27, 19, 1), 0),             # 512 x 2, 513
    ((16, 12, 12), (7, 6, 1), 2), ((16, 12, 12), (43, 1, 1), 0),          # no four planes of 192 cells
    ((4, 4, 4), (40, 32, 4), 4),
])
def test_lines_of_the_rule(cu256, block, blocks, planes):
    assert _planes(block, tuple(b * n for b, n in zip(block, blocks))) == planes


def test_tuned_schedules(tmp_path):
    block, n = (12, 12, 12), (60, 24, 48)                # 40 blocks
    ref = _sim(block, n)
    rule = ref.stage_planes()
    assert rule > 0
    ref.advance(1e9, max_steps=6)
    U = ref.state()[1]
    ref.close()
    cache = tmp_path / "tune.txt"
    sim = _sim(block, n)
    r = sim.autotune(str(cache), reps=2)
    tuned = (r["waves_per_simd"], r["grid"], r["xcd_order"], r["ksplit"])
    assert r["from_cache"] == 0 and sim.tuning() == tuned and sim.stage_planes() in (0, rule)
    line = cache.read_text().split()
    assert line[0].endswith("/tile") == (sim.stage_planes() > 0)
    again = _sim(block, n)
    assert again.autotune(str(cache))["from_cache"] == 1
    assert again.tuning() == tuned and again.stage_planes() == sim.stage_planes()
    sim.close()
    again.close()
    key = line[0][:-len("/tile")] if line[0].endswith("/tile") else line[0]
    for mark, planes in (("", 0), ("/tile", rule)):
        cache.write_text("%s%s 2 0 0 4 0.020000 0.050000\n" % (key, mark))
        sim = _sim(block, n)
        assert sim.autotune(str(cache))["from_cache"] == 1
        assert sim.tuning() == (2, 0, 0, 4) and sim.stage_planes() == planes
        sim.advance(1e9, max_steps=6)
        assert np.array_equal(sim.state()[1], U)
        sim.set_tuning(2, 0, 0, 2)
        assert sim.stage_planes() == 0
        sim.autotune(str(cache))
        assert sim.stage_planes() == planes
        sim.close()


def test_choice_follows_the_work_list():
    """Between a tuned size and others: the rule again where nothing was measured."""
    import paper_2211_12867_amd as ic
    w = workload("learned_flags")
    sim = ic.Sim(dict(as_dict(w.grid), max_level=2), as_dict(w.wind), [as_dict(w.cmes[0])], as_dict(w.amr),
                 max_blocks=1024)
    rule = sim.stage_planes()
    sim.autotune(reps=1)
    tuned = sim.stage_planes()
    assert rule > 0 and tuned in (0, rule)
    sim.regrid([np.ones(len(sim.blocks()), np.int8)])
    assert len(sim.blocks()) == 320 and sim.stage_planes() == 4
    sim.regrid([np.full(len(sim.blocks()), -1, np.int8)])
    assert len(sim.blocks()) == 40 and sim.stage_planes() == tuned
    sim.close()
