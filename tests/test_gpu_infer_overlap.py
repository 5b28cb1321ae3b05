"""Allocation-free inference whose probabilities lie on its inputs (a caller
that is done with them): the bits of the call with an array of its own, on
every position that reaches another row, and nothing written beside them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _net(seed):
    import paper_2211_12867_amd as ic
    g = np.random.default_rng(seed)
    mean = g.uniform(-1.0, 1.0, ic.MLP_IN).astype(np.float32)
    std = g.uniform(0.5, 2.0, ic.MLP_IN).astype(np.float32)
    return ic.mlp_init(seed).astype(np.float32), mean, std


def _call(buf, at, n):
    """The call with its arrays in one buffer at the given offsets (floats)."""
    import torch
    import paper_2211_12867_amd as ic
    p = buf.data_ptr()
    ic.mlp_infer_noalloc(p + 4 * at["raw"], n, p + 4 * at["params"], p + 4 * at["mean"], p + 4 * at["std"],
                         p + 4 * at["prob"])
    torch.cuda.synchronize()


# where prob begins, in floats from the start of an array (negative: before it)
@pytest.mark.parametrize("n", [1, 16, 17, 700, 4096])
@pytest.mark.parametrize("on,where", [("raw", 0), ("raw", 1), ("raw", 511), ("raw", -1), ("raw", "middle"),
                                      ("raw", "last"), ("raw", "end"), ("mean", 0), ("std", 5), ("std", -1),
                                      ("params", 0), ("params", "last")])
def test_prob_on_inputs(n, on, where):
    import torch
    import paper_2211_12867_amd as ic
    params, mean, std = _net(7)
    g = np.random.default_rng(n)
    raw = (g.standard_normal((n, ic.MLP_IN)) * 1.5 + 0.3).astype(np.float32)
    ref = ic.mlp_infer(raw, params, mean, std)
    size = dict(raw=raw.size, params=params.size, mean=mean.size, std=std.size)
    data = dict(raw=raw.ravel(), params=params, mean=mean, std=std)
    # the array that prob lies on first, with room for prob around it
    at, end = {}, 4096 + 4
    for k in [on] + [k for k in size if k != on]:
        at[k] = end
        end += size[k] + 4096 + 4
    host = g.standard_normal(end).astype(np.float32)
    for k in size:
        host[at[k]:at[k] + size[k]] = data[k]
    off = {"middle": size[on] // 2 + 3, "last": size[on] - 1, "end": size[on]}.get(where, where)
    at["prob"] = at[on] + off
    buf = torch.from_numpy(host).cuda()
    _call(buf, at, n)
    want = host.copy()
    want[at["prob"]:at["prob"] + n] = ref
    assert np.array_equal(buf.cpu().numpy(), want)
