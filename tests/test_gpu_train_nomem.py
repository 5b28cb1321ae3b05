"""Training and gradients whose device memory runs out at any of their
allocations: an error, every buffer given back, and none while the device still
works on it (the caller's allocator may hand it out again at once)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class Allocator:
    """Device memory from torch; the allocation number `fail` fails.  Nothing is
    really given back before the end of the test."""

    def __init__(self, ic, fail):
        import torch
        self.fail, self.held, self.all, self.n, self.busy = fail, {}, [], 0, 0

        def alloc(size, user):
            self.n += 1
            if self.n == self.fail:
                return None
            t = torch.empty(size, dtype=torch.uint8, device="cuda")
            self.all.append(t)
            self.held[t.data_ptr()] = t
            return t.data_ptr()

        def release(p, user):
            self.busy += not torch.cuda.default_stream().query()
            del self.held[p]

        self.fns = ic._ALLOC_FN(alloc), ic._FREE_FN(release)
        assert ic.lib.ic_set_device_allocator(*self.fns, None) == 0


@pytest.mark.parametrize("call", ["train", "grad", "infer"])
def test_allocation_fails(call):
    import torch
    import paper_2211_12867_amd as ic
    n = 40000 if call == "train" else 2000
    g = np.random.default_rng(1)
    raw = g.standard_normal((n, ic.MLP_IN)).astype(np.float32)
    y = (g.random(n) < 0.3).astype(np.uint8)
    p = ic.mlp_init(1).astype(np.float32)
    one, zero = np.ones(ic.MLP_IN, np.float32), np.zeros(ic.MLP_IN, np.float32)
    run = dict(train=lambda: ic.mlp_train(raw, y, p, epochs=1, batch=4096), grad=lambda: ic.mlp_grad(raw, y, p, 1.0),
               infer=lambda: ic.mlp_infer(raw, p, zero, one))[call]
    torch.zeros(1, device="cuda")
    try:
        a = Allocator(ic, 0)
        run()
        assert not a.held and a.n > 3
        for k in range(1, a.n + 1):
            b = Allocator(ic, k)
            with pytest.raises(ic.ICError):
                run()
            assert b.n >= k and not b.held and b.busy == 0, k
            torch.cuda.synchronize()
    finally:
        ic.use_torch_allocator(False)
