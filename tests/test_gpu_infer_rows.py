"""Inference at the edges of its 16-row tiles and of its grid (one work-group
per tile up to 256, several tiles a group beyond): the raw-input launch, the
bf16-input launch and the reference network agree."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4096, 4097, 4096 + 16 * 256 + 5])
def test_rows(n):
    import torch
    import paper_2211_12867_amd as ic
    from oracle import mlp
    g = np.random.default_rng(n)
    p = ic.mlp_init(11).astype(np.float32)
    mean = g.uniform(-1.0, 1.0, ic.MLP_IN).astype(np.float32)
    std = g.uniform(0.5, 2.0, ic.MLP_IN).astype(np.float32)
    raw = (g.standard_normal((n, ic.MLP_IN)) * 1.5 + 0.3).astype(np.float32)
    prob = ic.mlp_infer(raw, p, mean, std)
    tp, tm, ts = (torch.from_numpy(a).cuda() for a in (p, mean, std))
    for off in (0, 1):                            # the input array 16-byte aligned, and 4 bytes off
        for a in range(0, n, ic.MLP_NOALLOC_ROWS):
            part = raw[a:a + ic.MLP_NOALLOC_ROWS]
            buf = torch.zeros(off + part.size, device="cuda")
            buf[off:] = torch.from_numpy(part.ravel()).cuda()
            out = torch.full((len(part) + 1,), -1.0, device="cuda")
            ic.mlp_infer_noalloc(buf.data_ptr() + 4 * off, len(part), tp.data_ptr(), tm.data_ptr(), ts.data_ptr(),
                                 out.data_ptr())
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            assert np.array_equal(got[:-1], prob[a:a + len(part)]) and got[-1] == -1.0
    # every value is rounded at the reference's points; sums of at most 512 products of size about 0.1 differ by
    # their order (1e-5), which moves a hidden value by a bf16 step (2^-9 of it) now and then: 1e-2 in the logit
    x = (raw - mean) * (np.float32(1.0) / std)
    rows = slice(max(0, n - 64), n)
    z = mlp.forward(x[rows], p)[0]
    assert np.abs(prob[rows] - 1.0 / (1.0 + np.exp(-z.astype(np.float64)))).max() < 0.25 * 1e-2
