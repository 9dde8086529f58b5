"""GPU: one layer on 4 x 32 tiles (an image alone: few tiles) and on 4 x 64 tiles
(the same image in a batch) gives the same values bit for bit."""
import numpy as np
import pytest
import torch

from paper_2003_06027_amd import cnn as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(9, 64), (4, 61), (30, 128), (7, 190), (5, 33), (6, 74), (1, 1)])
@pytest.mark.parametrize("extras", [False, True])
def test_image_alone_and_in_a_batch(h, w, extras):
    rng = np.random.default_rng(h * w)
    tiles = -(-h // 4) * -(-w // 64)
    n = 256 // tiles + 2                                  # more than 256 tiles of 64
    bf = lambda *s: torch.as_tensor(rng.standard_normal(s), dtype=torch.float32, device="cuda").bfloat16()
    x, wgt = bf(n, h, w, 32), bf(32, 9, 32) * 0.1
    bias = torch.as_tensor(rng.standard_normal(32), dtype=torch.float32, device="cuda")
    kw = dict(bias=bias, relu=True, want_fp32=True)
    if extras:
        kw.update(res=bf(n, h, w, 32), gate=bf(n, h, w, 32))
    one = {k: (v[:1].contiguous() if k in ("res", "gate") else v) for k, v in kw.items()}
    yb, yb32 = N.conv3x3(x, wgt, **kw)
    y1, y132 = N.conv3x3(x[:1].contiguous(), wgt, **one)
    assert float(yb32.abs().max()) > 0.0
    assert torch.equal(yb[:1].view(torch.int16), y1.view(torch.int16))
    assert torch.equal(yb32[:1], y132)
