"""GPU: the reductions of the weight gradients that ride in the next launch,
with room for them in its grid and without (65535 images): images whose output
gradient is zero change no parameter gradient, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2003_06027_amd import cnn as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w", [(3, 2, 2), (65500, 2, 2), (65535, 2, 2), (40, 5, 67)])
def test_images_without_gradient(n, h, w):
    k = min(n, 3)
    rng = np.random.default_rng(5)
    g = torch.zeros(n, h, w, device="cuda")
    dp = torch.zeros_like(g)
    g[:k] = torch.as_tensor(rng.standard_normal((k, h, w)), dtype=torch.float32)
    g[k:] = 0.25
    dp[:k] = torch.as_tensor(rng.standard_normal((k, h, w)), dtype=torch.float32)
    params = torch.as_tensor(N.init_params(2), dtype=torch.float32, device="cuda")
    out = []
    for m in (n, k):
        ws = N.new_workspace(m, h, w)
        N.forward(params, g[:m].contiguous(), ws)
        out.append(N.backward(params, g[:m].contiguous(), dp[:m].contiguous(), ws))
        out.append(N.backward(params, g[:m].contiguous(), dp[:m].contiguous(), ws))
    assert torch.isfinite(out[0]).all() and float(out[0].abs().max()) > 0.0
    for o in out[1:]:
        assert torch.equal(o, out[0])
