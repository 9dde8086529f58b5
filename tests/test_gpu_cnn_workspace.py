"""GPU: the single-layer weight gradient takes a workspace at any float
boundary (its argument checks ask for 16 bytes of dy and x only)."""
import pytest
import torch

from gpu_common import S
from paper_2003_06027_amd import cnn as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [4, 8, 12])
def test_weight_gradient_in_a_shifted_workspace(shift):
    n, h, w = 3, 21, 70
    gen = torch.Generator(device="cuda").manual_seed(shift)
    x, dy = (torch.randn(n, h, w, 32, generator=gen, device="cuda").bfloat16() for _ in range(2))
    nb = N.workspace_bytes(1, 1, 1)
    ws = torch.zeros(nb + 256, dtype=torch.uint8, device="cuda")
    out = []
    for o in (0, shift):
        dw = torch.empty(9 * 32 * 32 + 32, device="cuda")
        S._check(N.lib().cnn_conv3x3_wgrad(dy.data_ptr(), x.data_ptr(), n, h, w, dw.data_ptr(), ws.data_ptr() + o, nb,
                                           S._stream()))
        out.append(dw)
    assert float(out[0].abs().max()) > 0.0 and torch.equal(out[0], out[1])
