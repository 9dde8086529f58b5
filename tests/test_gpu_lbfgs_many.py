"""GPU: a direction whose chunks would take more threads than one launch holds
(2^32) is formed by one workgroup per model."""
import pytest
import torch

from gpu_common import S

pytestmark = pytest.mark.gpu


def test_more_chunks_than_a_launch_holds():
    B, n = 1 << 16, 1 << 17                    # 256 chunks of 512 elements per model, 256 threads each: 2^32
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GiB of device memory")
    v = torch.empty(B, n, device="cuda").uniform_(1.0, 2.0)
    p = torch.empty_like(v)
    vv = torch.cat([(c.double() ** 2).sum(1) for c in v.split(1024)])
    ysyy = torch.stack([vv, vv], -1)[None].contiguous()
    hist = torch.tensor([[1, 0]], dtype=torch.int32, device="cuda").repeat(B, 1).contiguous()
    # s = y = g: alpha = 1, q = g - y = 0, gamma = 1, beta = 0 and p = -s
    S._check(S.lib().lbfgs_direction(B, n, 1, S._ptr(hist), S._ptr(v), S._ptr(v), S._ptr(ysyy), S._ptr(v), S._ptr(p),
                                     S._stream()))
    # alpha and gamma are sums of 2^17 FP64 products in another order, applied in FP32 to elements below 2
    worst = max(float((a + b).abs().max()) for a, b in zip(p.split(1024), v.split(1024)))
    assert worst <= 4 * 2.0 ** -23
