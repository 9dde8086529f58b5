"""GPU: directions of many models.  Few models of a size take the products over
the whole chip, many one workgroup each; a direction whose chunks would take
more threads than one launch holds (2^32) is formed by one workgroup per model."""
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
    del v, p
    torch.cuda.empty_cache()
    assert worst <= 4 * 2.0 ** -23


@pytest.mark.parametrize("n,mem,few,many", [(8000, 2, 20, 400), (2000, 5, 1, 1500), (20000, 1, 10, 120)])
def test_few_and_many_models(n, mem, few, many):
    gen = torch.Generator(device="cuda").manual_seed(n)
    new = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    Sh = new(mem, many, n)
    Y = (1.0 + new(many, n).abs()) * Sh + 0.3 * new(mem, many, n)
    g = new(many, n)
    out = []
    for B in (few, many):
        s, y, gb = Sh[:, :B].contiguous(), Y[:, :B].contiguous(), g[:B].contiguous()
        ysyy = torch.stack([(y.double() * s.double()).sum(-1), (y.double() ** 2).sum(-1)], -1).contiguous()
        hist = torch.tensor([[mem, mem - 1]], dtype=torch.int32, device="cuda").repeat(B, 1).contiguous()
        p = torch.empty_like(gb)
        S._check(S.lib().lbfgs_direction(B, n, mem, S._ptr(hist), S._ptr(s), S._ptr(y), S._ptr(ysyy), S._ptr(gb),
                                         S._ptr(p), S._stream()))
        out.append(p)
    q, al = g[:few].double(), [None] * mem                  # the two-loop recursion in 64 bits
    s, y = Sh[:, :few].double(), Y[:, :few].double()
    ys = (y * s).sum(-1, keepdim=True)
    for j in range(mem - 1, -1, -1):
        al[j] = (s[j] * q).sum(-1, keepdim=True) / ys[j]
        q = q - al[j] * y[j]
    q = q * ys[-1] / (y[-1] ** 2).sum(-1, keepdim=True)
    for j in range(mem):
        q = q + (al[j] - (y[j] * q).sum(-1, keepdim=True) / ys[j]) * s[j]
    for p in out:                                           # FP32 vectors, FP64 inner products
        assert float((p[:few].double() + q).norm() / q.norm()) <= 1e-5
