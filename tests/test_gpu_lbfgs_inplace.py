"""GPU: lbfgs_push forms a pair apart from its inputs or in place, in history
slots that hold a model and a gradient (elementwise differences), at the ends
of a workgroup's runs of elements and below and above the length from which
several workgroups share a pair."""
import pytest
import torch

from gpu_common import S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1024, 3073, 4096, 4097, 16384, 16385, 20000, 24576, 24577, 32768, 32769, 40001])
@pytest.mark.parametrize("where", ["old", "new", "apart"])
def test_pair_in_place(n, where):
    mem, k = 3, 1
    gen = torch.Generator(device="cuda").manual_seed(n)
    new = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    m_new, m_old, g_new, g_old = (new(1, n) for _ in range(4))
    Sh, Y = new(mem, 1, n), new(mem, 1, n)
    ysyy = torch.zeros(mem, 1, 2, dtype=torch.float64, device="cuda")
    s, y = m_new - m_old, g_new - g_old
    a = [m_new, m_old, g_new, g_old]
    for i, h in {"old": ((1, Sh), (3, Y)), "new": ((0, Sh), (2, Y)), "apart": ()}[where]:
        h[k] = a[i]
        a[i] = h[k]
    keep = Sh[::2].clone(), Y[::2].clone()
    slot = torch.tensor([k], dtype=torch.int32, device="cuda")
    S._check(S.lib().lbfgs_push(1, n, mem, *[S._ptr(t) for t in [slot] + a + [Sh, Y, ysyy]], S._stream()))
    assert torch.equal(Sh[k], s) and torch.equal(Y[k], y)
    assert torch.equal(Sh[::2], keep[0]) and torch.equal(Y[::2], keep[1])
    want = torch.stack([(y.double() * s.double()).sum(), (y.double() ** 2).sum()])
    assert float((ysyy[k, 0, 1] - want[1]).abs() / want[1]) <= 1e-12
    # y.s cancels: n products of about 1 rounded at 2^-53, summed in another order
    assert float((ysyy[k, 0, 0] - want[0]).abs()) <= 1e-12 * float((y.double() * s.double()).abs().sum())
