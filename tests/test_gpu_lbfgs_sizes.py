"""GPU: the L-BFGS direction and pair update at the sizes where their kernels
change (one workgroup or the whole chip, chunk and head edges, odd lengths,
histories below and above the products' limit) against the FP64 oracle:
FP32 vectors, FP64 inner products, rel-L2 <= 1e-5 as for the batched loop."""
import numpy as np
import pytest
import torch

from gpu_common import S, rel_l2, dev
from oracle import lbfgs as LB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n,mem,counts", [
    (2, 1, 1, (1, 0)),
    (3, 749, 8, (8, 3, 0)),            # last length of the one-workgroup loop at 8 pairs
    (3, 750, 8, (8, 1, 0)),            # first length of the products
    (2, 1025, 5, (5, 2)),
    (2, 3001, 5, (5, 2)),
    (2, 1023, 15, (15, 1)),            # no room for two chunks' partial sums
    (2, 1024, 15, (15, 1)),            # just enough
    (4, 10201, 8, (8, 7, 0, 1)),
    (1, 16385, 12, (12,)),             # pair formed by many workgroups
    (2, 3001, 15, (15, 4)),            # the most pairs the products take
    (2, 3001, 16, (16, 4)),            # and one more
    (1, 300007, 10, (9,)),
])
def test_pair_and_direction(B, n, mem, counts):
    rng = np.random.default_rng(n)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    curv = 1.0 + np.abs(f(n))
    Sh = f(mem, B, n)
    Yh = (curv * Sh + 0.3 * f(mem, B, n)).astype(np.float32)
    m_old, g_old = f(B, n), f(B, n)
    m_new = m_old + 0.1 * f(B, n)
    g_new = (g_old + curv * (m_new - m_old) + 0.01 * f(B, n)).astype(np.float32)
    ysyy = np.stack([(Yh.astype(np.float64) * Sh).sum(-1), (Yh.astype(np.float64) ** 2).sum(-1)], -1)
    newest = [(3 * b + 1) % mem for b in range(B)]
    slot = np.array([newest[b] if counts[b] else -1 for b in range(B)], np.int32)
    hist = np.array([[counts[b], newest[b]] for b in range(B)], np.int32)
    d = [dev(slot, torch.int32), dev(m_new), dev(m_old), dev(g_new), dev(g_old), dev(Sh), dev(Yh),
         dev(ysyy, torch.float64), dev(hist, torch.int32)]
    S._check(S.lib().lbfgs_push(B, n, mem, *[S._ptr(t) for t in d[:8]], S._stream()))
    p = torch.full((B, n), float("nan"), device="cuda")
    S._check(S.lib().lbfgs_direction(B, n, mem, S._ptr(d[8]), S._ptr(d[5]), S._ptr(d[6]), S._ptr(d[7]), S._ptr(d[3]),
                                     S._ptr(p), S._stream()))
    Sd, Yd, yd = (t.cpu().numpy() for t in d[5:8])
    for b in range(B):
        if counts[b]:
            k = newest[b]
            np.testing.assert_array_equal(Sd[k, b], m_new[b] - m_old[b])
            np.testing.assert_array_equal(Yd[k, b], g_new[b] - g_old[b])
            s, y = Sd[k, b].astype(np.float64), Yd[k, b].astype(np.float64)
            assert yd[k, b, 0] == pytest.approx(float(y @ s), rel=1e-12)
            assert yd[k, b, 1] == pytest.approx(float(y @ y), rel=1e-12)
        others = [j for j in range(mem) if not (counts[b] and j == newest[b])]
        np.testing.assert_array_equal(Sd[others, b], Sh[others, b])
        np.testing.assert_array_equal(yd[others, b], ysyy[others, b])
        order = [(newest[b] - j) % mem for j in range(counts[b])][::-1]
        want = LB.two_loop(g_new[b], [Sd[k, b] for k in order], [Yd[k, b] for k in order])
        assert rel_l2(p[b].cpu().numpy(), want) <= 1e-5, b
    again = torch.empty_like(p)
    S._check(S.lib().lbfgs_direction(B, n, mem, S._ptr(d[8]), S._ptr(d[5]), S._ptr(d[6]), S._ptr(d[7]), S._ptr(d[3]),
                                     S._ptr(again), S._stream()))
    assert torch.equal(again, p)
