"""GPU: a 2-D acoustic step launched as one grid gives the seismograms, the
model gradient and the wavelet gradient of its tile lists launched apart, bit
for bit: few tiles (every list in one grid, 8 or 16 rows per workgroup) and
many (the other one-step tiles apart), one- and two-step launches, one source
and several nodes per shot, receivers at depth, no layer."""
import numpy as np
import pytest
import torch

from gpu_common import S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("two", [1, 2])
@pytest.mark.parametrize("nx,nz,P,shots,nsrc,deep", [
    (260, 160, 20, 1, 5, True),        # 8 rows, all three lists, source nodes
    (300, 170, 16, 8, 1, True),        # 16 rows
    (420, 270, 20, 8, 1, True),        # whole tiles, others apart
    (420, 270, 20, 8, 3, False),
    (200, 130, 0, 2, 2, False),        # no tiles by the layer
    (101, 90, 20, 2, 1, True),         # none away from it
])
def test_one_grid_equals_lists_apart(nx, nz, P, shots, nsrc, deep, two):
    nt, K = 33, 8
    c = 1700.0 + 1500.0 * synth.smooth_random(13, (nz, nx), 6.0, 0.0, 1.0)
    d = S.desc(ndim=2, nx=nx, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=3200.0)
    rng = np.random.default_rng(17)
    src = np.stack([rng.integers(0, nx, (shots, nsrc)), rng.integers(0, nz if deep else 20, (shots, nsrc))], -1).astype(np.int32)
    if nsrc == 1:
        src = src[:, 0]
    else:
        src[:, 1] = src[:, 0]                                  # two nodes on one cell
    rec = np.stack([np.stack([rng.integers(0, nx, 40), rng.integers(0, nz if deep else 3, 40)], 1)] * shots)
    rec = rec.astype(np.int32)
    wav = torch.stack([S.ricker(20.0 + i, 0.01, 1e-3, nt) for i in range(shots * nsrc)])
    if nsrc > 1:
        wav = wav.reshape(shots, nsrc, nt).contiguous()
    m = S.Model(d, dev(c), shots, rec.shape[1], K)
    sh = S.Shots(src, rec, wav)
    m.set_tuning(S.SG_TUNE_TIME_BLOCKING, two)

    def sweep():
        seis = m.forward(sh).clone()
        assert torch.equal(m.forward(sh, save_ckpt=False), seis)
        m.forward(sh)
        w = torch.cos(torch.arange(seis.numel(), device="cuda", dtype=torch.float32)).reshape(seis.shape).contiguous()
        gw = torch.full_like(wav, float("nan"))
        g = m.gradient(sh, w, g_wavelet=gw).clone()
        return seis, g, gw
    one = sweep()
    m.set_tuning(S.SG_TUNE_PAIR, 0)
    apart = sweep()
    m.close()
    for a, b in zip(one, apart):
        assert torch.isfinite(a).all() and float(a.abs().max()) > 0.0
        assert torch.equal(a, b)
