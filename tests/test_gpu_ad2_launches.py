"""GPU: divergence-form launches of 8 rows, of 16 rows with every load early
and of 16 rows with late loads give the same values: a shot alone, in a batch
of 96 to 128 tiles and in one of more than 256, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,P,nsrc,nrec", [
    (101, 101, 20, 1, 101),        # 15 tiles
    (150, 57, 16, 9, 600),         # 9 tiles, over 512 receivers
    (130, 97, 0, 5, 40),           # 12 tiles, no layer
    (33, 9, 16, 2, 3),             # 4 tiles, two of 9 rows
])
def test_early_and_late_loads(nx, nz, P, nsrc, nrec):
    rng = np.random.default_rng(nx + nsrc)
    nt, K = 17, 5
    vp = 1600.0 + 1400.0 * synth.smooth_random(7, (nz, nx), 4.0, 0.0, 1.0)
    src = np.stack([rng.integers(0, nx, nsrc), rng.integers(0, nz, nsrc)], 1).astype(np.int32)
    rec = np.stack([(src[0, 0] + rng.integers(-8, 9, nrec)) % nx, rng.integers(0, nz, nrec)], 1).astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + j % 7, 0.006, 0.8e-3, nt) for j in range(nsrc)])
    tiles = -(-(nx + 2 * P) // 64) * -(-(nz + 2 * P) // 32)
    mid, many = 128 // tiles, 256 // tiles + 1
    assert 96 <= mid * tiles <= 128 and many * tiles > 256
    out = []
    for shots in (1, mid, many):
        d = S.desc(physics=S.SG_ACOUSTIC_DIV, nx=nx, nz=nz, npml=P, nt=nt, nmodels=shots, dx=10.0, dt=0.8e-3,
                   pml_vmax=3000.0, f0_pml=20.0)
        m = S.Model(d, dev(np.stack([vp] * shots)), shots, nrec, K)
        sh = S.Shots(np.stack([src] * shots), np.stack([rec] * shots), wav[None].repeat(shots, 1, 1).contiguous())
        seis = m.forward(sh)
        w = torch.sin(torch.arange(seis[0].numel(), device="cuda", dtype=torch.float32)).reshape(seis[0].shape)
        gw = torch.empty_like(sh.wavelet)
        g = m.gradient(sh, w[None].repeat(shots, 1, 1, 1).contiguous(), g_wavelet=gw)
        out.append((seis[-1].clone(), g[-1].clone(), gw[-1].clone()))
        m.close()
    for a, b, c in zip(*out):
        assert float(a.abs().max()) > 0.0
        assert torch.equal(a, b) and torch.equal(a, c)
