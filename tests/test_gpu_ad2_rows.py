"""GPU: divergence-form workgroups of 16 and of 8 rows (launches of few
tiles) give the same values: a shot alone and in a batch, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,P,nsrc,nrec", [
    (101, 101, 20, 1, 101),        # 15 tiles, the last 13 rows high
    (60, 57, 16, 9, 700),          # several nodes in a cell, over 512 receivers in a tile
    (300, 160, 18, 300, 0),        # interior tiles, a row of nodes, no receivers
    (130, 97, 0, 5, 40),           # no layer
    (33, 9, 16, 2, 3),             # 41 rows: one past a multiple of 8
])
def test_shot_alone_and_in_a_batch(nx, nz, P, nsrc, nrec):
    rng = np.random.default_rng(nx + nsrc)
    nt, K = 23, 6
    vp = 1600.0 + 1400.0 * synth.smooth_random(7, (nz, nx), 4.0, 0.0, 1.0)
    src = np.stack([rng.integers(0, nx, nsrc), rng.integers(0, nz, nsrc)], 1)
    if nsrc > 4:
        src[3] = src[1]
    if nsrc == nx:
        src = np.stack([np.arange(nx), np.full(nx, nz - 3)], 1)
    rec = np.stack([rng.integers(0, min(nx, 40), nrec), rng.integers(0, nz, nrec)], 1).astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + j % 7, 0.006, 0.8e-3, nt) for j in range(nsrc)])
    tiles = -(-(nx + 2 * P) // 64) * -(-(nz + 2 * P) // 32)
    out = []
    for shots in (1, -(-120 // tiles) + 1):
        d = S.desc(physics=S.SG_ACOUSTIC_DIV, nx=nx, nz=nz, npml=P, nt=nt, nmodels=shots, dx=10.0, dt=0.8e-3,
                   pml_vmax=3000.0, f0_pml=20.0)
        m = S.Model(d, dev(np.stack([vp] * shots)), shots, nrec, K)
        sh = S.Shots(np.stack([src.astype(np.int32)] * shots), np.stack([rec] * shots),
                     wav[None].repeat(shots, 1, 1).contiguous())
        seis = m.forward(sh)
        w = torch.sin(torch.arange(seis[0].numel(), device="cuda", dtype=torch.float32)).reshape(seis[0].shape)
        gw = torch.empty_like(sh.wavelet)
        g = m.gradient(sh, w[None].repeat(shots, 1, 1, 1).contiguous(), g_wavelet=gw)
        assert torch.equal(m.forward(sh, save_ckpt=False), seis)
        out.append((seis[-1].clone(), g[-1].clone(), gw[-1].clone()))
        m.close()
    if nrec:
        assert float(out[0][0].abs().max()) > 0.0 and float(out[0][1].abs().max()) > 0.0
    for a, b in zip(*out):
        assert torch.equal(a, b)
