"""GPU: 3-D steps whose layer tiles and other tiles go out in one launch give
the values of steps that send them out as two, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P,shots", [((80, 40, 50), 6, 70), ((100, 64, 30), 8, 90)])
def test_one_launch_equals_two(n, P, shots):
    nx, ny, nz = n
    nt, K = 12, 5
    c = 1600.0 + 1200.0 * synth.smooth_random(9, (nz, ny, nx), 3.0, 0.0, 1.0)
    d = S.desc(ndim=3, nx=nx, ny=ny, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    rng = np.random.default_rng(4)
    src = np.stack([rng.integers(0, k, shots) for k in n], 1).astype(np.int32)
    rec = np.stack([np.stack([rng.integers(0, k, 9) for k in n], 1) for _ in range(shots)]).astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + 0.2 * i, 0.005, 1e-3, nt) for i in range(shots)])
    weight = torch.cos(torch.arange(shots * nt * 9, device="cuda", dtype=torch.float32)).reshape(shots, 1, nt, 9)

    # other tiles (no cell within 4 of the layer in x or y), in workgroups of 16 planes
    def away(k, t):
        return sum(1 for x in range(0, k + 2 * P, t) if x - 4 >= P and x + t + 4 <= P + k)
    per_shot = -(-away(nx, 32) * away(ny, 16) // 8) * 8 * -(-(nz + 2 * P) // 16)
    assert 0 < per_shot * 10 <= 2048 < per_shot * shots

    def sweep(k):
        sh = S.Shots(src[k], np.ascontiguousarray(rec[k]), wav[k].contiguous())
        m = S.Model(d, dev(c), len(src[k]), 9, K)
        m.set_tuning(S.SG_TUNE_CHUNK_FWD3, 16)
        seis = m.forward(sh).clone()
        gw = torch.empty_like(wav[k])
        m.gradient(sh, weight[k].contiguous(), g_wavelet=gw)
        only = m.forward(sh, save_ckpt=False)
        assert torch.equal(only, seis)
        m.close()
        return seis, gw
    seis, gw = sweep(slice(0, shots))
    assert float(seis.abs().max()) > 0.0 and float(gw.abs().max()) > 0.0
    for i in range(0, shots, 10):
        s2, g2 = sweep(slice(i, i + 10))
        assert torch.equal(s2, seis[i:i + 10]), i
        assert torch.equal(g2, gw[i:i + 10]), i
