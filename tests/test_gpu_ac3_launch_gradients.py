"""GPU: model gradients of 3-D shots whose layer tiles and other tiles go out
in one launch equal those of launches apart, bit for bit: one model per shot,
so that each shot's gradient (formed from the recomputed snapshots) is seen."""
import numpy as np
import pytest
import torch

from gpu_common import S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P,shots", [((80, 40, 50), 6, 70), ((100, 64, 30), 8, 90)])
def test_gradients_of_one_launch_and_two(n, P, shots):
    nx, ny, nz = n
    nt, K, few = 14, 5, 10
    c = 1600.0 + 1200.0 * synth.smooth_random(9, (nz, ny, nx), 3.0, 0.0, 1.0)
    rng = np.random.default_rng(4)
    src = np.stack([rng.integers(k // 4, 3 * k // 4, shots) for k in n], 1).astype(np.int32)
    rec = np.clip(src[:, None] + rng.integers(-4, 5, (shots, 9, 3)), 0, np.array(n) - 1).astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + 0.2 * i, 0.005, 1e-3, nt) for i in range(shots)])
    weight = torch.cos(torch.arange(shots * nt * 9, device="cuda", dtype=torch.float32)).reshape(shots, 1, nt, 9)

    # other tiles (no cell within 4 of the layer in x or y), in workgroups of 16 planes: one launch up to 2048
    def away(k, t):
        return sum(1 for x in range(0, k + 2 * P, t) if x - 4 >= P and x + t + 4 <= P + k)
    per_shot = -(-away(nx, 32) * away(ny, 16) // 8) * 8 * -(-(nz + 2 * P) // 16)
    assert 0 < per_shot * few <= 2048 < per_shot * shots

    def sweep(k):
        B = len(src[k])
        d = S.desc(ndim=3, nx=nx, ny=ny, nz=nz, npml=P, nt=nt, nmodels=B, dx=10.0, dt=1e-3, pml_vmax=1500.0)
        m = S.Model(d, dev(np.stack([c] * B)), B, 9, K)
        m.set_tuning(S.SG_TUNE_CHUNK_FWD3, 16)
        sh = S.Shots(src[k], np.ascontiguousarray(rec[k]), wav[k].contiguous())
        m.forward(sh)
        g = m.gradient(sh, weight[k].contiguous()).clone()
        m.close()
        return g
    g = sweep(slice(0, shots))
    assert float(g.flatten(1).abs().amax(1).min()) > 0.0                # every shot has one
    for i in range(0, shots, few):
        assert torch.equal(sweep(slice(i, i + few)), g[i:i + few]), i
