"""GPU: the 2-D gradient's fold of the layer cells onto end and corner cells,
each set by itself against the FP64 oracle: rows past two runs of 64 columns,
one column, one row, a layer thicker than a run of 64 cells, no layer."""
import numpy as np
import pytest
import torch

from gpu_common import O, S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,P,models,spm", [
    (200, 21, 9, 1, 1),
    (33, 130, 20, 2, 2),
    (1, 40, 12, 1, 1),
    (40, 1, 12, 2, 1),
    (20, 15, 70, 1, 1),
    (66, 64, 0, 1, 2),
])
def test_fold_of_the_layer(nx, nz, P, models, spm):
    nt, B = 30, models * spm
    rng = np.random.default_rng(11)
    c = np.stack([1600.0 + 900.0 * synth.smooth_random(3 + i, (nz, nx), 2.0, 0.0, 1.0) for i in range(models)])
    src = np.stack([rng.integers(0, nx, B), rng.integers(0, nz, B)], 1).astype(np.int32)
    rec = np.stack([np.stack([rng.integers(0, n, 12) for n in (nx, nz)], 1) for _ in range(B)]).astype(np.int32)
    wav = torch.stack([S.ricker(30.0, 0.008, 1e-3, nt)] * B)
    wo = np.stack([O.ricker(30.0, 0.008, 1e-3, nt)] * B)
    d = S.desc(nx=nx, nz=nz, npml=P, nt=nt, nmodels=models, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    m = S.Model(d, dev(c), B, rec.shape[1], 6)
    seis = m.forward(S.Shots(src, rec, wav))
    w = torch.cos(torch.arange(seis.numel(), device="cuda", dtype=torch.float32)).reshape(seis.shape) * 1e-3
    g = m.gradient(S.Shots(src, rec, wav), w.contiguous()).cpu().numpy()
    m.close()
    go = O.grid(ndim=2, nx=nx, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    wn = w.cpu().numpy()
    ends = sum(((np.arange(n) == 0) | (np.arange(n) == n - 1)).reshape(s).astype(int)
               for n, s in ((nz, (-1, 1)), (nx, (1, -1))))
    for i in range(models):
        k = slice(i * spm, (i + 1) * spm)
        ref = np.asarray(O.ac2_gradient(go, c[i], src[k], wo[k], rec[k], wn[k, 0], ckpt=6)[0]).reshape(nz, nx)
        got = g[i].reshape(nz, nx)
        # interior, ends, corners: relative to the set itself, as the
        # gradients elsewhere (1e-3), plus FP32 noise of the whole
        for q in range(3):
            a, b = got[ends == q].astype(np.float64), ref[ends == q]
            assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b) + 1e-6 * np.linalg.norm(ref), (i, q)
