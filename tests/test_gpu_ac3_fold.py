"""GPU: the 3-D gradient's fold of the layer cells onto the face, edge and
corner cells that they replicate, each set by itself against the FP64
oracle."""
import numpy as np
import pytest
import torch

from gpu_common import O, S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,P,models,spm", [
    (70, 21, 33, 9, 1, 1),         # rows past one wavefront
    (5, 130, 4, 20, 2, 2),         # long in y; corners of 21^3 cells; two models of two shots
    (1, 9, 6, 7, 1, 1),            # one cell in x
    (8, 1, 1, 6, 2, 1),            # one cell in y and z
    (64, 6, 129, 6, 1, 2),
    (12, 11, 10, 0, 1, 1),         # no layer
])
def test_fold_of_the_layer(nx, ny, nz, P, models, spm):
    nt, B = 20, models * spm
    rng = np.random.default_rng(11)
    c = np.stack([1600.0 + 900.0 * synth.smooth_random(3 + i, (nz, ny, nx), 2.0, 0.0, 1.0) for i in range(models)])
    src = np.stack([rng.integers(0, nx, B), rng.integers(0, ny, B), rng.integers(0, nz, B)], 1).astype(np.int32)
    rec = np.stack([np.stack([rng.integers(0, n, 12) for n in (nx, ny, nz)], 1) for _ in range(B)]).astype(np.int32)
    wav = torch.stack([S.ricker(30.0, 0.008, 1e-3, nt)] * B)
    wo = np.stack([O.ricker(30.0, 0.008, 1e-3, nt)] * B)
    d = S.desc(ndim=3, nx=nx, ny=ny, nz=nz, npml=P, nt=nt, nmodels=models, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    m = S.Model(d, dev(c), B, rec.shape[1], 6)
    sh = S.Shots(src, rec, wav)
    seis = m.forward(sh)
    w = torch.cos(torch.arange(seis.numel(), device="cuda", dtype=torch.float32)).reshape(seis.shape) * 1e-3
    g = m.gradient(sh, w.contiguous()).cpu().numpy()
    m.close()
    go = O.grid(ndim=3, nx=nx, ny=ny, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    wn = w.cpu().numpy()
    for i in range(models):
        k = slice(i * spm, (i + 1) * spm)
        ref, _ = O.ac3_gradient(go, c[i], src[k], wo[k], rec[k], wn[k, 0], ckpt=6)
        ref = np.asarray(ref).reshape(nz, ny, nx)
        got = g[i].reshape(nz, ny, nx)
        # interior, faces, edges, corners: relative to the set itself, as the
        # gradients elsewhere (1e-3), plus FP32 noise of the whole
        ends = sum(((np.arange(n) == 0) | (np.arange(n) == n - 1)).reshape(s).astype(int)
                   for n, s in ((nz, (-1, 1, 1)), (ny, (1, -1, 1)), (nx, (1, 1, -1))))
        for q in range(4):
            a, b = got[ends == q].astype(np.float64), ref[ends == q]
            if b.size:
                assert np.linalg.norm(b) > 0.0
                assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b) + 1e-6 * np.linalg.norm(ref), (i, q)
