"""GPU: 3-D receivers at several depths, duplicate receivers among them, give
the same records whatever z chunk their plane falls in, and the chunk
lengths taken by rule give the values of the set ones bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,P,planes", [
    (40, 21, 70, 12, (0,)),                       # one receiver plane, near the top
    (33, 40, 50, 8, (0, 7, 8, 23, 24, 49)),       # planes on both sides of 8- and 16-plane chunk edges
    (70, 24, 20, 0, (19, 3)),                     # no layer, the last plane
    (24, 17, 9, 6, ()),                           # no receivers, fewer planes than a default chunk
])
def test_receiver_planes_and_chunk_rule(nx, ny, nz, P, planes):
    nt, K = 24, 7
    c = 1600.0 + 1200.0 * synth.smooth_random(5, (nz, ny, nx), 3.0, 0.0, 1.0)
    d = S.desc(ndim=3, nx=nx, ny=ny, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    rng = np.random.default_rng(3)
    src = np.stack([rng.integers(0, nx, 2), rng.integers(0, ny, 2), rng.integers(0, nz, 2)], 1).astype(np.int32)
    per = [np.stack([rng.integers(0, nx, 40), rng.integers(0, ny, 40), np.full(40, p)], 1) for p in planes]
    r = np.concatenate(per + [per[0][:5]]) if per else np.zeros((0, 3))   # five duplicates
    rng.shuffle(r)
    rec = np.stack([r, r]).astype(np.int32)
    wav = torch.stack([S.ricker(25.0, 0.01, 1e-3, nt), S.ricker(30.0, 0.008, 1e-3, nt)])
    sh = S.Shots(src, rec, wav)
    m = S.Model(d, dev(c), 2, rec.shape[1], K)

    def sweep():
        seis = m.forward(sh)
        w = torch.cos(torch.arange(seis.numel(), device="cuda", dtype=torch.float32)).reshape(seis.shape).contiguous()
        gw = torch.empty_like(wav)
        return seis, m.gradient(sh, w, g_wavelet=gw), gw

    by_rule = sweep()                             # 8-plane chunks: these grids have few tiles
    for fwd, adj in ((64, 64), (16, 32)):
        m.set_tuning(S.SG_TUNE_CHUNK_FWD3, fwd)
        m.set_tuning(S.SG_TUNE_CHUNK_ADJ3, adj)
        for a, b in zip(by_rule, sweep()):
            assert torch.equal(a, b), (fwd, adj)
    if planes:
        assert float(by_rule[0].abs().max()) > 0.0 and float(by_rule[1].abs().max()) > 0.0
    # every receiver's record against one receiver at a time
    for i in range(0, rec.shape[1], 17):
        one = m.forward(S.Shots(src, np.ascontiguousarray(rec[:, i:i + 1]), wav), save_ckpt=False)
        assert torch.equal(one[..., 0], by_rule[0][..., i])
    m.close()
