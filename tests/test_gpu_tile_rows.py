"""GPU: a launch of few 2-D acoustic tiles splits them into workgroups of 16
or 8 rows; every shot's records, gradient and wavelet gradients equal those
of a batch large enough for whole tiles, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


def _sweep(nx, nz, P, nt, K, vp, src, rec, wav, shots):
    """`shots` copies of one shot, each on its own model."""
    d = S.desc(nx=nx, nz=nz, npml=P, nt=nt, nmodels=shots, dx=10.0, dt=0.8e-3, pml_vmax=3000.0)
    m = S.Model(d, dev(np.stack([vp] * shots)), shots, rec.shape[0], K)
    sh = S.Shots(np.stack([src] * shots), np.stack([rec] * shots), wav[None].repeat(shots, 1, 1).contiguous())
    seis = m.forward(sh)
    w = torch.sin(torch.arange(seis[0].numel(), device="cuda", dtype=torch.float32)).reshape(seis[0].shape)
    gw = torch.empty_like(sh.wavelet)
    g = m.gradient(sh, w[None].repeat(shots, 1, 1, 1).contiguous(), g_wavelet=gw)
    plain = m.forward(sh, save_ckpt=False)
    assert torch.equal(plain, seis)
    m.close()
    return seis, g, gw


# padded extents of 1, 5 and 9 rows past a multiple of 8 and 32; receivers at the
# surface, at depth (one-step tiles away from the layer), over 512 in one tile, none;
# one source or several nodes, some sharing a cell
@pytest.mark.parametrize("nx,nz,P,nsrc,recs", [
    (101, 101, 20, 1, "surface"),
    (60, 57, 16, 9, "many"),
    (300, 160, 18, 1, "surface"),            # blocked tiles
    (300, 160, 18, 30, "deep"),              # and one-step tiles around nodes and receivers
    (130, 97, 0, 5, "deep"),                 # no layer
    (70, 33, 16, 1, "none"),
])
def test_split_tiles_equal_whole_tiles(nx, nz, P, nsrc, recs):
    rng = np.random.default_rng(nx + nsrc)
    nt, K = 23, 6
    vp = 1600.0 + 1400.0 * synth.smooth_random(7, (nz, nx), 4.0, 0.0, 1.0)
    node = np.stack([rng.integers(nx // 3, 2 * nx // 3, nsrc), rng.integers(nz // 3, 2 * nz // 3, nsrc)], 1)
    if nsrc > 4:
        node[3] = node[1]                    # two nodes in one cell
    n = {"surface": nx, "deep": 60, "many": 700, "none": 0}[recs]
    rec = np.stack([rng.integers(0, nx, n), rng.integers(0, nz, n)], 1)
    if recs == "surface":
        rec = np.stack([np.arange(nx), np.zeros(nx, int)], 1)
        node[:, 1] = 3                       # the wave reaches the receivers within the run
    if recs == "many":
        rec[:, 0] %= 40                      # one or two tiles, many duplicates
        rec[:, 1] %= 8
    src = node.astype(np.int32) if nsrc > 1 else node[0].astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + j, 0.006, 0.8e-3, nt) for j in range(nsrc)])
    tiles = -(-(nx + 2 * P) // 64) * -(-(nz + 2 * P) // 32)
    # 8 rows; 16 and 32 rows in the launch of all tiles (a launch of a subset may split further)
    out = {s: _sweep(nx, nz, P, nt, K, vp, src, rec.astype(np.int32), wav, s)
           for s in (1, max(2, -(-300 // tiles)), max(3, -(-2200 // tiles)))}
    ref = out[1]
    if n:
        assert float(ref[0].abs().max()) > 0.0 and float(ref[1].abs().max()) > 0.0
    for s, (seis, g, gw) in out.items():
        for i in (0, s // 2, s - 1):
            assert torch.equal(seis[i], ref[0][0]), (s, i)
            assert torch.equal(g[i], ref[1][0]), (s, i)
            assert torch.equal(gw[i], ref[2][0]), (s, i)
