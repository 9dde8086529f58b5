"""GPU: the divergence form's workgroups (8 rows, 16 rows with early loads, 16
rows with late ones, chosen by the number of tiles of a launch) give the same
values bit for bit, tiles away from the layer among them: a shot alone and as
the last of batches that take each of them."""
import numpy as np
import pytest
import torch

from gpu_common import S, dev
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


def _variant(tiles):
    if tiles < 96 or 128 < tiles <= 192:
        return "8 rows"
    return "16 rows early" if tiles <= 256 else "16 rows late"


def _away(n, P, t):
    """Tile origins whose 3-node halo stays off the layer on one axis."""
    return [x for x in range(0, n + 2 * P, t) if x - 3 >= P and x + t + 3 <= P + n]


@pytest.mark.parametrize("nx,nz,P,nsrc", [
    (300, 160, 18, 300),           # a row of nodes through tiles away from the layer
    (300, 160, 18, 1),
    (210, 118, 16, 6),
    (101, 101, 20, 1),             # every tile by the layer
])
def test_every_variant_gives_the_values_of_one_shot(nx, nz, P, nsrc):
    rng = np.random.default_rng(nx + nsrc)
    nt, K, nrec = 44, 9, 120
    vp = 1600.0 + 1400.0 * synth.smooth_random(7, (nz, nx), 4.0, 0.0, 1.0)
    tiles = -(-(nx + 2 * P) // 64) * -(-(nz + 2 * P) // 32)
    away = [(x, z) for x in _away(nx, P, 64) for z in _away(nz, P, 32)]     # whole tiles
    if nsrc == nx:
        src = np.stack([np.arange(nx), np.full(nx, nz // 2)], 1)
    else:
        cx, cz = (away[0][0] + 40 - P, away[0][1] + 5 - P) if away else (nx // 2, nz // 2)
        src = np.stack([cx + 3 * np.arange(nsrc), np.full(nsrc, cz)], 1)
    at = src[rng.integers(0, nsrc, nrec)]
    rec = np.clip(at + rng.integers(-12, 13, at.shape), 0, [nx - 1, nz - 1]).astype(np.int32)
    wav = torch.stack([S.ricker(25.0 + j % 7, 0.012, 0.8e-3, nt) for j in range(nsrc)])
    shots = [1] + [next(n for n in range(1, 400) if lo <= n * tiles <= hi)
                   for lo, hi in ((96, 128), (129, 192), (193, 256), (257, 400))]
    seen = [_variant(n * tiles) for n in shots]
    assert seen == ["8 rows", "16 rows early", "8 rows", "16 rows early", "16 rows late"]
    assert bool(away) == (nx > 101)
    first = None
    for n in shots:
        d = S.desc(physics=S.SG_ACOUSTIC_DIV, nx=nx, nz=nz, npml=P, nt=nt, nmodels=n, dx=10.0, dt=0.8e-3,
                   pml_vmax=3000.0, f0_pml=20.0)
        m = S.Model(d, dev(np.stack([vp] * n)), n, nrec, K)
        sh = S.Shots(np.stack([src.astype(np.int32)] * n), np.stack([rec] * n), wav[None].repeat(n, 1, 1).contiguous())
        seis = m.forward(sh)
        w = torch.sin(torch.arange(seis[0].numel(), device="cuda", dtype=torch.float32)).reshape(seis[0].shape)
        gw = torch.empty_like(sh.wavelet)
        g = m.gradient(sh, w[None].repeat(n, 1, 1, 1).contiguous(), g_wavelet=gw)
        out = (seis[-1].clone(), g[-1].clone(), gw[-1].clone())
        m.close()
        if first is None:
            first = out
            assert all(float(t.abs().max()) > 0.0 for t in out)
            for x, z in away[:1] if nsrc < nx else away:             # the path away from the layer is at work
                if nsrc < nx or z <= nz // 2 + P < z + 32:
                    assert float(g[-1][z - P:z - P + 32, x - P:x - P + 64].abs().max()) > 0.0
        for a, b in zip(out, first):
            assert torch.equal(a, b), n
