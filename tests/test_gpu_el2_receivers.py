"""GPU: the receiver workgroups that ride in the elastic launches: no
receivers, one, exactly a workgroup and one more, against runs of a few
receivers at a time and of the receivers in another order, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shots", [1, 4])
@pytest.mark.parametrize("nrec", [0, 1, 256, 257])
def test_receivers(nrec, shots):
    nx, nz, P, nt, K = 61, 37, 8, 19, 5
    c = 2000.0 + 600.0 * synth.smooth_random(3, (nz, nx), 3.0, 0.0, 1.0)
    d = S.desc(ndim=2, physics=S.SG_ELASTIC, nx=nx, nz=nz, npml=P, nt=nt, dx=10.0, dt=1e-3, pml_vmax=1800.0,
               f0_pml=20.0)
    rng = np.random.default_rng(5)
    cells = np.stack([rng.permutation(nx * nz)[:nrec] for _ in range(shots)])
    rec = np.stack([cells % nx, cells // nx], -1).astype(np.int32)
    src = np.stack([rng.integers(10, nx - 10, shots), rng.integers(10, nz - 10, shots)], 1).astype(np.int32)
    wav = torch.stack([S.ricker(30.0 + i, 0.006, 1e-3, nt) for i in range(shots)])

    def run(r, w=None):
        m = S.Model(d, dev(c), shots, max(r.shape[1], 1), K, vs=dev(c / 1.8), rho=dev(0 * c + 2000.0))
        sh = S.Shots(src, np.ascontiguousarray(r), wav, mt=np.array([[1.0, 0.7, 0.2]] * shots))
        seis = m.forward(sh).clone()
        g = None if w is None else [t.clone() for t in m.gradient(sh, w.contiguous())]
        m.close()
        return seis, g
    w = torch.cos(torch.arange(shots * 2 * nt * nrec, device="cuda", dtype=torch.float32)).reshape(shots, 2, nt, nrec)
    seis, g = run(rec, w)
    assert seis.shape == w.shape
    if nrec == 0:
        assert all(float(t.abs().max()) == 0.0 for t in g)
        return
    if nrec > 1:
        assert float(seis.abs().max()) > 0.0 and float(g[0].abs().max()) > 0.0
    order = rng.permutation(nrec)
    s2, g2 = run(rec[:, order], w[..., torch.as_tensor(order, device="cuda")])
    assert torch.equal(s2, seis[..., torch.as_tensor(order, device="cuda")])
    assert all(torch.equal(a, b) for a, b in zip(g, g2))
    for b in range(0, nrec, 100):
        assert torch.equal(run(rec[:, b:b + 3])[0], seis[..., b:b + 3])
