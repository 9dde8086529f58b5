"""GPU: a model with room for more shots than the batch (fields that are not
contiguous over the batch), reused after a larger batch, gives the gradients
of a model of the batch's own size bit for bit, with checkpoints restored and
with kept snapshots."""
import numpy as np
import pytest
import torch

from gpu_common import dev
from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phys", ["ac2", "ad2", "el2", "ac3"])
@pytest.mark.parametrize("kept", [0, 2, 100])
def test_room_for_more_shots(phys, kept):
    three = phys == "ac3"
    n = (30, 22, 26) if three else (70, 50)
    nt, K, P = 23, 6, 8
    c = 2000.0 + 600.0 * synth.smooth_random(3, n[::-1], 3.0, 0.0, 1.0)
    d = S.desc(ndim=3 if three else 2, nx=n[0], **({"ny": n[1]} if three else {}), nz=n[-1], npml=P, nt=nt, dx=10.0,
               dt=1e-3, pml_vmax=1800.0, f0_pml=20.0,
               physics={"el2": S.SG_ELASTIC, "ad2": S.SG_ACOUSTIC_DIV}.get(phys, S.SG_ACOUSTIC))
    par = {"vs": dev(c / 1.8), "rho": dev(0 * c + 2000.0)} if phys == "el2" else {}
    rng = np.random.default_rng(1)

    def shots(b):
        pick = lambda m: np.stack([rng.integers(2, k - 2, m) for k in n], 1).astype(np.int32)
        src = pick(b)
        rec = np.stack([np.clip(src[i] + rng.integers(-4, 5, (7, len(n))), 0, np.array(n) - 1) for i in range(b)])
        wav = torch.stack([S.ricker(30.0 + i, 0.006, 1e-3, nt) for i in range(b)])
        mt = {"mt": np.array([[1.0, 0.7, 0.2]] * b)} if phys == "el2" else {}
        return S.Shots(src, rec.astype(np.int32), wav, **mt)
    big, small = shots(5), shots(3)

    def sweep(m, sh):
        seis = m.forward(sh)
        w = torch.cos(torch.arange(seis.numel(), device="cuda", dtype=torch.float32)).reshape(seis.shape).contiguous()
        g = m.gradient(sh, w)
        return [seis.clone()] + [t.clone() for t in (g if isinstance(g, tuple) else (g,))]
    a = S.Model(d, dev(c), 5, 7, K, store_segments=kept, **par)
    sweep(a, big)
    got = sweep(a, small)
    a.close()
    b = S.Model(d, dev(c), 3, 7, K, **par)
    want = sweep(b, small)
    b.close()
    for x, y in zip(got, want):
        assert float(y.abs().max()) > 0.0 and torch.isfinite(y).all()
        assert torch.equal(x, y)
