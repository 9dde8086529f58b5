"""GPU: update_model with the parameters that a model has leaves its workspace
as it was, the misfit's partial sums among it: the parameter check must not
share scratch memory with a misfit that another stream may be running."""
import numpy as np
import pytest
import torch

from gpu_common import S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,physics", [(2, S.SG_ACOUSTIC), (2, S.SG_ACOUSTIC_DIV), (2, S.SG_ELASTIC),
                                          (3, S.SG_ACOUSTIC)])
def test_update_with_equal_parameters_changes_no_byte(ndim, physics):
    n, nt = 40, 12
    vp = (2000.0 + 300.0 * torch.rand((n,) * ndim, device="cuda"))[None].contiguous()
    el = [vp / 1.8, torch.full_like(vp, 2100.0)] if physics == S.SG_ELASTIC else [None, None]
    d = S.desc(ndim=ndim, physics=physics, nx=n, ny=n if ndim == 3 else 1, nz=n, npml=8, nt=nt, dt=8e-4, pml_vmax=1500.0)
    src = np.full((1, ndim), 20, np.int32)
    rec = np.full((1, 5, ndim), 22, np.int32)
    mt = np.ones((1, 3), np.float32) if physics == S.SG_ELASTIC else None
    m = S.Model(d, vp, 1, 5, vs=el[0], rho=el[1])
    seis = m.forward(S.Shots(src, rec, S.ricker(25.0, 0.004, 8e-4, nt)[None], mt=mt))
    a = torch.randn(50000, device="cuda")
    J, _ = m.misfit(a, torch.zeros_like(a))            # 49 workgroups: partial sums in the workspace
    torch.cuda.synchronize()
    before = m.ws.clone()
    m.update(vp, *el)
    torch.cuda.synchronize()
    assert torch.equal(m.ws, before)
    assert float((J - 0.5 * (a.double() ** 2).sum()).abs() / J) <= 1e-12 and torch.isfinite(seis).all()
    m.close()
