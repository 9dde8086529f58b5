"""GPU: the parameter check on models of one workgroup and of several (up to
8192 cells and above): a bad value or the fastest cell anywhere decides."""
import pytest
import torch

from gpu_common import S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz", [(1, 1), (64, 128), (2731, 3), (130, 90)])
@pytest.mark.parametrize("where", [0.0, 0.5, 1.0])
def test_one_cell_decides(nx, nz, where):
    n = nx * nz
    cell = int(where * (n - 1))
    d = S.desc(nx=nx, nz=nz, npml=10, nt=4, dx=10.0, dt=1e-3, pml_vmax=1500.0)
    v = torch.full((nz, nx), 2000.0, device="cuda")
    m = S.Model(d, v, 1, 1)
    limit = 0.95 * 2.0 / (6.501587301587301 * 2) ** 0.5 * 10.0 / 1e-3
    for value, code in ((0.0, S.SG_EINVAL), (float("nan"), S.SG_EINVAL), (float("inf"), S.SG_EINVAL),
                        (1.001 * limit, S.SG_EUNSTABLE), (0.999 * limit, None)):
        w = v.clone()
        w.view(-1)[cell] = value
        if code is None:
            m.update(w)
            continue
        with pytest.raises(S.SeisError) as e:
            m.update(w)
        assert e.value.code == code
    m.update(v)                            # nothing of an earlier check is left
    m.close()
