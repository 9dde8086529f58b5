"""GPU: the parameter check of init_model and update_model (its range is
reduced on the device) refuses a bad value wherever it sits, and accepts and
measures the largest velocity exactly."""
import pytest
import torch

from paper_2003_06027_amd import seisgrad as S

pytestmark = pytest.mark.gpu

NX, NZ = 67, 41           # 2747 cells: a last block that is not full


def _desc(physics, dt=1e-3):
    return S.desc(ndim=2, physics=physics, nx=NX, nz=NZ, npml=10, nt=4, dx=10.0, dt=dt, pml_vmax=1500.0, f0_pml=10.0)


@pytest.mark.parametrize("cell", [0, 255, 256, NX * NZ - 1])
@pytest.mark.parametrize("value", [0.0, -1.0, float("nan"), float("inf"), float("-inf")])
def test_bad_velocity_is_refused(cell, value):
    d = _desc(S.SG_ACOUSTIC)
    good = torch.full((NZ, NX), 2000.0, device="cuda")
    bad = good.clone()
    bad.view(-1)[cell] = value
    with pytest.raises(S.SeisError) as e:
        S.Model(d, bad, 1, 1)
    assert e.value.code == S.SG_EINVAL
    m = S.Model(d, good, 1, 1)
    with pytest.raises(S.SeisError) as e:
        m.update(bad)
    assert e.value.code == S.SG_EINVAL
    m.update(good)
    m.close()


@pytest.mark.parametrize("field,value", [("vs", 0.0), ("vs", 2000.0), ("vs", float("nan")), ("rho", 0.0),
                                         ("rho", float("inf")), ("rho", float("nan"))])
def test_bad_elastic_parameters_are_refused(field, value):
    d = _desc(S.SG_ELASTIC)
    p = {"vp": torch.full((NZ, NX), 2000.0, device="cuda"), "vs": torch.full((NZ, NX), 1100.0, device="cuda"),
         "rho": torch.full((NZ, NX), 1800.0, device="cuda")}
    m = S.Model(d, p["vp"], 1, 1, vs=p["vs"], rho=p["rho"])
    p[field] = p[field].clone()
    p[field].view(-1)[NX * NZ - 1] = value
    with pytest.raises(S.SeisError) as e:
        m.update(p["vp"], p["vs"], p["rho"])
    assert e.value.code == S.SG_EINVAL
    m.close()


def test_one_fast_cell_decides_the_stability_check():
    limit = 0.95 * 2.0 / (6.501587301587301 * 2) ** 0.5           # c dt / dx
    v = torch.full((NZ, NX), 2000.0, device="cuda")
    v.view(-1)[1234] = 0.999 * limit * 10.0 / 1e-3
    m = S.Model(_desc(S.SG_ACOUSTIC), v, 1, 1)
    v.view(-1)[1234] = 1.001 * limit * 10.0 / 1e-3
    with pytest.raises(S.SeisError) as e:
        m.update(v)
    assert e.value.code == S.SG_EUNSTABLE
    m.close()
