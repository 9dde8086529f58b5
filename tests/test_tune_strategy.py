"""A default Strategy leaves a model's 3-D launch settings to the library's
rule, whatever was set before, and the tuner times that rule first."""
import pytest
import torch

from paper_2003_06027_amd import seisgrad as S
from paper_2003_06027_amd import tune

CHUNKS = (S.SG_TUNE_CHUNK_FWD3, S.SG_TUNE_CHUNK_ADJ3, S.SG_TUNE_CHUNK_LAYER3)


class Recorder:
    def __init__(self, d):
        self.d, self.set = d, {}

    def set_tuning(self, key, value):
        self.set[key] = value


def test_default_strategy_is_the_librarys_rule():
    d = S.desc(ndim=3, nx=64, ny=64, nz=64, npml=8, nt=10)
    m = Recorder(d)
    tune.Strategy(graphs=True).apply(m)
    assert [m.set[k] for k in CHUNKS] == [0, 0, 0] and m.set[S.SG_TUNE_GRAPHS] == 1
    tune.Strategy(chunk_fwd3=48).apply(m)
    assert [m.set[k] for k in CHUNKS] == [48, 0, 0]
    assert tune.candidates(d)[0] == tune.Strategy()
    assert 0 in tune.CHUNKS_ADJ3 and 0 in tune.CHUNKS_LAYER3
    assert tune.Strategy().label() == "default"


@pytest.mark.gpu
def test_zero_restores_the_rule():
    d = S.desc(ndim=3, nx=40, ny=36, nz=70, npml=12, nt=8, dx=10.0, dt=1e-3, pml_vmax=2800.0)
    vp = torch.full((1, 70, 36, 40), 2000.0, device="cuda")
    m = S.Model(d, vp, 1, 1)
    torch.cuda.synchronize()
    start = m.ws.clone()                   # the layer's work list among it
    tune.Strategy(chunk_fwd3=32, chunk_adj3=64, chunk_layer3=32).apply(m)
    assert not torch.equal(m.ws, start)
    tune.Strategy().apply(m)
    assert torch.equal(m.ws, start)        # (32-plane lists are shorter: nothing is left behind the list)
    for k in CHUNKS:
        for bad in (-8, 8, 20, 72):
            with pytest.raises(S.SeisError):
                m.set_tuning(k, bad)
    m.close()
