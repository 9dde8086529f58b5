"""bench.py reports counted traffic for the launches that were counted only:
those of the library's default settings."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402
from paper_2003_06027_amd import tune  # noqa: E402


@pytest.mark.parametrize("wl", sorted(bench.TRAFFIC_FILES))
def test_traffic_of_default_launches_only(wl):
    for ph in ("forward", "recompute", "adjoint"):
        assert bench.measured_traffic(ph, wl, tune.Strategy().label()) == bench.measured_traffic(ph, wl)
        for s in (tune.Strategy(chunk_fwd3=16, chunk_adj3=48), tune.Strategy(shot_group=2), tune.Strategy(time_blocking=1)):
            assert bench.measured_traffic(ph, wl, s.label()) is None
