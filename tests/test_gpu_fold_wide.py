"""GPU: the 2-D gradient's fold on grids of few, long rows, whose columns go to
several workgroups per row (run edges, a last run of few columns, no layer),
against the FP64 oracle as the fold of square grids."""
import pytest

import test_gpu_fold2 as fold

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nz,P,models,spm", [
    (255, 5, 8, 1, 1),             # one run
    (256, 5, 8, 1, 1),             # two runs of 127 columns
    (385, 4, 8, 2, 1),             # three, the last of 127
    (1500, 6, 7, 1, 2),            # eleven of 137
    (700, 1, 0, 1, 1),
])
def test_runs_of_columns(nx, nz, P, models, spm):
    fold.test_fold_of_the_layer(nx, nz, P, models, spm)
