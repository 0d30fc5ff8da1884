"""The obstruction map computes the samples next to the roots of the cut
condition only: sample counts at the edges of its 64-sample anchors, grids with
a row on the real axis (where the condition vanishes identically), next to
x = 0 and at large cutoffs, against the oracle, which walks every sample."""
import numpy as np
import pytest

import oracle
import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import Grid, Params

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BOXES = [Grid(23, 21, -12.0, 6.0, -6.0, 6.0),          # middle row on the real axis
         Grid(19, 16, -1e-2, 1e-2, -1e-2, 1e-2),
         Grid(22, 14, -9.0, 1.0, 0.0, 1e-3)]
MASSES = [Params(1.0, 1.0, 1.0, 1e6), Params(1 + 0.5j, 1 - 0.5j, 1.0, 1e6),
          Params(-0.3 + 1.1j, 0.4 - 0.2j, 1.0, 1e4), Params(1e-3, 20.0, 1.0, 1e10)]


@pytest.mark.parametrize("n", [4, 64, 65, 66, 129, 4096])
@pytest.mark.parametrize("p", MASSES, ids=["real", "conjugate", "complex", "unequal"])
def test_map_equals_the_full_walk(p, n):
    for grid in BOXES:
        got = gf.obstruction_map(p, grid, n)
        torch.cuda.synchronize()
        got = got.cpu().numpy().ravel()
        want, tie = oracle.obstruction(p, oracle.grid_points(grid), n)
        bad = (got != want) & ~tie
        assert not np.any(bad), (grid, np.nonzero(bad)[0][:5])


@pytest.mark.parametrize("n", [2, 3, 7, 8, 9, 16])
@pytest.mark.parametrize("p", MASSES, ids=["real", "conjugate", "complex", "unequal"])
def test_short_walks_compute_every_sample(p, n):
    """Up to eight samples a part are all computed, more go by the roots."""
    test_map_equals_the_full_walk(p, n)
