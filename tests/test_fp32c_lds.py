"""FP32C scans read the angular nodes from LDS at up to 8 lanes per point and up to 512
folded pairs, and through scalar registers otherwise.  The two read the same
FP32 numbers into the same operations, so scans at few lanes equal one at 64 lanes
up to the order of the FP64 sum over nodes: 64 eps kappa |G| with the oracle's
condition number kappa, far below the FP32 rounding of either."""
import numpy as np
import pytest

import oracle
import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import FP32C, Grid, Params, Propagators, Quadrature
from parity_bars import EPS

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

GRID = Grid(27, 10, -9.0, 4.0, -3.1, 3.3)


# one pair; below, at and above a step of eight, a block of sixteen and the LDS table
@pytest.mark.parametrize("n_a", [2, 3, 15, 16, 18, 31, 32, 34, 41, 1023, 1024, 1026])
@pytest.mark.parametrize("form", ["plain", "taylor", "split", "numerator"])
def test_nodes_from_lds_equal_nodes_from_scalar_registers(n_a, form):
    p = Params(1.0, 0.25, 1.0, 1e6, 1.0, 2 if form == "taylor" else 0)
    q = Quadrature(16, n_a, 5, FP32C, radial_split=int(form == "split"))
    props = None
    if form == "numerator":
        props = Propagators(((0.4, 1.0), (2.5, -0.3)), ((1.0, 0.6), (3.0, 0.4)),
                            ((0, 0, 1.0), (1, 0, 0.3), (0, 1, 0.2)))
    plan = gf.Plan(p, q, props)
    out = {}
    for lanes in (1, 2, 4, 8, 64):
        out[lanes] = gf.scan_plan(plan, GRID, lanes=lanes).cpu().numpy().ravel()
    plan.close()
    x = oracle.grid_points(GRID)
    ref = out.pop(64)
    _, _, cond = oracle.eval_points(p, q, x, want_cond=True, props=props)
    for lanes, got in out.items():
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        ok = ~np.isnan(ref)
        err = np.abs(got - ref)[ok]
        assert np.all(err <= 64 * EPS * cond[ok] * np.abs(ref[ok]) + 1e-15), (lanes, err.max())
