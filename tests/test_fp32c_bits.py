"""FP32C results bit for bit.  An FP32C sum rounds U^2 and V^2 to FP32 and takes a
node's form by their values, so a last-bit change of a ray's direction or an
arc's angles, harmless in FP64, moves a result by up to FP32 rounding.  The values in
golden/fp32c_values.npz were recorded with the directions (cos phi, sin phi) of the
device math library and the scalar-register nodes; one lane per point, every
contour class, D = 2, 3, 4."""
import os

import numpy as np
import pytest

import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import FP32C, Grid, Params, Propagators, Quadrature

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fp32c_values.npz")
GRID = Grid(21, 18, -8.0, 4.0, -4.0, 4.0)
CASES = {
    "real": (Params(1.3, 0.6, 2.0, 1e6), Quadrature(32, 64, 16, FP32C), None),
    "conjugate": (Params(1 + 0.5j, 1 - 0.5j, 1.0, 1e6), Quadrature(32, 129, 9, FP32C), None),
    "complex_d3": (Params(-0.3 + 1.1j, 0.4 - 0.2j, 1.0, 1e6, 1.0, 0, 3),
                   Quadrature(24, 32, 9, FP32C), None),
    "real_d2": (Params(1.0, 1.0, 1.0, 1e6, 1.0, 1, 2), Quadrature(24, 40, 9, FP32C), None),
    "split": (Params(1.0, 0.25, 1.0, 1e6), Quadrature(32, 48, 9, FP32C, radial_split=1), None),
    "poles": (Params(1.0, 1.0, 1.0, 1e6), Quadrature(24, 48, 9, FP32C),
              Propagators(((0.4, 1.0), (2.5, -0.3)), ((1.0, 0.6), (3.0, 0.4)))),
}


def scan(name):
    p, q, props = CASES[name]
    plan = gf.Plan(p, q, props)
    g = gf.scan_plan(plan, GRID, lanes=1).cpu().numpy().ravel()
    plan.close()
    return g


@pytest.mark.parametrize("name", CASES)
def test_values_are_the_recorded_ones(name):
    with np.load(GOLDEN) as f:
        want = f[name]
    got = scan(name)
    assert got.dtype == want.dtype and got.shape == want.shape
    differ = got.view(np.uint64) != want.view(np.uint64)
    assert not np.any(differ & ~np.isnan(want.view(np.float64))), int(differ.sum())
    assert np.array_equal(np.isnan(got), np.isnan(want))


def test_served_results_are_the_recorded_ones():
    """The serving kernels compute the same bits."""
    srv = gf.Server(budget_bytes=32 << 20)
    names = [n for n in CASES if CASES[n][2] is None]
    tickets = {srv.submit(CASES[n][0], GRID, CASES[n][1]): n for n in names}
    with np.load(GOLDEN) as f:
        for _ in names:
            t = srv.wait_any(30000.0)
            got, want = np.asarray(srv.result(t)).ravel(), f[tickets[t]]
            srv.release(t)
            assert np.array_equal(got[~np.isnan(want)], want[~np.isnan(want)])
    srv.close()
