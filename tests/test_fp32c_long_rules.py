"""FP32C scans of long rules: the six-wave kernel, taken without an LDS table (16 lanes per
point and more, or over 512 pairs) from 2048 pairs a lane on where there is more than one round of
waves, runs the same operations as the other kernel, so its results have the same bits at
equal lanes."""
import numpy as np
import pytest

import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import FP32C, Grid, Params, Quadrature

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("lanes,side,n_r,n_a", [
    (16, 160, 120, 512),   # 9 nodes x 256 pairs a lane, 6,400 tiles
    (16, 160, 120, 501),   # 250 pairs and a middle node
    (32, 110, 250, 512), (64, 72, 500, 512),
    (1, 640, 6, 1026), (2, 460, 9, 1026), (8, 260, 30, 1026)])
@pytest.mark.parametrize("taylor", [0, 2])
def test_same_bits_beside_a_small_scan(lanes, side, n_r, n_a, taylor):
    """The scan's lowest rows alone, a grid of one round of waves at most, run the other
    kernel: the same points to the same bits (step 2^-6, exact in both boxes)."""
    p = Params(1.0, 0.25, 1.0, 1e6, 1.0, taylor)
    q = Quadrature(n_r, n_a, 8, FP32C)
    h = 2.0 ** -6
    grid = Grid(side, side, -4.0, -4.0 + side * h, -1.0, -1.0 + side * h)
    few = Grid(side, 16, -4.0, -4.0 + side * h, -1.0, -1.0 + 16 * h)
    plan = gf.Plan(p, q)
    a = gf.scan_plan(plan, grid, lanes=lanes).cpu().numpy()[:16]
    b = gf.scan_plan(plan, few, lanes=lanes).cpu().numpy()
    plan.close()
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)])


def test_served_long_rule_equals_the_scan():
    p, q, grid = Params(1.0, 0.25, 1.0, 1e6), Quadrature(16, 1030, 8, FP32C), Grid(48, 40, -8., 4., -4., 4.)
    plan = gf.Plan(p, q)
    want = gf.scan_plan(plan, grid, lanes=1).cpu().numpy().ravel()
    plan.close()
    srv = gf.Server(budget_bytes=16 << 20)
    t = srv.submit(p, grid, q)
    assert srv.wait_any(30000.0) == t
    got = np.asarray(srv.result(t)).ravel()
    srv.release(t)
    srv.close()
    ok = ~np.isnan(want)
    assert np.array_equal(got[ok], want[ok]) and np.all(np.isnan(got[~ok]))
