"""gf_scan_noalloc, whose node and group tables and subtraction coefficients are
computed on the device, against gf_scan with the tables of the host, at the edges of
the table kernels: the smallest and largest orders, odd rules (middle node), a
partly filled group, every rule and dimension, the split radial rule.

Tolerance: the scans' own rounding is within 64 eps kappa |G|, kappa the oracle's
condition number of the point; a Gauss-Legendre node or weight carries the
rounding of an n-step recurrence on either side, 2 n eps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1205_0752_amd as gf  # noqa: E402
from paper_1205_0752_amd.workloads import Grid, Params, Quadrature  # noqa: E402

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


def _quad(n_r, n_a, n_arc, rule, split=False):
    return Quadrature(n_r, n_a, n_arc, gf.FP64, rule, radial_split=split)


def _compare(params, quad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    side = 1 if quad.n_radial * quad.n_angular > 1 << 24 else 3  # the oracle sums every node
    grid = Grid(side, side, -6.0, 4.5, -2.0, 3.0)
    out = gf.empty_result(grid)
    gf.scan_noalloc(params, grid, quad, out)
    ref = gf.scan(params, grid, quad)
    torch.cuda.synchronize()
    g, g_ref = out.cpu().numpy().ravel(), ref.cpu().numpy().ravel()
    _, _, cond = oracle.scan(params, quad, grid, want_cond=True)
    ok = ~np.isnan(g_ref)
    assert np.array_equal(np.isnan(g), ~ok)
    n = max(quad.n_radial, quad.n_arc, quad.n_angular if quad.angular_rule == gf.GL else 0)
    bound = (64 + 4 * n) * EPS * cond[ok] * np.abs(g_ref[ok])
    assert np.all(np.abs(g - g_ref)[ok] <= bound)


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("quad", [
    _quad(1, 1, 1, gf.GL), _quad(2, 2, 2, gf.GL), _quad(3, 15, 3, gf.GL), _quad(65, 127, 64, gf.GL),
    _quad(64, 129, 65, gf.GC2), _quad(63, 16, 7, gf.GC1), _quad(33, 49, 16, gf.TANH_SINH),
    _quad(257, 4097, 16, gf.GC2), _quad(8192, 33, 1024, gf.GC2), _quad(16, 8192, 8, gf.GL),
    _quad(8192, 8192, 1024, gf.GL), _quad(96, 17, 9, gf.GL, True),
], ids=lambda q: f"{q.n_radial}x{q.n_angular}x{q.n_arc}")
def test_device_tables_equal_the_host_tables(quad, dim):
    params = Params(1 + 0.5j, 1 - 0.5j, 1.0, 1e4, 1.0, dimension=dim)
    if quad.radial_split:
        params = Params(1.0, 0.25, 1.0, 1e4, 1.0, dimension=dim)
    _compare(params, quad)


@pytest.mark.parametrize("mu2,taylor", [(0.0, 0), (1.5, -1), (1.5, 3), (1.5, 8)])
@pytest.mark.parametrize("quad", [_quad(64, 64, 16, gf.GC2), _quad(300, 24, 8, gf.GC2)],
                         ids=["groups", "pairs"])
def test_subtraction_coefficients_on_the_device(quad, mu2, taylor):
    _compare(Params(1.0, 0.25, mu2, 1e4, 1.0, taylor), quad)
