"""The server's buffers for group coefficients stand outside its budget: requests of more
rules than one buffer holds are admitted side by side while none of them is released,
and their results equal the scans'."""
import numpy as np
import pytest

import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import FP32C, FP64, Grid, Params, Quadrature

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

P, GRID = Params(1.0, 0.25, 1.0, 1e4), Grid(9, 7, -6.0, 3.0, -2.0, 2.5)


def test_more_rules_than_one_buffer_holds():
    # 128 KiB a rule, 31 to a buffer of 4 MiB; twice over, FP32C and FP64 requests in turn
    orders = range(8192 - 40, 8192)
    srv = gf.Server(budget_bytes=64 << 20, max_inflight=256)
    first = [srv.submit(P, GRID, Quadrature(6, n, 3, prec)) for n in orders for prec in (FP32C, FP64)]
    assert all(srv.wait(t, 5000.0) for t in first)
    got = np.asarray(srv.result(first[-1])).ravel()
    plan = gf.Plan(P, Quadrature(6, orders[-1], 3, FP64))
    want = gf.scan_plan(plan, GRID, lanes=1).cpu().numpy().ravel()
    plan.close()
    assert np.array_equal(got, want, equal_nan=True)
    for t in first:
        srv.release(t)
    # released rules' ranges serve others
    again = [srv.submit(P, GRID, Quadrature(6, n - 40, 3, FP64)) for n in orders]
    assert all(srv.wait(t, 5000.0) for t in again)
    srv.close()
