"""GPU parity of the tiled regime's small batches, whose problems have many row
blocks: the merge split over row groups (sk_tiled_merge_rows) on both sides of
its rule and at ragged column counts, with and without an early stop, the
exact first v-update's merge, and one to three problems of rows wider than 2048
columns in the shared-cost sweep."""
import numpy as np
import pytest
import torch

import oracle
import paper_1907_01729_amd as sk
import workloads
from parity_util import LOSS_RTOL, POT_ATOL, gauge_fixed_errors, loss_rel_err

pytestmark = pytest.mark.gpu


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


@pytest.mark.parametrize("B, d1, d2, batched, tol, merge", [
    (1, 130, 65, False, 0.0, "rows"),    # 33 row blocks, one column past a slice
    (1, 128, 129, True, 0.0, "rows"),    # exactly 32 row blocks
    (1, 124, 129, True, 0.0, "cols"),    # 31
    (8, 300, 517, False, 2e-4, "rows"),  # compacted batch, split stop test
    (4, 259, 1030, False, 2e-4, "rows"),
    (3, 700, 250, True, 2e-4, "rows"),
    (1, 70, 2100, False, 0.0, "cols"),   # wide rows, too few for the shared-cost sweep
    (3, 150, 2305, False, 1e-3, "rows"),
    (1, 300, 2100, False, 0.0, "rows"),  # enough rows for the shared-cost sweep
    (3, 301, 2305, False, 1e-3, "rows"),
    (2, 70, 2901, False, 0.0, "cols"),
    (20, 300, 2700, False, 1e-3, "cols"),  # 75 row blocks, but 860 slices under an early stop
    (1, 64, 200, False, 0.0, "cols"),    # 16 row blocks: the exact merge of one wavefront
    (1, 68, 200, False, 0.0, "cols"),    # 17: of 16
])
def test_small_batch(B, d1, d2, batched, tol, merge):
    p = workloads.random_problem(900 + d1, B, d1, d2, 0.02 if d2 < 2000 else 0.05, 40, c_batched=batched,
                                 zero_frac=0.1, tol=tol)
    batched = batched and B > 1
    assert f"sk_tiled_merge_{merge}" in sk.sinkhorn_describe(B, d1, d2, int(batched), p.lam, p.n_iter, tol)
    out = {k: v.cpu().numpy() for k, v in
           sk.sinkhorn_forward(_t(p.mu), _t(p.nu), _t(p.C), p.lam, p.n_iter, tol).items()}
    if tol > 0:
        free = oracle.forward(p.mu, p.nu, p.C, p.lam, p.n_iter, tol=tol)
        assert np.all(np.abs(free["iters"] - out["iters"]) <= 1)
        assert out["iters"].min() < p.n_iter
    ref = oracle.forward(p.mu, p.nu, p.C, p.lam, p.n_iter, n_iter_b=out["iters"])
    ea, eb = gauge_fixed_errors(p.mu, p.nu, out["alpha"], out["beta"], ref["alpha"], ref["beta"])
    assert loss_rel_err(out["loss"], ref["loss"]) <= LOSS_RTOL and max(ea, eb) <= POT_ATOL
    again = sk.sinkhorn_forward(_t(p.mu), _t(p.nu), _t(p.C), p.lam, p.n_iter, tol)
    assert np.array_equal(again["alpha"].cpu().numpy(), out["alpha"])  # fixed summation order
