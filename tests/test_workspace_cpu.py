"""Workspace of a plan: what its kernels use of it, and no product's
intermediate where the column kernels form it on chip."""
import numpy as np
import pytest

from paper_2307_10675_amd import ifci, synthetic


def _bytes(k, na, solver):
    p = synthetic.Problem(np.zeros((k, k)), None, [list(range(k))], [na], 1)
    plan = ifci.Plan(p, solver=solver, max_space=2)
    n_str = int(round(plan.increment(0).n_det ** 0.5))
    ws = plan.info()["workspace_bytes"]
    plan.close()
    return ws, n_str


@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("k,na", [(11, 5), (12, 6), (13, 4), (14, 7)])
def test_column_shapes_reserve_no_intermediate(k, na, solver):
    ws, n = _bytes(k, na, solver)
    sym = n * (n + 1) // 2
    # basis, sigma, diagonal and Ritz vector (6 packed vectors at a subspace of
    # two), four temporaries; C and S of two products and one slot of the
    # batched solver (C, S, two vectors): 4 and 4 matrices; tables and partial
    # sums of at most 8 MB
    assert ws <= 8 * (10 * sym + 8 * n * n) + (8 << 20)


@pytest.mark.parametrize("k,na", [(15, 2), (16, 2)])
def test_stored_product_has_its_intermediate(k, na):
    ws, n = _bytes(k, na, ifci.PLAIN)
    assert ws >= 8 * (k * (k + 1) // 2) * n * n
