"""Device-wide solves at odd orbital counts and away from half filling repeat
to the bit: energies, residuals, iteration counts and vectors of the same
call made again on the same plan.  (Half-filled increments of 10, 12, 14 and
16 orbitals agree to rounding only.)"""
import numpy as np
import pytest

from paper_2307_10675_amd import ifci
from tests.test_gpu_column_shapes import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("precision", [ifci.FP64, ifci.MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("k,na", [(9, 4), (10, 4), (11, 5), (12, 3), (13, 3), (14, 2)])
def test_solve_repeats_to_the_bit(k, na, precision, solver):
    import torch
    p = _problem(k, na, 500 + 16 * k + na)
    plan = ifci.Plan(p, precision=precision, solver=solver, r_tol=1e-8, r_tol_inner=1e-5,
                     max_iter=600).attach(p.h, p.eri)
    print(f"[repeat] {k}o{na} precision {precision} solver {solver}", flush=True)
    first = None
    for _ in range(4):
        e, st, it, rs = plan.davidson()
        got = [t.cpu() for t in (e, st, it, rs, plan.vector(0))]
        assert int(got[1][0]) == ifci.INC_DONE
        first = first or got
        for a, b in zip(first, got):
            assert torch.equal(a, b), float((a - b).abs().max())
    plan.close()
