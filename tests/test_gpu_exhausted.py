"""Device-wide Davidson where the space that H reaches from the start vector
is spanned before the residual meets the tolerance: two interacting orbitals
(a space of three symmetric combinations) among inert ones, which carry a
diagonal h and no two-electron integrals.  A correction then lies in the span
of the basis, and there is no direction left."""
import numpy as np
import pytest

from oracle import ifci as oifci
from paper_2307_10675_amd import ifci, synthetic

pytestmark = pytest.mark.gpu


def _problem(k, na, seed):
    """k orbitals, na of them occupied; orbitals na - 1 and na interact.
    Returns the problem and its exact energy."""
    h2, eri2 = synthetic.integrals(2, 4, seed)
    h = np.diag(np.arange(k, dtype=float) * 1.5 - 8.0)
    at = np.array([na - 1, na])
    h[np.ix_(at, at)] = h2 + np.diag(h[at, at])
    eri = np.zeros((k,) * 4)
    eri[np.ix_(at, at, at, at)] = eri2
    p = synthetic.Problem(h, eri, [list(range(k))], [na], 1)
    two = synthetic.Problem(h[np.ix_(at, at)], eri2, [[0, 1]], [1], 1)
    return p, oifci.run(two)["E"][(0,)] + 2.0 * sum(h[i, i] for i in range(na - 1))


@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("space", [3, 4, 12])
@pytest.mark.parametrize("k,na", [(9, 4), (10, 5), (15, 1)])
def test_ends_when_no_direction_is_left(k, na, space, solver):
    """FP64, a tolerance that rounding does not reach."""
    p, want = _problem(k, na, 31 + k)
    print(f"[exhausted] {k}o{na} max_space {space} solver {solver}", flush=True)
    _, r = ifci.solve(p, solver=solver, max_space=space, r_tol=1e-30, max_iter=80)
    # three directions and the rounding of the third: far from 80 iterations
    assert int(r["iters"][0]) <= 12
    assert int(r["status"][0]) in (ifci.INC_NOT_CONVERGED, ifci.INC_DONE)
    assert float(r["resid"][0]) <= 1e-12
    assert abs(float(r["E"][0]) - want) <= 1e-12 * abs(want)


@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("k,na", [(9, 4), (10, 5), (15, 1)])
def test_first_stage_without_a_direction_goes_on_in_fp64(k, na, solver):
    """The FP32 stage cannot reach r_tol_inner: the FP64 stage takes over."""
    p, want = _problem(k, na, 57 + k)
    print(f"[exhausted] mixed {k}o{na} solver {solver}", flush=True)
    _, r = ifci.solve(p, solver=solver, precision=ifci.MIXED, r_tol=1e-10, r_tol_inner=1e-20, max_iter=80)
    assert int(r["status"][0]) == ifci.INC_DONE
    assert int(r["iters"][0]) <= 30
    assert abs(float(r["E"][0]) - want) <= 1e-12 * abs(want)
