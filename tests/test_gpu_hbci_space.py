"""The large-space forms of the HBCI solve against its own list forms: the
blocked product of H (full spaces of more than 1024 keys, windows of 8192
entries of x) against ifci_hbci_sigma over the returned keys, the PT2 sum over
the array of string pairs against ifci_hbci_pt2 and against the same solve
with a table too small for the array, and the row form of the product (spaces
past the blocked form's limits) against the exact energy of the FCI solver.

Tolerances: c solves H c = e c to the residual that the solve reports, which
both products see to rounding (sums of up to 1e4 terms of order 1, 1e-11); the
PT2 sums differ in the order of their additions only (1e-11).
"""
import numpy as np
import pytest

from paper_2307_10675_amd import synthetic
from tests.helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2307_10675_amd import ifci  # noqa: E402


def one_body(bodies, seed):
    p = synthetic.merged(synthetic.chain(bodies, seed=seed, order=1))
    return ifci.Plan(p, tuning=None).attach(p.h, p.eri), p


@pytest.mark.parametrize("bodies,eps1", [(4, 1e-3), (5, 1e-3), (6, 2e-3), (7, 2e-3)])
def test_solve_against_the_list_forms(bodies, eps1):
    plan, p = one_body(bodies, 5100 + bodies)
    o = ifci.hbci_options(eps1=eps1, eps2=1e-6)
    r = plan.hbci(0, o, with_space=True)
    print(f"[space] {2 * bodies} orbitals, {r['n_det']} keys, {r['nnz']} nonzeros", flush=True)
    assert r["converged"]
    lo = ifci.hbci_options(max_det=r["n_det"], max_nnz=2 * r["nnz"] + 1)
    s = plan.hbci_sigma(0, r["dets"], r["c"], lo).cpu().numpy()
    c = r["c"].cpu().numpy()
    e = float(c @ s)
    assert abs(np.linalg.norm(s - e * c) - r["residual"]) < 1e-9
    e2, n_ext = plan.hbci_pt2(0, r["dets"], r["c"], r["E_var"], 1e-6, o)
    assert n_ext == r["n_ext"] and abs(e2 - r["E_pt2"]) < 1e-11
    plan.close()


def test_pt2_table_where_the_array_does_not_fit():
    plan, p = one_body(6, 5106)
    wide = plan.hbci(0, ifci.hbci_options(eps1=5e-3, eps2=1e-3))
    cap = max(wide["n_ext"], 1)
    assert 4 * 2 * cap < 924 * 924  # fewer than two array places for each table slot
    tight = plan.hbci(0, ifci.hbci_options(eps1=5e-3, eps2=1e-3, max_ext=cap))
    assert tight["n_ext"] == wide["n_ext"] and tight["n_det"] == wide["n_det"]
    assert abs(tight["E_pt2"] - wide["E_pt2"]) < 1e-11
    plan.close()


def test_row_form_of_the_product():
    """12o12e at eps1 = 0: all 853776 determinants, past the blocked form."""
    plan, p = one_body(6, 5112)
    e, _, _, _ = plan.davidson()
    r = plan.hbci(0, ifci.hbci_options(eps1=0.0, eps2=0.0, max_nnz=800_000_000, max_ext=1 << 20, r_tol=1e-6))
    print(f"[space] {r['n_det']} keys, {r['nnz']} nonzeros", flush=True)
    assert r["converged"] and r["n_det"] > 1 << 19
    assert abs(r["E_var"] - float(e[0])) < 1e-9
    plan.close()
