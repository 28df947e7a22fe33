"""Heat-bath CI over the range of its Davidson options: every form of the
subspace steps (up to 4, 8, 12 and 16 vectors, restarts that keep one, two and
four), the one-workgroup solve of small spaces and the device-wide one, against
the list form of the product; and a solve that runs out of steps."""
import numpy as np
import pytest

from paper_2307_10675_amd import ifci, synthetic
from tests.helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from tests.test_gpu_hbci_space import one_body  # noqa: E402


def _residual(plan, r):
    lo = ifci.hbci_options(max_det=max(2, r["n_det"]), max_nnz=2 * r["nnz"] + 1)
    c = r["c"].cpu().numpy()
    s = plan.hbci_sigma(0, r["dets"], r["c"], lo).cpu().numpy()
    e = float(c @ s)
    assert abs(np.linalg.norm(c) - 1.0) <= 1e-10
    return e, float(np.linalg.norm(s - e * c))


@pytest.mark.parametrize("m_max", [3, 4, 5, 9, 13, 16])
@pytest.mark.parametrize("bodies,eps1,large", [(3, 1e-3, False), (4, 1e-3, True), (5, 2e-3, True)])
def test_subspace_sizes(bodies, eps1, large, m_max):
    plan, p = one_body(bodies, 5200 + bodies)
    r = plan.hbci(0, ifci.hbci_options(eps1=eps1, m_max=m_max, max_dav=2000), with_space=True)
    print(f"[hbci] {2 * bodies} orbitals, m_max {m_max}: {r['n_det']} keys", flush=True)
    assert r["converged"] and r["residual"] <= 1e-6
    assert (r["n_det"] > 1024) == large
    _, rn = _residual(plan, r)
    # both see the residual to the rounding of sums of up to 1e4 terms
    assert abs(rn - r["residual"]) < 1e-9
    ref = plan.hbci(0, ifci.hbci_options(eps1=eps1, max_dav=2000))
    # the selected spaces may differ in keys whose |H c| lies within the error
    # of c (1e-6 / gap) of eps1, each worth less than eps1^2 / gap; with equal
    # spaces the energies agree to r_tol^2 / gap
    if ref["n_det"] == r["n_det"]:
        assert abs(ref["E_var"] - r["E_var"]) < 1e-10
    else:
        assert abs(ref["n_det"] - r["n_det"]) <= 0.01 * ref["n_det"]
        assert abs(ref["E_var"] - r["E_var"]) < abs(ref["n_det"] - r["n_det"]) * eps1 ** 2 * 10
    plan.close()


@pytest.mark.parametrize("bodies,eps1,converges", [(3, 1e-3, False), (4, 1e-3, True), (5, 2e-3, False)])
def test_subspace_of_two(bodies, eps1, converges):
    """A restart every step, from the Ritz vector alone: it need not converge,
    and says so; the reported residual is that of the vector handed back."""
    plan, p = one_body(bodies, 5200 + bodies)
    r = plan.hbci(0, ifci.hbci_options(eps1=eps1, m_max=2), with_space=True)
    print(f"[hbci] {2 * bodies} orbitals, m_max 2: {r['n_det']} keys, residual {r['residual']}", flush=True)
    assert r["converged"] or not converges
    assert r["residual"] <= 1e-6 or not r["converged"]
    _, rn = _residual(plan, r)
    assert abs(rn - r["residual"]) < 1e-9
    plan.close()


@pytest.mark.parametrize("max_dav", [1, 3, 13])
@pytest.mark.parametrize("bodies", [3, 5])
def test_out_of_steps(bodies, max_dav):
    """The reported residual is that of the vector and value handed back."""
    plan, p = one_body(bodies, 5300 + bodies)
    r = plan.hbci(0, ifci.hbci_options(eps1=1e-3, max_iter=2, max_dav=max_dav, r_tol=1e-13), with_space=True)
    print(f"[hbci] {2 * bodies} orbitals, max_dav {max_dav}: {r['n_det']} keys, residual {r['residual']}", flush=True)
    assert not r["converged"] and r["residual"] > 1e-13
    e, rn = _residual(plan, r)
    assert abs(rn - r["residual"]) < 1e-9
    plan.close()


def test_selection_beside_an_integral_that_is_not_a_number():
    """Elements that are NaN pass no threshold; all others are selected as
    before (from the reference alone: every single replacement but that of the
    NaN pair, and every double)."""
    import torch
    p = synthetic.merged(synthetic.chain(3, seed=5400, order=1))
    nocc = p.nocc[0]
    occ, emp = p.bodies[0][nocc - 1], p.bodies[0][nocc]
    o = ifci.hbci_options(max_det=1 << 12)
    got = []
    for bad in (False, True):
        h = p.h.copy()
        if bad:
            h[occ, emp] = h[emp, occ] = float("nan")
        plan = ifci.Plan(p, tuning=None).attach(h, p.eri)
        ref = plan.hbci(0, ifci.hbci_options(eps1=1e9, max_iter=1), with_space=True) if not bad else ref
        one = torch.ones(1, dtype=torch.float64, device="cuda")
        got.append(set(plan.hbci_select(0, ref["dets"], one, 1e-4, o).cpu().tolist()))
        plan.close()
    print(f"[hbci] {len(got[0])} keys, {len(got[1])} beside a NaN", flush=True)
    key = int(ref["dets"][0])
    order = sorted(p.bodies[0])
    bit = 1 << order.index(occ) | 1 << order.index(emp)
    assert got[1] == got[0] - {key ^ bit, key ^ (bit << 32)} and len(got[1]) == len(got[0]) - 2
