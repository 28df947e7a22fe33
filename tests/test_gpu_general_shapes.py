"""The product that stores E, on the only shapes that reach it device-wide
(15 orbitals, 16 away from half filling): products of vectors of any symmetry
against the plain FP64 product, and both device-wide solvers on them, through
thick restarts and the FP32-to-FP64 switch.  And the column kernel at 10o10e
against the same plain product, which shares no code with it."""
import numpy as np
import pytest

from paper_2307_10675_amd import ifci, synthetic
from tests.test_gpu_column_shapes import _problem, _product

pytestmark = pytest.mark.gpu

SHAPES = [(15, 1), (15, 2), (16, 2)]


@pytest.mark.parametrize("k,na", SHAPES)
def test_stored_product(k, na):
    import torch
    p = _problem(k, na, 300 + 16 * k + na)
    plan = ifci.Plan(p).attach(p.h, p.eri)
    n = int(round(plan.increment(0).n_det ** 0.5))
    c = np.random.default_rng(k + na).normal(size=(n, n))
    want = _product(p, k, na, c)
    cd = torch.tensor(c.reshape(-1), device="cuda")
    print(f"[stored] {k}o{na} strings {n}", flush=True)
    scale = max(np.abs(want).max(), 1.0) * max(1.0, np.abs(c).max())
    for precision, tol in ((ifci.FP64, 1e-12 * n), (ifci.MIXED, 2e-5)):
        got = plan.sigma(0, cd, precision=precision).cpu().numpy().reshape(n, n)
        assert np.abs(got - want).max() <= tol * scale
    plan.close()


@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["batched", "plain"])
@pytest.mark.parametrize("precision", [ifci.FP64, ifci.MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("k,na", SHAPES)
def test_solve(k, na, precision, solver):
    p = _problem(k, na, 400 + 16 * k + na)
    space = 5
    plan, r = ifci.solve(p, precision=precision, solver=solver, max_space=space, r_tol=1e-8, r_tol_inner=1e-4,
                         max_iter=900)
    print(f"[stored] solve {k}o{na} precision {precision} solver {solver}: {int(r['iters'][0])} iterations", flush=True)
    assert int(r["status"][0]) == ifci.INC_DONE
    assert int(r["iters"][0]) > space  # at least one thick restart
    n = int(round(plan.increment(0).n_det ** 0.5))
    c = plan.vector(0).cpu().numpy().reshape(n, n)
    Hc = _product(p, k, na, c)
    e = float(np.vdot(c, Hc))
    assert abs(e - float(r["E"][0])) <= 1e-11
    assert np.linalg.norm(Hc - e * c) <= 1.1e-8
    # the lowest root: the other solver and precision agree to r_tol^2 / gap
    _, ref = ifci.solve(p, r_tol=1e-8, max_iter=900)
    assert abs(float(ref["E"][0]) - float(r["E"][0])) <= 1e-10
    plan.close()


def test_column_product_of_symmetric_vectors():
    import torch
    k, na = 10, 5
    p = synthetic.single(k, 2 * k, 4221)
    plan = ifci.Plan(p).attach(p.h, p.eri)
    n = int(round(plan.increment(0).n_det ** 0.5))
    c = np.random.default_rng(11).normal(size=(n, n))
    c = c + c.T
    want = _product(p, k, na, c)
    a, b = np.triu_indices(n)
    s2 = np.where(a == b, 1.0, np.sqrt(2.0))
    packed = np.empty(n * (n + 1) // 2)
    packed[b * (b + 1) // 2 + a] = s2 * c[a, b]
    cd = torch.tensor(packed, device="cuda")
    scale = np.abs(want).max() * max(1.0, np.abs(c).max())
    for precision, tol in ((ifci.FP64, 1e-12 * n), (ifci.MIXED, 2e-5)):
        got = plan.sigma_sector(0, cd, precision=precision).cpu().numpy()
        assert np.abs(got[b * (b + 1) // 2 + a] - s2 * want[a, b]).max() <= tol * scale
    plan.close()
