"""Subspace eigenproblem of the Davidson solvers at the sizes where its
elimination is unrolled differently (4, 8, 12, 16) and around them, on chip
and device-wide, against the oracle's energies."""
import numpy as np
import pytest

from oracle import ifci as oifci
from paper_2307_10675_amd import ifci, synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def refs():
    out = {}
    # a chain, and non-interacting bodies (degenerate subspace values: the
    # full decomposition in place of the secular equation)
    for name, p in (("chain", synthetic.chain(3, seed=611, order=3)), ("separable", synthetic.separable(3, seed=612,
                                                                                                       order=3))):
        r = oifci.run(p)
        out[name] = p, np.array([r["E"][S] for S in oifci.increments(3, 3)])
    return out


@pytest.mark.parametrize("space", [2, 4, 5, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("solver", [ifci.BATCHED, ifci.PLAIN], ids=["on_chip", "device_wide"])
@pytest.mark.parametrize("name", ["chain", "separable"])
def test_subspace_sizes(refs, name, solver, space):
    import torch
    p, want = refs[name]
    for n_guess in (0, 64):
        print(f"[subspace] {name} solver {solver} max_space {space} n_guess {n_guess}", flush=True)
        _, r = ifci.solve(p, solver=solver, max_space=space, n_guess=n_guess, r_tol=1e-7, max_iter=900)
        torch.cuda.synchronize()
        assert (r["status"].cpu().numpy() == ifci.INC_DONE).all()
        # |E - E_exact| <= r_tol^2 / gap = 1e-14 / gap, far below the bar for any gap above 1e-5
        assert np.abs(r["E"].cpu().numpy() - want).max() <= 1e-9
