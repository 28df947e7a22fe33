"""The one-wave eigen-decomposition (ifci_sno_orbitals returns all its
vectors): off-diagonal part of R^T g R and orthogonality of R at the level of
rounding, for clusters of eigenvalues of every width, where a sweep of
rotations does not make the next one's pivots quadratically small."""
import numpy as np
import pytest

from paper_2307_10675_amd import ifci

pytestmark = pytest.mark.gpu


def _vectors(g):
    """R [N, m, m] of the matrices g [N, m, m] (eigenvectors as columns)."""
    import torch
    N, m, _ = g.shape
    gd = torch.tensor(g, device="cuda")
    vir = torch.arange(m, dtype=torch.int32, device="cuda")
    occ = torch.arange(N, dtype=torch.int32, device="cuda").reshape(N, 1).contiguous()
    rot = torch.empty((N, m, m), dtype=torch.float64, device="cuda")
    keep = torch.empty(N, dtype=torch.int32, device="cuda")
    ifci._check(ifci.lib().ifci_sno_orbitals(ifci._ptr(gd), m, ifci._ptr(vir), m, ifci._ptr(occ), N, 1, 300.0,
                                             ifci._ptr(rot), ifci._ptr(keep), ifci._stream()))
    torch.cuda.synchronize()
    assert (keep.cpu().numpy() == m).all()
    return rot.cpu().numpy()


def _check(g, m):
    R = _vectors(g).astype(np.longdouble)
    D = np.einsum("nia,nij,njb->nab", R, g.astype(np.longdouble), R)
    off = np.sqrt(((D * (1 - np.eye(m))) ** 2).sum((1, 2)))
    f = np.sqrt((g ** 2).sum((1, 2)))
    # rounding, at most: up to 8 sweeps of m - 1 rounds (m for an odd m), each a
    # two-sided rotation whose backward error is at most 6 units of rounding
    rounds = 8 * (m - 1 + m % 2)
    assert (off / f).max() <= rounds * 6 * 1.11e-16
    assert np.abs(np.einsum("nia,nib->nab", R, R) - np.eye(m)).max() <= rounds * 6 * 1.11e-16


@pytest.mark.parametrize("width", [1.0, 1e-4, 1e-6, 1e-8, 1e-9, 1e-10])
@pytest.mark.parametrize("m", [2, 3, 4, 7, 8, 12, 16])
def test_one_cluster(m, width):
    rng = np.random.default_rng(m)
    a = rng.normal(size=(64, m, m))
    a = a + a.transpose(0, 2, 1)
    print(f"[jacobi] {m} x {m}, width {width}", flush=True)
    _check((16.0 if width == 1.0 else 1.0) * np.eye(m) + width * a, m)


@pytest.mark.parametrize("m", [4, 7, 8, 12, 16])
def test_two_clusters(m):
    """Half of the eigenvalues near 1, half near 0.01, each within 1e-9."""
    rng = np.random.default_rng(100 + m)
    q = np.linalg.qr(rng.normal(size=(64, m, m)))[0]
    a = 1e-9 * rng.normal(size=(64, m, m))
    g = q @ (np.where(np.arange(m) < m // 2, 1.0, 1e-2)[None, :, None] * q.transpose(0, 2, 1))
    print(f"[jacobi] {m} x {m}, two clusters", flush=True)
    _check((g + g.transpose(0, 2, 1)) / 2 + a + a.transpose(0, 2, 1), m)
