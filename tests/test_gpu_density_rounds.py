"""The density step over sectors of every number of 32-wide blocks around the
padding steps, alone and together (sectors with fewer blocks sit out part of
each sweep): eigenvalues, residuals and orthonormality in FP64 against LAPACK.

Tolerances, relative to the largest eigenvalue: a few n rounding errors
(n <= 300) for eigenvalues and residuals, 1e-12 for orthonormality."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def psi_of(n, r, scale, seed):
    return np.random.default_rng(seed).standard_normal((n, r)) * scale


def check(psi, w, V):
    rho = psi @ psi.T
    ref = np.linalg.eigvalsh(rho)[::-1]
    w, V = w.cpu().numpy(), V.cpu().numpy()
    top = max(ref[0], np.finfo(float).tiny)
    assert np.all(np.diff(w) <= 0)
    assert np.abs(w - ref).max() <= 1e-13 * top
    assert np.abs(rho @ V - V * w[None, :]).max() <= 1e-13 * top
    assert np.abs(V.T @ V - np.eye(len(w))).max() <= 1e-12


@pytest.mark.parametrize("n", [1, 2, 31, 33, 64, 65, 128, 129, 192, 193, 256, 300])
def test_single_sector(rot, n):
    psi = psi_of(n, n + 5, 1.0 / n, 50 + n)
    w, V, kept, eps = rot.density_basis([torch.from_numpy(psi).cuda()], n)
    check(psi, w[0], V[0])
    assert kept.tolist() == [n] and eps.item() == 0.0


def test_sectors_of_all_sizes_together(rot):
    """Mixed block counts in one call, rank-deficient and diagonal sectors among
    them (finished at once, or never rotating), very small and large norms."""
    shapes = [(300, 310, 1.0), (40, 50, 1e-3), (129, 20, 1.0), (64, 64, 1e-90), (200, 230, 1e80), (3, 1, 1.0),
              (96, 100, 1.0), (257, 260, 1.0)]
    psi = [psi_of(n, r, s / n, 70 + k) for k, (n, r, s) in enumerate(shapes)]
    psi.append(np.diag(np.arange(1.0, 101.0)))
    w, V, kept, eps = rot.density_basis([torch.from_numpy(p).cuda() for p in psi], 500)
    for k, p in enumerate(psi):
        check(p, w[k], V[k])
    assert int(kept.sum()) == 500
