"""Products of few operators of the two blocks (rot_expect_cross) around the
pair tiles of 8 x 8, the switch to the matrix product and short sums, and
one-point values around the unrolled steps, against the definition in FP64.

Tolerance: 1e-12 of the norm of psi (one) times the operators' norms."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,mR,nl,nr", [(3, 2, 1, 1), (7, 20, 8, 9), (20, 23, 9, 1), (24, 40, 32, 32), (24, 33, 33, 5),
                                        (40, 64, 3, 17), (30, 91, 7, 8)])
def test_cross_pairs(rot, m, mR, nl, nr):
    rng = np.random.default_rng(m * 100 + mR)
    d = 4
    psi = rng.standard_normal((m * d, d * mR))
    psi /= np.linalg.norm(psi)
    L, R = rng.standard_normal((nl, m, m)), rng.standard_normal((nr, mR, mR))
    got = rot.expect_cross(*(torch.from_numpy(x).cuda() for x in (psi, L, R)), d, d).cpu().numpy()
    X = psi.reshape(m, d, d, mR)
    left = (L.transpose(0, 2, 1) @ X.reshape(m, -1)).reshape(nl, -1)
    right = (X.reshape(-1, mR) @ R.transpose(0, 2, 1)).reshape(nr, -1)
    ref = left @ right.T
    scale = np.linalg.norm(L, axis=(1, 2))[:, None] * np.linalg.norm(R, axis=(1, 2))[None]
    assert (np.abs(got - ref) / scale).max() <= 1e-12


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m", [1, 45, 46, 127, 129, 200])
def test_one_point_values(rot, m, dtype):
    rng = np.random.default_rng(m)
    d, n = 2, 3
    psi = rng.standard_normal((m * d, 3 * m + 1))
    psi /= np.linalg.norm(psi)
    Z = torch.from_numpy(rng.standard_normal((n, m, m))).to(dtype).cuda()
    got = rot.expect_block(torch.from_numpy(psi).cuda(), Z, d).cpu().numpy()
    Z64 = Z.double().cpu().numpy()
    X = psi.reshape(m, -1)
    ref = ((X @ X.T) * Z64).sum((1, 2))
    assert (np.abs(got - ref) / np.linalg.norm(Z64, axis=(1, 2))).max() <= 1e-12
