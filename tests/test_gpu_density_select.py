"""The choice of the kept states over sectors: ties, negative zeros and counts
at the edges of the eight-bit passes, against a sort on the host.

Eigenvalues of diagonal density matrices are exact, so the counts are compared
as whole numbers and the weight left out to the last bits of a short sum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", [0, 1, 63, 64, 100, 255, 256, 400, 511, 512])
def test_kept_counts(rot, keep):
    """Eigenvalues equal across sectors go to the earlier sector; zeros of
    rank-deficient sectors come last."""
    rng = np.random.default_rng(71)
    values = [2.0 ** -rng.integers(0, 40, n).astype(float) for n in (64, 200, 7, 130, 1, 110)]
    values[1][150:] = 0.0
    psi = [torch.from_numpy(np.diag(np.sqrt(v))).cuda() for v in values]
    w, _, kept, eps = rot.density_basis(psi, keep)
    squares = [np.sort(np.sqrt(v) ** 2)[::-1] for v in values]
    for got, want in zip(w, squares):
        assert np.array_equal(got.cpu().numpy(), want)
    flat = sorted(((-x, k) for k, v in enumerate(squares) for x in v))[:keep]
    want = np.bincount([k for _, k in flat], minlength=len(values))
    assert kept.tolist() == want.tolist()
    rest = sum(v[c:].sum() for v, c in zip(squares, want))
    assert abs(eps.item() - rest) <= 1e-13 * max(rest, 1e-300)
