"""The adjoint with one upstream gradient for all operators (stride 0), which
sums the operators first: against the oracle's adjoint at the edges of its
tiles, K parts and column groups, for every precision, flag and output.

Tolerances: relative Frobenius error <= 1e-5 (FP32, split-BF16), 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def rel(got, ref):
    got = got.double().cpu().numpy()
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


# m a multiple of 16 and of 4, odd; one row group and several; K = m, m', d*m'
# with and without parts; d = 1, 2, 4; two operators and more than four
SHAPES = [(96, 4, 80, 5), (257, 4, 130, 2), (131, 2, 77, 9), (320, 4, 272, 4), (150, 1, 90, 6), (5, 4, 3, 3),
          (544, 4, 48, 3)]


@pytest.mark.parametrize("precision", ["fp32", "fp64", "split_bf16"])
@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_shared_gradient(rot, oracle_mod, precision, symmetric, shape):
    m, d, mp, n = shape
    case = workloads.dense_case(m, d, mp, n, cfg=800 + m, dtype="f64" if precision == "fp64" else "f32",
                                symmetric=symmetric)
    dt = torch.float64 if precision == "fp64" else torch.float32
    G = np.random.default_rng(21).standard_normal((mp, mp)).astype(np.float32).astype(np.float64)
    U = torch.full((m * d, mp + 3), float("nan"), dtype=dt, device="cuda")[:, :mp]
    O = torch.full((n, m + 1, m + 5), float("nan"), dtype=dt, device="cuda")[:, :m, :m]
    U.copy_(torch.from_numpy(case.U))
    O.copy_(torch.from_numpy(case.O))
    Gd = torch.from_numpy(G).to(dt).cuda()
    dO, dU = rot.rotate_backward(U, O, d, Gd, precision, symmetric_O=symmetric)
    only_dO, none_dU = rot.rotate_backward(U, O, d, Gd, precision, need_dU=False, symmetric_O=symmetric)
    none_dO, only_dU = rot.rotate_backward(U, O, d, Gd, precision, need_dO=False, symmetric_O=symmetric)
    rdO, rdU = oracle_mod.adjoint(case.U, case.O, G, d)
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert none_dU is None and none_dO is None
    assert torch.equal(only_dO, dO) and torch.equal(only_dU, dU)
    assert rel(dU, rdU) <= tol
    for b in range(n):
        assert rel(dO[b], rdO[b]) <= tol
