"""Products in 64 x 64 tiles: rotations whose extents end on and next to the
edges of tiles and K slices, operands at odd addresses and strides, row
strides past 32-bit offsets, and the measurements formed from diagonal blocks.

Tolerances: relative Frobenius error per operator <= 1e-5 (FP32), 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "fp64": 1e-12}


def rel_fro(got, ref):
    axes = tuple(range(1, ref.ndim))
    return np.sqrt(((got - ref) ** 2).sum(axes)) / np.sqrt((ref ** 2).sum(axes))


def at_odd_address(a, dt, pad):
    """Device copy with `pad` elements before it and after every row, NaN."""
    a = np.asarray(a)
    rows = int(np.prod(a.shape[:-1]))
    buf = torch.full((rows * (a.shape[-1] + pad) + pad + 1,), float("nan"), dtype=dt, device="cuda")
    view = buf[pad:pad + rows * (a.shape[-1] + pad)].view(*a.shape[:-1], a.shape[-1] + pad)[..., : a.shape[-1]]
    view.copy_(torch.from_numpy(np.ascontiguousarray(a)).to(dt))
    return view


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("symmetric", [False, True])
@pytest.mark.parametrize("shape,pad", [((65, 4, 64, 3), 0), ((63, 4, 65, 2), 1), ((127, 3, 129, 2), 3),
                                       ((16, 1, 16, 1), 1), ((17, 4, 68, 5), 2), ((128, 4, 192, 2), 0),
                                       ((193, 2, 131, 4), 1), ((2, 4, 3, 70), 1)])
def test_edges(rot, oracle_mod, precision, symmetric, shape, pad):
    m, d, mp, n = shape
    dt = torch.float64 if precision == "fp64" else torch.float32
    case = workloads.dense_case(m, d, mp, n, cfg=900 + m, dtype="f64" if precision == "fp64" else "f32",
                                symmetric=symmetric)
    out = rot.rotate(at_odd_address(case.U, dt, pad), at_odd_address(case.O, dt, pad), d, precision,
                     symmetric_O=symmetric)
    ref = oracle_mod.rotate(case.U, case.O, d)
    assert rel_fro(out.double().cpu().numpy(), ref).max() <= TOL[precision]
    if symmetric:
        assert torch.equal(out, out.transpose(1, 2))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_row_strides_past_32_bit_offsets(rot, oracle_mod, precision):
    m, d, mp = 5, 2, 4
    dt = torch.float64 if precision == "fp64" else torch.float32
    case = workloads.dense_case(m, d, mp, 1, cfg=930, dtype="f64" if precision == "fp64" else "f32", symmetric=False)
    ld = 2 ** 24 + 3  # 64 rows span over 4 GiB
    O = torch.empty((1, m, ld), dtype=dt, device="cuda")[:, :, :m]
    O.copy_(torch.from_numpy(case.O).to(dt))
    out = rot.rotate(torch.from_numpy(case.U).to(dt).cuda(), O, d, precision)
    ref = oracle_mod.rotate(case.U, case.O, d)
    assert rel_fro(out.double().cpu().numpy(), ref).max() <= TOL[precision]


@pytest.mark.parametrize("m,d,mR,dR,nL,nR", [(20, 4, 33, 4, 3, 2), (65, 2, 64, 3, 1, 5), (130, 4, 67, 1, 2, 2),
                                             (9, 3, 5, 2, 7, 1)])
def test_cross_block_products(rot, oracle_mod, m, d, mR, dR, nL, nR):
    g = np.random.default_rng(940 + m)
    psi = g.standard_normal((m * d, dR * mR))
    psi /= np.linalg.norm(psi)
    Z, W = g.standard_normal((nL, m, m)), g.standard_normal((nR, mR, mR))
    dev = [torch.from_numpy(x).cuda() for x in (psi, Z, W)]
    ref = np.asarray(oracle_mod.expect_cross(psi, Z, W, d, dR))
    whole = rot.expect_cross(*dev, d, dR)
    assert np.abs(whole.cpu().numpy() - ref).max() <= 1e-12 * max(1.0, np.abs(ref).max())
    assert torch.equal(whole, rot.expect_cross(*dev, d, dR, ops_per_chunk=1))
