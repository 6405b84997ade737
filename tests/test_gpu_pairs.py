"""FP32 rotations that run on FP16 pairs: parity with the oracle where tiles,
blocks and slabs end, on every layout the entry point takes, and the
operators those kernels leave to the FP32 ones.

Tolerance: the FP32 bound, relative Frobenius error per operator <= 1e-5."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def rel_fro(got, ref):
    axes = tuple(range(1, ref.ndim))
    return np.sqrt(((got - ref) ** 2).sum(axes)) / np.sqrt((ref ** 2).sum(axes))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).float().cuda()


def smallest_batch(m, d, mp):
    """Operators of a shape from which a batch takes the pairs (4 GFLOP)."""
    return int(4e9 / (2 * m * d * mp * (m + mp))) + 1


def used_pairs(rot, call):
    rot.profile_enable(True)
    out = call()
    torch.cuda.synchronize()
    kinds = rot.profile_read()
    rot.profile_enable(False)
    return out, "stage1_f16x3" in kinds


# every remainder of the 64-row M tiles (m' and d*m'), of the 32-column
# blocks (m, m') and of the 16-wide slabs (m, m*d); a last N tile with one
# block; d = 1, 2, 3, 8; K split into parts; one operator
EDGES = [(64, 4, 64), (65, 4, 97), (79, 4, 129), (96, 3, 191), (129, 1, 128), (145, 2, 250), (100, 8, 333),
         (257, 4, 193), (300, 4, 257), (404, 4, 391)]


@pytest.mark.parametrize("shape", EDGES)
@pytest.mark.parametrize("symmetric", [False, True])
def test_pairs_parity(rot, oracle_mod, shape, symmetric):
    m, d, mp = shape
    n = smallest_batch(m, d, mp)
    case = workloads.dense_case(m, d, mp, n, cfg=700 + m, symmetric=symmetric)
    U, O = dev(case.U), dev(case.O)
    out, pairs = used_pairs(rot, lambda: rot.rotate(U, O, d, "fp32", symmetric_O=symmetric))
    assert pairs
    assert rel_fro(out.double().cpu().numpy(), oracle_mod.rotate(case.U, case.O, d)).max() <= TOL32
    if symmetric:
        assert torch.equal(out, out.transpose(1, 2))


@pytest.mark.parametrize("symmetric", [False, True])
def test_pairs_padded_layouts(rot, oracle_mod, symmetric):
    """Padded rows and matrices filled with NaN, odd leading dimensions; the
    output's padding is kept."""
    m, d, mp = 131, 4, 118
    n = smallest_batch(m, d, mp)
    case = workloads.dense_case(m, d, mp, n, cfg=730, symmetric=symmetric)
    Ub = torch.full((m * d, mp + 3), float("nan"), device="cuda")
    Ob = torch.full((n, m + 2, m + 5), float("nan"), device="cuda")
    outb = torch.full((n, mp + 1, mp + 9), 7.0, device="cuda")
    U, O, out = Ub[:, :mp], Ob[:, :m, :m], outb[:, :mp, :mp]
    U.copy_(dev(case.U))
    O.copy_(dev(case.O))
    _, pairs = used_pairs(rot, lambda: rot.rotate(U, O, d, "fp32", out=out, symmetric_O=symmetric))
    assert pairs
    assert rel_fro(out.double().cpu().numpy(), oracle_mod.rotate(case.U, case.O, d)).max() <= TOL32
    kept = torch.ones_like(outb, dtype=torch.bool)
    kept[:, :mp, :mp] = False
    assert torch.all(outb[kept] == 7.0)


def test_pairs_leave_out_of_range_operators(rot, oracle_mod):
    """Operators with infinities, NaN or rows of very different size are
    computed by the FP32 kernels, the others of the batch are not affected;
    scaled operators keep their accuracy over FP32's range."""
    m, d, mp = 150, 4, 130
    n = smallest_batch(m, d, mp)
    case = workloads.dense_case(m, d, mp, n, cfg=740, symmetric=False)
    O = case.O.copy()
    O[3] *= 2.0 ** -116
    O[4] *= 2.0 ** 100
    O[6, 10, :] *= 2.0 ** 30
    O[7] = 0
    O[7, 2, 5] = 1.0
    O[9] *= np.logspace(0, -8, m)[:, None]
    O = O.astype(np.float32).astype(np.float64)
    ref = oracle_mod.rotate(case.U, O, d)
    bad = dev(O)
    bad[1, 3, 5] = float("inf")
    bad[2, 7, :] = float("nan")
    out, pairs = used_pairs(rot, lambda: rot.rotate(dev(case.U), bad, d, "fp32"))
    assert pairs
    got = out.double().cpu().numpy()
    rest = [b for b in range(n) if b not in (1, 2)]
    assert rel_fro(got[rest], ref[rest]).max() <= TOL32
    assert np.isnan(got[2]).all()
    alone = rot.rotate(dev(case.U), bad[1:2].contiguous(), d, "fp32").cpu()  # one operator: FP32 kernels
    assert torch.equal(torch.isnan(out[1]).cpu(), torch.isnan(alone[0]))
    assert torch.equal(torch.isinf(out[1]).cpu(), torch.isinf(alone[0]))
    # a NaN in U reaches one row and column of every result
    U = dev(case.U)
    U[5, 7] = float("nan")
    nan = torch.isnan(rot.rotate(U, dev(case.O), d, "fp32"))
    expect = torch.zeros_like(nan)
    expect[:, 7, :] = True
    expect[:, :, 7] = True
    assert torch.equal(nan, expect)


def test_pairs_chunks_and_column_scales(rot, oracle_mod):
    """A workspace for some of the operators gives the same bits, whatever it
    holds before; columns of U of very different size keep their accuracy."""
    m, d, mp, n = 200, 4, 150, 240
    case = workloads.dense_case(m, d, mp, n, cfg=750, symmetric=False)
    scale = 2.0 ** -np.round(np.linspace(0, 60, mp))
    U, O = dev(case.U * scale), dev(case.O)
    full = rot.rotate(U, O, d, "fp32")
    p = rot._problem(U, O, full, d)
    need = rot.rot_workspace_size([p], rot.ROT_FP32)  # two chunks
    parts, pairs = used_pairs(rot, lambda: rot.rotate(
        U, O, d, "fp32", workspace=torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")))
    assert pairs
    assert torch.equal(full, parts)
    got = full[:40].double().cpu().numpy() / (scale[:, None] * scale[None, :])
    assert rel_fro(got, oracle_mod.rotate(case.U, case.O[:40], d)).max() <= TOL32


def test_pairs_in_a_graph(rot):
    """Captured once and replayed with eager work in between: every replay
    equals the eager result."""
    m, d, mp, n = 260, 4, 200, 24
    case = workloads.dense_case(m, d, mp, n, cfg=760, symmetric=False)
    U, O = dev(case.U), dev(case.O)
    out = torch.empty((n, mp, mp), device="cuda")
    ws = torch.empty(rot.rot_workspace_preferred([rot._problem(U, O, out, d)], rot.ROT_FP32), dtype=torch.uint8,
                     device="cuda")
    want = rot.rotate(U, O, d, "fp32")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rot.rotate(U, O, d, "fp32", out=out, workspace=ws)
    for k in range(3):
        out.zero_()
        O.mul_(2.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want * 2.0 ** (k + 1))
