"""Block operators times a site operator on FP16 pairs, over the site states
that the site operator's non-zero columns name: parity with the oracle, chunks,
and the operators that those kernels leave to the FP32 ones.

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


def site_operator(d, columns, rng):
    S = np.zeros((d, d))
    S[:, columns] = rng.standard_normal((d, len(columns)))
    return S


def inputs(m, d, mp, n, cfg):
    case = workloads.dense_case(m, d, mp, n, cfg=cfg, symmetric=False)
    U, X = dev(case.U), dev(case.O)
    return U, X, U.double().cpu().numpy(), X.double().cpu().numpy()


def kinds_of(rot, call):
    rot.profile_enable(True)
    out = call()
    torch.cuda.synchronize()
    kinds = rot.profile_read()
    rot.profile_enable(False)
    return out, kinds


# one to eight listed states of up to ten, remainders of tiles, blocks and slabs
CASES = [(64, 4, 64, [1, 3]), (131, 4, 118, [0]), (131, 2, 119, [0, 1]), (300, 4, 257, [0, 1, 2, 3]), (145, 3, 250, [2]), (97, 10, 333, [9, 0, 4]),
         (100, 8, 191, list(range(8)))]


@pytest.mark.parametrize("m,d,mp,columns", CASES)
def test_site_pairs_parity(rot, oracle_mod, m, d, mp, columns):
    n = int(4e9 / (2 * m * d * mp * (m + mp))) + 1
    U, X, U64, X64 = inputs(m, d, mp, n, 900 + m)
    S = site_operator(d, columns, np.random.default_rng(900 + m))
    got, kinds = kinds_of(rot, lambda: rot.rotate_site(U, X, S, "fp32"))
    assert "stage1_f16x3" in kinds
    some = list(range(0, n, max(1, n // 6)))
    assert rel_fro(got[some].double().cpu().numpy(), oracle_mod.rotate_site(U64, X64[some], S)).max() <= TOL32


def test_site_pairs_chunks_and_graph(rot, oracle_mod):
    """A workspace for half of the operators, whatever it holds before, and a
    captured call replayed with eager work in between."""
    m, d, mp, n = 260, 4, 300, 60
    U, X, U64, X64 = inputs(m, d, mp, n, 930)
    S = site_operator(d, [1, 3], np.random.default_rng(930))
    want = rot.rotate_site(U, X, S, "fp32")
    least = rot.rot_site_workspace_size([_site(rot, U, X, S, want)], rot.ROT_FP32)
    ws = torch.full((least // 2,), 0xFF, dtype=torch.uint8, device="cuda")
    half, kinds = kinds_of(rot, lambda: rot.rotate_site(U, X, S, "fp32", workspace=ws))
    assert kinds["stage1_f16x3"][0] > 1
    for out in (want, half):
        assert rel_fro(out[:6].double().cpu().numpy(), oracle_mod.rotate_site(U64, X64[:6], S)).max() <= TOL32
        assert ((out - want).norm() / want.norm()).item() <= 1e-6
    graph = torch.cuda.CUDAGraph()
    big = torch.empty(2 * least, dtype=torch.uint8, device="cuda")
    with torch.cuda.graph(graph):
        out = rot.rotate_site(U, X, S, "fp32", workspace=big)
    for _ in range(3):
        out.fill_(float("nan"))
        assert torch.isfinite(torch.randn(1 << 20, device="cuda").sum())
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def _site(rot, U, X, S, out):
    import ctypes
    n, m, _ = X.shape
    S = np.ascontiguousarray(S, dtype=np.float64)
    return rot.RotSiteProblem(m, len(S), U.shape[1], n, rot.ROT_BLOCK_DENSE, U.data_ptr(),
                              S.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), X.data_ptr(), m * m, out.data_ptr(),
                              U.shape[1] ** 2)


def test_site_pairs_leave_out_of_range_operators(rot, oracle_mod):
    """NaN in an operator, rows of very different size, NaN in U rows of a
    site state that S does not list: as the FP32 kernels give them."""
    m, d, mp = 150, 4, 130
    n = int(4e9 / (2 * m * d * mp * (m + mp))) + 1
    U, X, U64, X64 = inputs(m, d, mp, n, 940)
    S = site_operator(d, [1, 3], np.random.default_rng(940))
    X64[3] *= np.logspace(0, -8, m)[:, None]
    X = dev(X64)
    X64 = X.double().cpu().numpy()
    X[5, 7, :] = float("nan")
    got, kinds = kinds_of(rot, lambda: rot.rotate_site(U, X, S, "fp32"))
    assert "stage1_f16x3" in kinds
    assert torch.isnan(got[5]).all()
    keep = [0, 3, 4, 6]
    assert rel_fro(got[keep].double().cpu().numpy(), oracle_mod.rotate_site(U64, X64[keep], S)).max() <= TOL32
    U[4 * 11 + 2, 7] = float("nan")  # site state 2
    few = rot.rotate_site(U, X[:2].contiguous(), S, "fp32")  # FP32 kernels
    many = rot.rotate_site(U, X, S, "fp32")
    assert torch.equal(torch.isnan(many[:2]), torch.isnan(few)) and torch.isnan(few).any()
