"""FP32 batches, site products and plans on FP16 pairs whose operators or U hold
entries of very different size: whole results and blocks of them against 64
bits and the FP32 kernels.

Tolerance, per block: the FP32 kernels' own relative Frobenius error on it plus
2^-21 (the four conversions into pairs, each within 2^-23 of an entry), and
never above the FP32 bound of 1e-5."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL32 = 1e-5
M, D, MP = 160, 4, 130
N = int(4e9 / (2 * M * D * MP * (M + MP))) + 1  # the least batch on pairs
HALF, KEPT = M // 2, MP // 2


def isometry(rows, cols, rng):
    return np.linalg.qr(rng.standard_normal((rows, cols)))[0]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).float().cuda()


def host(t):
    return t.double().cpu().numpy()


ALL = np.arange(MP)


def left_out(size, rng):
    """Large columns (rows) of operators on a state that U leaves out."""
    U = np.zeros((M, D, MP))
    U[1:] = isometry((M - 1) * D, MP, rng).reshape(M - 1, D, MP)
    O = rng.standard_normal((2, M, M)) * size
    O[0, :, 0] = rng.standard_normal(M)
    O[1, 0, :] = rng.standard_normal(M)
    return U, O, [(ALL, ALL)]


def one_reaches(size, rng):
    """The same with one kept state on the large column."""
    U, O, _ = left_out(size, rng)
    U[:, :, 7] = 0
    U[0, 1, 7] = 1
    rest = np.delete(ALL, 7)
    return U, O, [(ALL, ALL), (rest, rest), ([7], rest), (rest, [7])]


def hardly_kept(size, rng):
    """Operators on states that U hardly reaches: zero columns, one block."""
    U = isometry(M * D, MP, rng).reshape(M, D, MP)
    U[:HALF] *= size
    O = rng.standard_normal((2, M, M))
    O[:, :, HALF:] = 0
    O[1, HALF:] = 0
    return U, O, [(ALL, ALL)]


def sectors(size, rng):
    """Two sectors, operators' blocks of different size; in order and mixed."""
    U = np.zeros((M, D, MP))
    U[:HALF, :, :KEPT] = isometry(HALF * D, KEPT, rng).reshape(HALF, D, KEPT)
    U[HALF:, :, KEPT:] = isometry((M - HALF) * D, MP - KEPT, rng).reshape(M - HALF, D, MP - KEPT)
    O = rng.standard_normal((2, M, M))
    O[0, :HALF, HALF:] *= size
    O[1, HALF:] *= size
    O[1, :, HALF:] *= size
    return U, O, [(a, b) for a in (ALL[:KEPT], ALL[KEPT:]) for b in (ALL[:KEPT], ALL[KEPT:])]


def mixed_sectors(size, rng):
    U, O, blocks = sectors(size, rng)
    old, kept = rng.permutation(M), rng.permutation(MP)
    at = np.argsort(kept)
    return U[old][:, :, kept], O[:, old][:, :, old], [(at[a], at[b]) for a, b in blocks]


def tails(size, rng):
    """Small tails of kept states in the other sector, operators in one sector."""
    U, O, blocks = sectors(1.0, rng)
    U[:HALF, :, KEPT:] = size * rng.standard_normal((HALF, D, MP - KEPT)) / np.sqrt(M)
    O[:, HALF:] = 0
    O[1] = O[1].T
    return U, O, blocks


KINDS = [left_out, one_reaches, hardly_kept, sectors, mixed_sectors, tails]


def inputs(kind, size, seed):
    """U (M*D, MP) and a batch whose operators 1 and N - 2 are the kind's, the
    others Gaussian; blocks of the result."""
    rng = np.random.default_rng(seed)
    U, two, blocks = kind(size, rng)
    O = rng.standard_normal((N, M, M))
    O[[1, N - 2]] = two
    U, O = dev(U.reshape(M * D, MP)), dev(O)
    return U, O, blocks


def fp32_kernels(rot, U, O):
    out = torch.empty((len(O), MP, MP), device="cuda")
    p = rot._problem(U, O, out, D)
    ws = torch.empty(rot.rot_workspace_size([p], rot.ROT_FP32), dtype=torch.uint8, device="cuda")
    rot.rot_batch_fp32([p], ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    return out


def check(got, fp32, ref, blocks):
    for b in range(len(ref)):
        for rows, cols in blocks:
            at = np.ix_(rows, cols)
            size = np.linalg.norm(ref[b][at])
            if size == 0:
                assert np.all(got[b][at] == 0)
                continue
            ours, theirs = np.linalg.norm(got[b][at] - ref[b][at]) / size, np.linalg.norm(fp32[b][at] - ref[b][at]) / size
            assert ours <= min(TOL32, theirs + 2.0 ** -21), (b, ours, theirs)


SIZES = [1e-2, 2.0 ** -14, 2.0 ** -20, 2.0 ** -40]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("kind", KINDS)
def test_batch_of_uneven_entries(rot, oracle_mod, kind, size):
    U, O, blocks = inputs(kind, size, 7100)
    got = rot.rotate(U, O, D, "fp32")
    fp32 = fp32_kernels(rot, U, O)
    some = [0, 1, 2, N - 2, N - 1]
    check(host(got[some]), host(fp32[some]), oracle_mod.rotate(host(U), host(O[some]), D), blocks)


def test_even_operators_stay_on_pairs(rot):
    """Beside operators out of range, and over zeros and entries of one size."""
    U, O, _ = inputs(left_out, 2.0 ** -20, 7200)
    O[3] = torch.eye(M, device="cuda")
    O[4] = torch.sign(O[4])
    O[5, :HALF, HALF:] = 0
    got, fp32 = rot.rotate(U, O, D, "fp32"), fp32_kernels(rot, U, O)
    same = [torch.equal(got[b], fp32[b]) for b in range(N)]
    assert [b for b in range(N) if same[b]] == [1, N - 2]


def test_operators_whose_row_sums_overflow(rot, oracle_mod):
    """T's scale comes from row sums of |O|; near FP32's largest value it comes
    from the largest entry."""
    U, O, blocks = inputs(left_out, 1.0, 7240)
    O[3] *= 2.0 ** 124
    O[4] *= 2.0 ** -100
    got, fp32 = rot.rotate(U, O, D, "fp32"), fp32_kernels(rot, U, O)
    assert not torch.equal(got[3], fp32[3]) and not torch.equal(got[4], fp32[4])
    check(host(got[2:5]), host(fp32[2:5]), oracle_mod.rotate(host(U), host(O[2:5]), D), blocks)


def test_single_rows_and_columns_are_found(rot):
    """One small row of an operator that acts on states U hardly reaches (a column
    of T), or one kept state that only an operator's small column reaches (a row
    of T), wherever it lies in a tile: computed by the FP32 kernels, to the bit;
    their neighbours are not."""
    rng = np.random.default_rng(7250)
    kept = [0, 7, 8, 31, 32, 63, 64, 101, MP - 1]
    rows = [0, 15, 16, 31, 32, 95, M - 1]
    U = isometry(M * D, MP, rng).reshape(M, D, MP)
    U[100:120] *= 2.0 ** -8
    O = rng.standard_normal((N, M, M))
    for k, beta in enumerate(kept):
        U[:, :, beta] = 0
        U[10 + k, k % D, beta] = 1
        O[2 * k, :, 10 + k] *= 2.0 ** -11
    for k, i in enumerate(rows):
        O[20 + 2 * k, i, :100] = 0
        O[20 + 2 * k, i, 120:] = 0
        O[20 + 2 * k, i] *= 2.0 ** -6
    U, O = dev(U.reshape(M * D, MP)), dev(O)
    got, fp32 = rot.rotate(U, O, D, "fp32"), fp32_kernels(rot, U, O)
    same = [b for b in range(N) if torch.equal(got[b], fp32[b])]
    assert same == [2 * k for k in range(len(kept))] + [20 + 2 * k for k in range(len(rows))]


def picked(per_column, rng):
    """U with a few entries per column, anywhere (one: states picked out)."""
    U = np.zeros((M * D, MP))
    for beta in range(MP):
        rows = rng.permutation(M * D)[:per_column]
        U[rows, beta] = 1 if per_column == 1 else rng.standard_normal(per_column) / np.sqrt(per_column)
    return U.reshape(M, D, MP), rng.standard_normal((2, M, M)), [(ALL, ALL)]


@pytest.mark.parametrize("per_column", [1, 5, 40, 160])
def test_sparse_U(rot, oracle_mod, per_column):
    """Short sums are exact, or nearly, on the FP32 instructions: batches, site
    products and plans with such a U stay there."""
    U, O, _ = inputs(lambda size, rng: picked(per_column, rng), 0, 7260)
    got, fp32 = rot.rotate(U, O, D, "fp32"), fp32_kernels(rot, U, O)
    assert torch.equal(got, fp32)
    if per_column == 1:
        assert np.array_equal(host(got[:3]), oracle_mod.rotate(host(U), host(O[:3]), D))
    S = np.eye(D)
    assert torch.equal(rot.rotate_site(U, O, S, "fp32")[:3], rot.rotate_site(U, O[:3].contiguous(), S, "fp32"))
    out = torch.empty_like(got)
    plan = rot.Plan([(U, O, out, D)])
    assert sum(c["pairs"] for c in plan.describe()["classes"]) == N
    plan.execute()
    torch.cuda.synchronize()
    check(host(out[:3]), host(fp32[:3]), oracle_mod.rotate(host(U), host(O[:3]), D), [(ALL, ALL)])
    if per_column == 1:
        assert torch.equal(out, got)
    plan.close()


def test_sectors_in_order_stay_on_pairs(rot):
    """Four sectors, operators between neighbours: runs of entries and zeros."""
    rng = np.random.default_rng(7270)
    U, O, n, k = np.zeros((M, D, MP)), np.zeros((N, M, M)), M // 4, MP // 4
    for q in range(4):
        U[q * n:(q + 1) * n, :, q * k:(q + 1) * k] = isometry(n * D, k, rng).reshape(n, D, k)
        r = (q + 1) % 4
        O[:, q * n:(q + 1) * n, r * n:(r + 1) * n] = rng.standard_normal((N, n, n))
    U, O = dev(U.reshape(M * D, MP)), dev(O)
    got, fp32 = rot.rotate(U, O, D, "fp32"), fp32_kernels(rot, U, O)
    assert not any(torch.equal(got[b], fp32[b]) for b in range(N))


@pytest.mark.parametrize("kind", [left_out, hardly_kept, sectors])
def test_plan_of_uneven_entries(rot, oracle_mod, kind):
    """Two groups, one of even operators: each is judged by itself, at every
    execution."""
    U, O, blocks = inputs(kind, 2.0 ** -20, 7300)
    rng = np.random.default_rng(7301)
    U1, O1 = dev(isometry(M * D, MP, rng)), dev(rng.standard_normal((9, M, M)))
    outs = [torch.empty((len(x), MP, MP), device="cuda") for x in (O1, O)]
    plan = rot.Plan([(U1, O1, outs[0], D), (U, O, outs[1], D)])
    some = [0, 1, N - 2, N - 1]
    for _ in range(2):
        for x in outs:
            x.fill_(float("nan"))
        plan.execute()
        torch.cuda.synchronize()
        check(host(outs[1][some]), host(fp32_kernels(rot, U, O)[some]),
              oracle_mod.rotate(host(U), host(O[some]), D), blocks)
        check(host(outs[0]), host(fp32_kernels(rot, U1, O1)), oracle_mod.rotate(host(U1), host(O1), D), [(ALL, ALL)])
    plan.close()


@pytest.mark.parametrize("size", [1e-2, 2.0 ** -20])
@pytest.mark.parametrize("kind", KINDS)
def test_site_products_of_uneven_entries(rot, oracle_mod, kind, size):
    U, X, blocks = inputs(kind, size, 7400)
    S = np.zeros((D, D))
    S[:, [1, 3]] = np.random.default_rng(7401).standard_normal((D, 2))
    got = rot.rotate_site(U, X, S, "fp32")
    few = [0, 1, 2, N - 2, N - 1]
    fp32 = rot.rotate_site(U, X[few].contiguous(), S, "fp32")  # too few for the pairs
    check(host(got[few]), host(fp32), oracle_mod.rotate_site(host(U), host(X[few]), S), blocks)
