"""Operators that FP32 batches on FP16 pairs leave to the FP32 kernels, in every
form of a batch: symmetric output, chunks of a small workspace, K parts, and the
two FP32 kernels behind the pairs; what a batch of nothing else costs.

Skipped operators: where the FP32 entry point runs the same kernels, the same
bits; otherwise, as their neighbours, within the FP32 bound of 1e-5."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL32 = 1e-5
D = 4


def inputs(m, mp, n, seed, symmetric=False):
    rng = np.random.default_rng(seed)
    U = np.linalg.qr(rng.standard_normal((m * D, mp)))[0]
    O = rng.standard_normal((n, m, m))
    O = 0.5 * (O + O.transpose(0, 2, 1)) if symmetric else O
    return [torch.from_numpy(np.ascontiguousarray(a)).float().cuda() for a in (U, O)]


def grade(O, at):
    """Operators whose first half of states is 2^-20 of the other's size."""
    h = O.shape[1] // 2
    for b in at:
        O[b, :h] *= 2.0 ** -20
        O[b, :, :h] *= 2.0 ** -20


def fp32_kernels(rot, U, O, symmetric=False):
    out = torch.empty((len(O), U.shape[1], U.shape[1]), device="cuda")
    p = rot._problem(U, O, out, D)
    ws = torch.empty(rot.rot_workspace_size([p], rot.ROT_FP32), dtype=torch.uint8, device="cuda")
    rot.rot_batch_fp32([p], ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream,
                       rot.ROT_ASSUME_SYMMETRIC_O if symmetric else 0)
    return out


def check(oracle_mod, U, O, got, some):
    ref = oracle_mod.rotate(U.double().cpu().numpy(), O[some].double().cpu().numpy(), D)
    err = np.sqrt(((got[some].double().cpu().numpy() - ref) ** 2).sum((1, 2)) / (ref ** 2).sum((1, 2)))
    assert err.max() <= TOL32


# 64-wide tiles; 128-wide ones (1024 and more in both stages), whole and partial
@pytest.mark.parametrize("m,mp,n", [(131, 118, 90), (128, 128, 1030), (144, 132, 400)])
@pytest.mark.parametrize("symmetric", [False, True])
def test_skipped_beside_others(rot, oracle_mod, m, mp, n, symmetric):
    U, O = inputs(m, mp, n, 7500 + m, symmetric)
    bad = [0, 5, n // 2, n - 1]
    grade(O, bad)
    O[7, 3, 3] = float("nan")
    got = rot.rotate(U, O, D, "fp32", symmetric_O=symmetric)
    fp32 = fp32_kernels(rot, U, O, symmetric)
    for b in bad:
        assert torch.equal(got[b], fp32[b])
    assert torch.isnan(got[7]).all()
    check(oracle_mod, U, O, got, bad + [1, 6, 8, n - 2])
    if symmetric:
        rest = [b for b in range(n) if b != 7]
        assert torch.equal(got[rest], got[rest].transpose(1, 2))


def test_skipped_in_later_chunks(rot, oracle_mod):
    """U's pairs and judgement come from the first chunk."""
    m, mp, n = 200, 150, 240
    U, O = inputs(m, mp, n, 7600)
    bad = [1, n // 2 + 3, n - 1]
    grade(O, bad)
    full = rot.rotate(U, O, D, "fp32")
    p = rot._problem(U, O, full, D)
    ws = torch.full((rot.rot_workspace_size([p], rot.ROT_FP32),), 0xFF, dtype=torch.uint8, device="cuda")
    rot.profile_enable(True)
    parts = rot.rotate(U, O, D, "fp32", workspace=ws)
    torch.cuda.synchronize()
    assert rot.profile_read()["stage1_f16x3"][0] > 1
    rot.profile_enable(False)
    assert torch.equal(full, parts)
    check(oracle_mod, U, O, parts, bad + [0, n // 2 + 2, n - 2])
    U[: 2 * m] *= 2.0 ** -20  # all of them
    parts = rot.rotate(U, O, D, "fp32", workspace=ws)
    assert torch.equal(parts, fp32_kernels(rot, U, O))


def test_skipped_with_k_parts(rot, oracle_mod):
    """Partial sums of a skipped operator are not its result; it has the FP32
    path's K parts, and so its bits."""
    m, mp, n = 404, 391, 4
    U, O = inputs(m, mp, n, 7700)
    grade(O, [1])
    rot.profile_enable(True)
    got = rot.rotate(U, O, D, "fp32")
    torch.cuda.synchronize()
    kinds = rot.profile_read()
    rot.profile_enable(False)
    assert "stage1_f16x3" in kinds and "stage2_sum" in kinds
    assert torch.equal(got[1], fp32_kernels(rot, U, O)[1])
    check(oracle_mod, U, O, got, list(range(n)))


def test_skipped_in_a_graph(rot):
    """A captured batch judges its operators and U at each replay."""
    U, O = inputs(200, 150, 90, 7750)
    out = torch.empty((90, 150, 150), device="cuda")
    ws = torch.empty(rot.rot_workspace_preferred([rot._problem(U, O, out, D)], rot.ROT_FP32), dtype=torch.uint8,
                     device="cuda")
    rot.rotate(U, O, D, "fp32", out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rot.rotate(U, O, D, "fp32", out=out, workspace=ws)
    U0, O0 = U.clone(), O.clone()
    for step in range(4):
        U.copy_(U0)
        O.copy_(O0)
        if step == 1:
            grade(O, [3, 88])
        if step == 2:
            U[:400] *= 2.0 ** -20
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, rot.rotate(U, O, D, "fp32"))
        fp32 = fp32_kernels(rot, U, O)
        same = [b for b in range(90) if torch.equal(out[b], fp32[b])]
        assert same == ([], [3, 88], list(range(90)), [])[step]


@pytest.mark.parametrize("which", ["U", "O"])
def test_skipped_batch_runs_no_products_on_pairs(rot, which):
    """The pairs' stages of a batch that is skipped whole take less than half of
    their time for one that is not (they look at flags)."""
    U, O = inputs(512, 512, 64, 7800)

    def times():
        best = {}
        for _ in range(4):
            rot.profile_enable(True)
            rot.rotate(U, O, D, "fp32")
            torch.cuda.synchronize()
            for k, (_, ms) in rot.profile_read().items():
                best[k] = min(best.get(k, 1e9), ms)
        rot.profile_enable(False)
        return best["stage1_f16x3"], best["stage2_f16x3"]

    run = times()
    if which == "U":
        U[:1024] *= 2.0 ** -20
    else:
        grade(O, range(64))
    skipped = times()
    assert skipped[0] < 0.5 * run[0] and skipped[1] < 0.5 * run[1]
