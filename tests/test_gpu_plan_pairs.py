"""Plans on FP16 pairs: chunks of groups of different sizes, the FP32 kernels
behind them, small workspaces and rebinding, against the oracle.

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


def build(shapes, cfg, offset=0):
    """(cases, groups) of shapes (m, d, mp, n); buffers `offset` floats past an aligned address."""
    cases = [workloads.dense_case(m, d, mp, n, cfg=cfg + i, symmetric=False) for i, (m, d, mp, n) in enumerate(shapes)]

    def dev(a):
        buf = torch.empty(a.size + offset, device="cuda")
        t = buf[offset:].view(a.shape)
        t.copy_(torch.from_numpy(np.ascontiguousarray(a)).float())
        return t

    groups = [(dev(c.U), dev(c.O), dev(np.full((c.O.shape[0], c.U.shape[1], c.U.shape[1]), np.nan)), s[1])
              for c, s in zip(cases, shapes)]
    return cases, groups


def check(oracle_mod, cases, groups):
    for c, (_, _, out, d) in zip(cases, groups):
        assert rel_fro(out.double().cpu().numpy(), oracle_mod.rotate(c.U, c.O, d)).max() <= TOL32


# tile heights 64 to 256 with remainders, one operator, shapes below 64 (FP32
# kernels), and d other than 4 beside it
MIXES = [
    [(64, 4, 64, 5), (65, 4, 97, 3), (300, 4, 257, 7), (404, 4, 391, 2), (129, 4, 191, 1), (40, 4, 30, 4)],
    [(100, 8, 333, 2), (257, 4, 193, 18), (145, 2, 250, 6), (200, 1, 128, 3), (96, 3, 191, 30), (64, 9, 70, 2)],
]


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_plan_on_pairs(rot, oracle_mod, mix, graph):
    cases, groups = build(MIXES[mix], cfg=800 + 20 * mix, offset=1 if graph else 0)
    plan = rot.Plan(groups, graph=graph)
    classes = plan.describe()["classes"]
    on_pairs = sum(n for m, d, mp, n in MIXES[mix] if min(m, mp) >= 64 and d <= 8)
    assert sum(c["pairs"] for c in classes) == on_pairs
    assert sum(c["ops"] for c in classes) == sum(s[3] for s in MIXES[mix])
    for _ in range(3):
        for g in groups:
            g[2].fill_(float("nan"))
        plan.execute()
        torch.cuda.synchronize()
        check(oracle_mod, cases, groups)
    plan.close()


def test_plan_on_pairs_in_chunks(rot, oracle_mod):
    """Workspaces for some of the operators, down to rot_workspace_size's
    least (the FP32 kernels), filled with NaN before."""
    shapes = [(500, 4, 480, 6), (260, 4, 300, 12), (130, 4, 120, 5)]
    cases, groups = build(shapes, cfg=850)
    probs = [rot._problem(*g) for g in groups]
    most = rot.rot_plan_workspace_preferred(probs, rot.ROT_FP32)
    seen = []
    for nbytes in (most, most // 2, most // 3, rot.rot_workspace_size(probs, rot.ROT_FP32, 1)):
        plan = rot.Plan(groups, workspace_bytes=nbytes, tune=False)
        plan.workspace.fill_(0xFF)
        for g in groups:
            g[2].fill_(float("nan"))
        plan.execute()
        torch.cuda.synchronize()
        check(oracle_mod, cases, groups)
        seen.append(sum(c["pairs"] for c in plan.describe()["classes"]))
        plan.close()
    assert seen[0] == 23 and 0 < seen[1] and seen[3] == 0


@pytest.mark.parametrize("graph", [True, False])
def test_plan_on_pairs_skips_and_rebind(rot, oracle_mod, graph):
    """Operators that the pairs cannot hold go to the FP32 kernels at each
    execution, whatever the one before held; new buffers at any alignment."""
    shapes = [(300, 4, 280, 9), (150, 4, 130, 12)]
    cases, groups = build(shapes, cfg=860)
    plan = rot.Plan(groups, graph=graph)
    assert sum(c["pairs"] for c in plan.describe()["classes"]) == 21
    plan.execute()
    torch.cuda.synchronize()
    check(oracle_mod, cases, groups)
    other, fresh = build(shapes, cfg=870, offset=3)
    other[0].O[2] *= np.logspace(0, -8, 300)[:, None]
    other[1].O[11, 5, :] *= 2.0 ** 30
    for c, g in zip(other, fresh):
        g[1].copy_(torch.from_numpy(c.O).float())
        c.O[:] = g[1].double().cpu().numpy()
    fresh[1][1][4, 7, :] = float("nan")
    plan.rebind(fresh)
    plan.execute()
    plan.rebind(groups)  # in stream order behind the execution
    torch.cuda.synchronize()
    assert torch.isnan(fresh[1][2][4]).all()
    fresh[1][2][4] = 0
    other[1].O[4] = 0
    for c, (_, _, out, d) in zip(other, fresh):
        ref = oracle_mod.rotate(c.U, c.O, d)
        keep = [b for b in range(len(ref)) if np.abs(ref[b]).max() > 0]
        assert rel_fro(out.double().cpu().numpy()[keep], ref[keep]).max() <= TOL32
    for g in groups:
        g[2].fill_(float("nan"))
    plan.execute()
    torch.cuda.synchronize()
    check(oracle_mod, cases, groups)
    plan.close()
