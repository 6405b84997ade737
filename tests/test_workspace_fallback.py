"""Calls that allocate their own workspace run in the smaller one that the
library takes where memory does not hold the preferred one."""
import numpy as np
import pytest
import torch

import paper_0909_5662_amd as rot_mod


def test_smaller_workspace_when_memory_is_short(monkeypatch):
    real, asked = torch.empty, []

    def short(n, **kw):
        asked.append(n)
        if n > 1000:
            raise torch.OutOfMemoryError("no memory")
        return real((n + 255) // 256 * 256, **kw)

    monkeypatch.setattr(rot_mod, "_workspace", lambda n, device: short(n, dtype=torch.uint8, device=device))
    assert rot_mod._workspace_or_less(2000, "cpu", int, 500).numel() >= 500
    assert asked == [2000, 500]
    assert rot_mod._workspace_or_less(900, "cpu", int, 500).numel() >= 900
    with pytest.raises(torch.OutOfMemoryError):
        rot_mod._workspace_or_less(5000, "cpu", int, 2000)
    asked.clear()
    with pytest.raises(torch.OutOfMemoryError):
        rot_mod._workspace_or_less(2000, "cpu", int, 2000)
    assert asked == [2000]


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["rotate", "site", "plan"])
def test_calls_in_little_memory(rot, call):
    """A memory limit between the two sizes: the same results (to rounding)."""
    m, d, mp, n = 512, 4, 512, 200
    g = torch.Generator(device="cuda")
    g.manual_seed(7900)
    U = torch.randn((m * d, mp), generator=g, device="cuda") / 45
    O = torch.randn((n, m, m), generator=g, device="cuda")
    out = torch.empty((n, mp, mp), device="cuda")
    S = np.eye(d) + np.roll(np.eye(d), 1, axis=1)  # lists all site states
    p = rot._problem(U, O, out, d)

    def run():
        if call == "rotate":
            return rot.rotate(U, O, d, "fp32", out=out)
        if call == "site":
            return rot.rotate_site(U, O, S, "fp32")
        plan = rot.Plan([(U, O, out, d)], tune=False)
        plan.execute()
        torch.cuda.synchronize()
        plan.close()
        return out

    want = run().clone()
    if call == "site":
        import ctypes
        q = rot.RotSiteProblem(m, d, mp, n, rot.ROT_BLOCK_DENSE, U.data_ptr(),
                               S.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), O.data_ptr(), m * m, out.data_ptr(),
                               mp * mp)
        most, least = rot.rot_site_workspace_preferred([q], rot.ROT_FP32), rot.rot_site_workspace_size([q], rot.ROT_FP32)
        extra = out.numel() * 4
    else:
        size = rot.rot_plan_workspace_preferred if call == "plan" else rot.rot_workspace_preferred
        most, least, extra = size([p], rot.ROT_FP32), rot.rot_workspace_size([p], rot.ROT_FP32), 0
    assert most - least > 64 << 20
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    limit = torch.cuda.memory_reserved() + extra + (most + least) // 2
    try:
        torch.cuda.set_per_process_memory_fraction(limit / total)
        got = run()
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert ((got - want).norm() / want.norm()).item() <= 1e-6
