"""Blocked rotations whose tables were seen before: still refused when they,
or the workspace, have become wrong, and unaffected by a refusal."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def test_known_tables_are_checked_by_content(rot):
    case = workloads.blocked_case(total=96, n_conserving=2, n_up_shift=1, n_dn_shift=1, cfg=97)
    pk = workloads.pack_blocked(case)
    U = torch.from_numpy(pk.U_blk).float().cuda()
    O = torch.from_numpy(pk.O_blk).float().cuda()
    out = torch.full((pk.out_size,), float("nan"), device="cuda")
    p, keep = rot.blocked_problem(pk.site_qn, pk.old, pk.new, pk.shift, U, pk.U_off, O, pk.O_off, pk.out_off, out)
    ws = torch.empty(rot.rot_blocked_workspace_size(p), dtype=torch.uint8, device="cuda")

    def call(ptr=ws.data_ptr(), size=ws.numel()):
        rot.rot_batch_blocked(p, rot.ROT_FP32, ptr, size, torch.cuda.current_stream().cuda_stream)

    call()
    torch.cuda.synchronize()
    want = out.clone()
    for bad in (lambda: call(size=ws.numel() - 256), lambda: call(ptr=0), lambda: call(ptr=ws.data_ptr() + 16)):
        with pytest.raises(rot.RotError):
            bad()
    # the same arrays with one entry made invalid, then restored
    for name, at, value in (("O_off", 0, -2), ("U_off", 1, -1), ("shift", 0, 50)):
        was = keep[name][at]
        keep[name][at] = value
        with pytest.raises(rot.RotError):
            call()
        keep[name][at] = was
    dim = p.old_sec[0].dim
    p.old_sec[0].dim = 0
    with pytest.raises(rot.RotError):
        call()
    p.old_sec[0].dim = dim
    p.site_qn = type(p.site_qn)()
    with pytest.raises(rot.RotError):
        call()
    p.site_qn = keep["site_qn"].ctypes.data_as(type(p.site_qn))
    out.fill_(float("nan"))
    call()
    torch.cuda.synchronize()
    assert torch.equal(out.nan_to_num(), want.nan_to_num())
