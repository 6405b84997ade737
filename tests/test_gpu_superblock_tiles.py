"""Superblock products over sectors of every extent around the tile and step
edges (1 to 16, 17, 32, 33 ... states), in 16 x 16 tiles and, at 1700 states,
in 32 x 32 tiles, against the oracle.

Tolerance: 1e-13 of the largest entry, FP64 sums of at most a few hundred
products."""
import numpy as np
import pytest
import torch

import workloads
from oracle import superblock as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("total", [12, 40, 90, 150, 300, 1700])
def test_tiles_and_steps(rot, total):
    case = workloads.superblock_random(total, cfg=20 + total)
    H = rot.SuperblockH(case.site_qn, case.left, case.right, case.target, case.left_ops, case.right_ops, case.terms)
    psi = np.random.default_rng(total).standard_normal(H.total)
    out = H.apply(torch.from_numpy(psi).cuda())
    torch.cuda.synchronize()
    L, R = workloads.superblock_dense_ops(case)
    terms = [(coef, L[lo] if lo >= 0 else None, sa, sat, R[ro] if ro >= 0 else None)
             for coef, lo, sa, sat, ro in case.terms]
    ref = sb.matvec(terms, workloads.superblock_to_dense(case, psi), case.m, 4, case.mR)
    got = workloads.superblock_to_dense(case, out.cpu().numpy())
    assert np.abs(got - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
