"""The plan's cells (keys, leaves, every level, near and far lists) against the
oracle's tree, bit for bit, where the one-pass construction can go wrong: the
sizes at which a workgroup, a wavefront's rounds or the sort's tile change, one
particle, all particles in one cell, cells of one parity only, the deepest
tree."""
import numpy as np
import pytest
import torch

import oracle
from paper_1206_0115_amd import fmm, inputs
from test_gpu_parity import check_plan

pytestmark = pytest.mark.gpu

CASES = [
    ("cube", 1, 4), ("cube", 2, 3), ("cube", 64, 3), ("cube", 1023, 4), ("cube", 1024, 4),
    ("cube", 1025, 5), ("sphere", 4097, 6), ("cube", 262_144, 5), ("cube", 262_145, 6),
    ("cube", 300, 21), ("point", 3000, 6), ("line", 2050, 7), ("cube", 5000, 2), ("cube", 70, 1),
]


@pytest.mark.parametrize("kind,n,h", CASES)
def test_cells_bit_exact(kind, n, h):
    print(f"plan cells {kind} n={n} h={h}", flush=True)
    if kind == "point":  # two corners, everything else at one position
        pos = np.full((n, 3), 0.3)
        pos[0], pos[-1] = 0.0, 1.0
    elif kind == "line":
        pos = np.repeat(np.linspace(0.0, 1.0, n)[:, None], 3, axis=1)[::-1].copy()
    else:
        pos, _ = inputs.make(kind, n, 900 + n)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), h, 2)
    check_plan(plan, oracle.Tree(pos, h))
    plan.release()
