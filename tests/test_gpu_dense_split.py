"""The dense M2L cut into ranges of far offsets (small plans, and larger ones
whose last round of workgroups would be partly empty) and its skipping of
16-target groups without a source, against the oracle: trees of one and
several M2L levels, tiles of a few targets, surfaces whose tiles have empty
groups, the smallest and largest orders.  FP64 within 1e-12, mixed within
1e-6 of it, as for the unsplit M2L."""
import numpy as np
import pytest
import torch

import oracle
from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)


CASES = [
    ("cube", 60, 3, 1, 301),      # single particles, most sources absent
    ("cube", 900, 3, 4, 302),     # level 2 only: tiles of eight targets
    ("cube", 3001, 4, 5, 303),
    ("sphere", 5003, 5, 3, 304),  # empty 16-target groups
    ("sphere", 900, 7, 2, 305),   # a few targets per parity and level
    ("cube", 1201, 3, 12, 306),   # two M-blocks of three M-tiles a wavefront, and more
    ("cube", 20001, 5, 7, 307),   # nearly full tiles, two or more rounds
]


@pytest.mark.parametrize("kind,n,h,l,seed", CASES)
def test_dense_split_matches_oracle(kind, n, h, l, seed):
    print(f"dense split {kind} n={n} h={h} l={l}", flush=True)
    pos, q = inputs.make(kind, n, seed)
    p_o, f_o = oracle.Tree(pos, h).fmm(l, q)
    qd = torch.from_numpy(q).cuda()
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), h, l)
    assert plan.m2l_split() == 1  # the compressed M2L's split
    for sched in ("serial", "pipelined"):
        plan.set_schedule(sched)
        phi, f = plan.evaluate(qd)
        assert rel(phi, p_o) <= 1e-12 and rel(f, f_o) <= 1e-12, sched
    plan.set_precision("mixed")
    phi, f = plan.evaluate(qd)
    assert rel(phi, p_o) <= 1e-6 and rel(f, f_o) <= 1e-6
