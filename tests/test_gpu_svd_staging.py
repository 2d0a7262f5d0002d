"""The compressed M2L of a shape whose two workgroups a CU leave no room for the
source rows in LDS (FP64 order 5 at ranks of 64): the rows come from memory, at
both item widths and with empty groups skipped; against the dense FP64 path
within ten times the tolerance."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


@pytest.mark.parametrize("kind,n,h", [("cube", 1001, 3), ("cube", 30_001, 5), ("sphere", 9001, 6)])
def test_rows_from_memory(kind, n, h):
    print(f"svd staging {kind} n={n} h={h}", flush=True)
    pos, q = inputs.make(kind, n, 1700)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, 5, "fp64", m2l_tolerance=1e-8)
    ref = plan.evaluate(q)
    plan.set_precision("fp64_svd")
    assert plan.svd_info().rmax_pad == 64
    out = plan.evaluate(q)
    assert max(rel(o, r) for o, r in zip(out, ref)) <= 1e-7
