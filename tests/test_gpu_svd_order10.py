"""The compressed M2L at order 10 in FP64, whose producers take three rank tiles
a pass at ranks up to 48 and five above, and whose consumers, on surfaces, pass over offsets without a source:
ranks of one tile up to the largest, i.e. every rest of a pass, against the
dense FP64 path within ten times the tolerance."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


@pytest.mark.parametrize("kind,n,h,eps", [
    ("cube", 1501, 3, 1e-1),    # one or two tiles
    ("cube", 1501, 3, 1e-4),
    ("cube", 1501, 3, 1e-7),    # three tiles
    ("cube", 1501, 3, 1e-8),    # four
    ("cube", 20_011, 5, 1e-10),  # the most, several passes
    ("sphere", 9001, 6, 1e-4),
    ("sphere", 9001, 6, 1e-10),
])
def test_order_10(kind, n, h, eps):
    print(f"svd order 10 {kind} n={n} h={h} eps={eps}", flush=True)
    pos, q = inputs.make(kind, n, 1600)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, 10, "fp64", m2l_tolerance=eps)
    ref = plan.evaluate(q)
    plan.set_precision("fp64_svd")
    assert plan.info().m2l_group_skip == (kind == "sphere")
    out = plan.evaluate(q)
    assert max(rel(o, r) for o, r in zip(out, ref)) <= 10 * eps
