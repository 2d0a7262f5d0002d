"""The compressed M2L at order 9 in FP32: at ranks up to 48 plans of full tiles
take two K-groups a producer, surfaces and higher ranks four.  The mixed sums
are the same whatever the split, so a tolerance on either side of the rule
agrees with the dense FP64 path within ten times itself plus the 1e-6 gate."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


@pytest.mark.parametrize("kind,n,h", [("cube", 60_001, 5), ("sphere", 60_001, 6)])
def test_ranks_on_both_sides(kind, n, h):
    print(f"svd order 9 {kind} n={n} h={h}", flush=True)
    pos, q = inputs.make(kind, n, 1800)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, 9, "fp64")
    ref = plan.evaluate(q)
    plan.set_precision("mixed_svd")
    for eps, rank in ((1e-5, 32), (1e-7, 48), (1e-8, 64)):
        plan.set_m2l_tolerance(eps)
        assert plan.svd_info().rmax_pad == rank
        out = plan.evaluate(q)
        assert max(rel(o, r) for o, r in zip(out, ref)) <= 10 * eps + 1e-6, eps
