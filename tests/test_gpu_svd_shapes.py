"""The compressed M2L kernel's item shapes (16, 32 or 64 target columns, one
or two M-blocks, the slab splits for ranks of tight tolerances, empty target
groups skipped) against the dense FP64 path: the compressed FP64 mode within
ten times its tolerance, the mixed one within that plus the 1e-6 gate."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


CASES = [
    ("cube", 700, 3, 1, 1e-1),     # one K-chunk, one M-tile
    ("cube", 30001, 5, 3, 1e-3),   # two M-tiles
    ("sphere", 9001, 6, 4, 1e-6),  # four M-tiles, empty groups
    ("cube", 5003, 4, 6, 1e-9),    # fourteen M-tiles
    ("cube", 60_001, 5, 6, 1e-10),  # two partial slabs for two workgroups a CU
    ("cube", 1001, 3, 7, 1e-7),    # few tiles: 16 columns
    ("cube", 40001, 5, 7, 1e-7),   # 32 columns
    ("cube", 99991, 6, 7, 1e-7),   # whole tiles
    ("cube", 99991, 6, 7, 1e-11),  # whole tiles, four partial slabs do not fit
    ("sphere", 9001, 6, 8, 1e-8),
    ("cube", 20011, 5, 9, 1e-9),
    ("cube", 20011, 5, 10, 1e-7),
    ("cube", 3001, 3, 12, 1e-10),  # two M-blocks
]


@pytest.mark.parametrize("kind,n,h,l,eps", CASES)
def test_shapes_match_dense(kind, n, h, l, eps):
    print(f"svd shapes {kind} n={n} h={h} l={l} eps={eps}", flush=True)
    pos, q = inputs.make(kind, n, 700 + l)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, l, "fp64", m2l_tolerance=eps)
    ref = plan.evaluate(q)
    for mode, tol in (("fp64_svd", 10 * eps), ("mixed_svd", 10 * eps + 1e-6)):
        plan.set_precision(mode)
        out = plan.evaluate(q)
        assert max(rel(o, r) for o, r in zip(out, ref)) <= tol, mode
