"""Requests that share a compressed M2L launch: the batch takes one item width
from all its tiles together, which for these small plans is twice the width
each takes alone, and the results still are the bits of the solo runs.  The
requests wait behind work on the caller's stream, so that they are planned
together."""
import numpy as np
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,l,n,h,k", [
    ("fp64_svd", 4, 4000, 4, 3),   # 64 tile ranges alone (16 columns), 192 together (32)
    ("fp64_svd", 5, 4000, 4, 3),
    ("fp64_svd", 7, 1000, 3, 3),   # 32 alone, 96 together
    ("fp64_svd", 9, 1000, 3, 3),
    ("mixed_svd", 5, 4000, 4, 3),
    ("mixed_svd", 9, 1000, 3, 3),
])
def test_batch_width_keeps_the_bits(precision, l, n, h, k):
    print(f"serve widths {precision} l={l} n={n} h={h} k={k}", flush=True)
    reqs = []
    for i in range(k):
        pos, q = inputs.uniform_cube(n + 7 * i, 1200 + 10 * l + i)
        reqs.append((torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()))
    solo = []
    for pos, q in reqs:
        plan = fmm.Plan(pos, h, l, precision)
        solo.append(plan.evaluate(q))
        torch.cuda.synchronize()
        plan.release()
    srv = fmm.Server(hbm_budget_bytes=8 << 30, max_active=8)
    a = torch.rand(8192, 8192, device="cuda")
    for _ in range(8):
        a = a @ a
        a = a / a.abs().max()
    tickets = [srv.submit(pos, q, h, l, precision) for pos, q in reqs]
    for i, (t, ref) in enumerate(zip(tickets, solo)):
        st = t.wait()
        assert st.status == fmm.FMM_OK, t.error()
        assert torch.equal(t.potential, ref[0]) and torch.equal(t.forces, ref[1]), i
    assert srv.stats().max_batch_jobs == k
    srv.close()
