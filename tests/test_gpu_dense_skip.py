"""The dense M2L with and without the skipping of 16-target groups that have no
source at an offset: a plan of full tiles runs without, a serving batch always
with, and both give the same bits.  Orders of two and three M-tiles a wavefront
(those of one always skip), and a last M-block with fewer."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("l", [5, 6, 7, 9])
def test_skipping_keeps_the_bits(l, precision):
    n, h = 120_001, 6
    print(f"dense skip n={n} h={h} l={l} {precision}", flush=True)
    pos, q = inputs.uniform_cube(n, 1500 + l)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, l, precision)
    i = plan.info()
    assert 0 < 4 * i.m2l_active_slots - (i.m2l_groups - i.m2l_groups_empty) \
        < 0.05 * 4 * i.m2l_active_slots
    ref = plan.evaluate(q)
    torch.cuda.synchronize()
    plan.release()
    srv = fmm.Server(hbm_budget_bytes=32 << 30, max_active=1)
    t = srv.submit(pos, q, h, l, precision)
    assert t.wait().status == fmm.FMM_OK, t.error()
    assert torch.equal(t.potential, ref[0]) and torch.equal(t.forces, ref[1])
    srv.close()
