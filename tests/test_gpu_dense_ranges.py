"""The dense M2L's offset ranges without the memory of their partial sums: a
server whose budget lies one byte below a plan's footprint runs it with one
item a tile that takes the ranges in turn, and the results are the bits of the
solo run, whose items take one range each.  The footprints differ by a whole
number of partial buffers, i.e. the solo run really had ranges; between them
the cases have a single level, more ranges than the eight loc_sum_kernel adds
at once, tiles of fewer active offsets than ranges, and empty groups."""
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,h,l,precision", [
    ("cube", 60, 3, 1, "fp64"),       # single particles
    ("cube", 900, 3, 4, "fp64"),      # level 2 only
    ("cube", 4000, 4, 5, "fp64"),
    ("cube", 4000, 4, 5, "mixed"),
    ("sphere", 5003, 5, 3, "fp64"),   # empty 16-target groups
    ("sphere", 900, 7, 2, "mixed"),   # tiles of a few targets and offsets
    ("cube", 1201, 3, 12, "fp64"),    # several M-blocks
    ("cube", 1201, 3, 7, "mixed"),
])
def test_ranges_without_partial_buffers(kind, n, h, l, precision):
    print(f"dense ranges {kind} n={n} h={h} l={l} {precision}", flush=True)
    pos, q = inputs.make(kind, n, 1300 + n + l)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    plan = fmm.Plan(pos, h, l, precision)
    ref = plan.evaluate(q)
    torch.cuda.synchronize()
    info = plan.info()
    part = 8 * info.ld * sum(info.ncell[2:h])
    whole = info.device_bytes
    plan.release()
    srv = fmm.Server(hbm_budget_bytes=whole - 1, max_active=2)
    t = srv.submit(pos, q, h, l, precision)
    st = t.wait()
    assert st.status == fmm.FMM_OK, t.error()
    parts, rest = divmod(whole - st.plan_bytes, part)
    print(f"  {parts + 1} ranges", flush=True)
    assert parts >= 1 and rest == 0
    assert torch.equal(t.potential, ref[0]) and torch.equal(t.forces, ref[1])
    srv.close()
