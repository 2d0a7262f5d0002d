"""The near field's wavefronts per leaf (1, 4 and 16) and the splits of small,
odd and crowded leaves, against the exact pairwise sums: with height 2 every
pair is a near one.  Coincident particles add zero.  FP64: each pair within a
few roundings, so 1e-13 of the sum of magnitudes; FP32 pairs: 1e-6 of it.
Distances whose squares leave the FP64 range take the library's root."""
import numpy as np
import pytest
import torch

import oracle
from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def exact(pos, q, p, sel):
    d = pos[sel, None, :] - pos[None, :, :]
    r2 = (d * d).sum(-1)
    ir = torch.where(r2 > 0, r2, torch.inf) ** -0.5
    w = q[None, :] * ir ** p
    return w.sum(1), q[sel, None] * (p * (w * ir * ir)[..., None] * d).sum(1), \
        w.abs().sum(1), q[sel].abs() * (p * (w * ir * ir).abs() * r2.sqrt()).sum(1)


@pytest.mark.parametrize("kernel", ["inv_r", "inv_r2"])
@pytest.mark.parametrize("n", [1, 2, 9, 131, 515, 4099, 9001])
def test_all_pairs_of_few_leaves(n, kernel):
    print(f"near n={n} {kernel}", flush=True)
    pos, q = inputs.uniform_cube(n, 900 + n)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    pos[n // 2] = pos[0]  # two at one place
    plan = fmm.Plan(pos, 2, 3)
    plan.set_kernel(kernel)
    sel = torch.linspace(0, n - 1, min(n, 300), device="cuda").long()
    p, f, ps, fs = exact(pos, q, 2 if kernel == "inv_r2" else 1, sel)
    for mode, tol in (("fp64", 1e-13), ("mixed", 1e-6)):
        plan.set_precision(mode)
        phi, force = plan.evaluate(q)
        assert ((phi[sel] - p).abs() <= tol * ps).all(), mode
        assert ((force[sel] - f).abs() <= tol * fs[:, None]).all(), mode


# leaves of about 1, 10, 20, 60, 200 and 1000 particles: the three widths, one
# and two batches of targets; tolerances as for the whole evaluation
@pytest.mark.parametrize("kind,n,h", [("cube", 900, 5), ("cube", 40_001, 5), ("cube", 80_001, 5),
                                      ("cube", 31_000, 4), ("sphere", 60_001, 4),
                                      ("cube", 20_001, 3)])
def test_widths_match_oracle(kind, n, h):
    print(f"near {kind} n={n} h={h}", flush=True)
    pos, q = inputs.make(kind, n, 950 + h)
    ref = oracle.Tree(pos, h).fmm(3, q)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), h, 3)
    for mode, tol in (("fp64", 1e-12), ("mixed", 1e-6)):
        plan.set_precision(mode)
        out = plan.evaluate(torch.from_numpy(q).cuda())
        for a, b in zip(out, ref):
            assert np.linalg.norm(a.cpu().numpy() - b) <= tol * np.linalg.norm(b), mode


def test_squares_out_of_range():
    """r^2 denormal: the potential scales as 1/r; infinite: 1/r is zero."""
    pos, q = inputs.uniform_cube(300, 990)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
    sel = torch.arange(300, device="cuda")
    p, _, ps, _ = exact(pos, q, 1, sel)
    small, _ = fmm.Plan(pos * 1e-154, 2, 3).evaluate(q)
    # squares down to 1e-312 keep 12 bits fewer than 1e-308: 1e-11 of it
    assert ((small * 1e-154 - p).abs() <= 1e-9 * ps).all()
    large = fmm.Plan(pos * 1e160, 2, 3).evaluate(q)
    assert (large[0] == 0).all() and (large[1] == 0).all()
