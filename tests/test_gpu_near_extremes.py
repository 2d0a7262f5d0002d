"""The FP64 near field where r^2, 1/r^2 or the force leaves the FP64 range: a
pair 2^e apart, in one leaf and in two, gives what IEEE division and square
root give, infinities and the NaN of zero times infinity included; finite
values within 4 roundings (1e-15)."""
import numpy as np
import pytest
import torch

from paper_1206_0115_amd import fmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [1, 2])  # one leaf, two leaves
@pytest.mark.parametrize("e", [-530, -515, -340, 515, 600])
@pytest.mark.parametrize("kernel", ["inv_r", "inv_r2"])
def test_pair_out_of_range(kernel, e, h):
    print(f"near extremes {kernel} 2^{e} h={h}", flush=True)
    d, q = 2.0 ** e, np.array([0.75, -1.25])
    with np.errstate(all="ignore"):
        ir2 = 1.0 / np.float64(d * d)
        ir = 1.0 / np.sqrt(np.float64(d * d))
        w = ir2 if kernel == "inv_r2" else ir
        t = q[::-1] * w
        s = 2.0 * t * ir2 if kernel == "inv_r2" else t * ir * ir
        dx = np.array([[-d, 0.0, 0.0], [d, 0.0, 0.0]])
        ref = t, q[:, None] * (s[:, None] * dx)
    pos = torch.tensor([[0.0, 0.0, 0.0], [d, 0.0, 0.0]], dtype=torch.float64, device="cuda")
    plan = fmm.Plan(pos, h, 3)
    plan.set_kernel(kernel)
    for a, b in zip(plan.evaluate(torch.from_numpy(q).cuda()), ref):
        np.testing.assert_allclose(a.cpu().numpy(), b, rtol=1e-15, atol=0, equal_nan=True)
