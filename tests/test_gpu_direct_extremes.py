"""Exact sums over pairs at infinite, overflowing and underflowing distances,
in full blocks of sources and in the ragged rest: every pair at r^2 > 0 adds
what IEEE division and square root give (an infinite 1/r^2 of a close pair, the
NaN of zero times an infinite difference), other pairs nothing.  The same
values that are not finite; finite ones within 1e-13 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

from paper_1206_0115_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def exact(pos, q, idx, p):
    with np.errstate(all="ignore"):
        d = pos[idx][:, None, :] - pos[None, :, :]
        r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        on = r2 > 0
        r2 = np.where(on, r2, 1.0)
        ir2 = 1.0 / r2
        w = np.where(on, q * (ir2 if p == 2 else 1.0 / np.sqrt(r2)), 0.0)
        t = (p * w * ir2)[..., None] * np.where(on[..., None], d, 0.0)
        return w.sum(1), q[idx, None] * t.sum(1), np.abs(w).sum(1), np.abs(t).sum(1)


def same(a, b, scale):
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(np.where(np.isinf(b), b, 0), np.where(np.isinf(a), a, 0))
    ok = np.isfinite(b)
    assert (np.abs(a[ok] - b[ok]) <= 1e-13 * scale[ok]).all()


# one chunk of 300 sources, a wavefront 75: a block of 64 and 11 more
@pytest.mark.parametrize("kernel", ["inv_r", "inv_r2"])
@pytest.mark.parametrize("at", [10, 70])
@pytest.mark.parametrize("what", ["infinite source", "infinite target", "both infinite",
                                  "overflow", "close pair"])
def test_pairs_out_of_range(what, at, kernel):
    print(f"direct extremes {what} at {at} {kernel}", flush=True)
    pos, q = inputs.uniform_cube(300, 1400 + at)
    idx = np.array([0, 5, 100, 299])
    if what == "infinite source":
        pos[at] = [np.inf, 0.5, 0.25]
    elif what == "infinite target":
        pos[at] = [0.5, -np.inf, 0.25]
        idx[1] = at
    elif what == "both infinite":
        pos[at] = pos[at + 1] = [np.inf, 0.5, 0.25]
        idx[1] = at
    elif what == "overflow":
        pos[at] = [1e200, 0.5, 0.25]
        idx[1] = at
    else:  # r^2 = 2^-1060
        pos[at] = 0.0
        pos[at + 1] = [2.0 ** -530, 0.0, 0.0]
        idx[1:3] = [at, at + 1]
    phi, f = fmm.direct_sampled(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda(),
                                torch.from_numpy(idx).cuda(), kernel=kernel)
    p_o, f_o, ps, fs = exact(pos, q, idx, 1 if kernel == "inv_r" else 2)
    same(phi.cpu().numpy(), p_o, ps)
    same(f.cpu().numpy(), f_o, np.abs(q[idx, None]) * fs)
