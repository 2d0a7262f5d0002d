"""Performance cases of the FMM library, through its Python binding.

What a program that uses the library has it do:

  step      positions that have just moved: plan, evaluate, release (the
            time step of a particle simulation; what ``bench.py`` times)
  evaluate  new charges on positions that stay: one evaluation of a plan the
            program keeps (an iterative solver, a boundary element method)
  serve     a burst of independent requests through the serving loop
  direct    exact sums at sampled targets, the check of an FMM result

Sizes, heights and orders are those of ``inputs.CONFIGS``, of the serving
request mixes and of the tests, and odd ones between them.  Inputs follow
``inputs.py`` (uniform cube, jittered unit sphere, charges in [-1, 1)) and are
drawn on the GPU.
"""
import math

import torch

from paper_1206_0115_amd import fmm

LISTED = [
    # The smallest call: a thousand particles, one M2L level; all latency.
    dict(name="step_cube_1k", path="step", kind="cube", n=1000, height=3, order=4,
         precision="fp64"),
    # A small kept plan with new charges, the size the smoke test evaluates:
    # the launches of one evaluation.
    dict(name="evaluate_cube_4k", path="evaluate", kind="cube", n=4000, height=4, order=5,
         precision="fp64"),
    # The smallest benchmark configuration, in the library's default mode.
    dict(name="step_cube_20k", path="step", kind="cube", n=20_000, height=4, order=5,
         precision="fp64"),
    # The upper end of the serving tests' requests, odd, on a surface, dense
    # mixed mode.
    dict(name="step_sphere_60k", path="step", kind="sphere", n=59_999, height=5, order=7,
         precision="mixed"),
    # The second kernel, 1/r^2, compressed, on a surface.
    dict(name="evaluate_sphere_200k_inv_r2", path="evaluate", kind="sphere", n=200_003, height=6,
         order=5, precision="mixed_svd", kernel="inv_r2"),
    # A solver's matrix-vector product at order 8, compressed FP64, full
    # leaves (73 particles each) and an odd count.
    dict(name="evaluate_cube_300k_order8", path="evaluate", kind="cube", n=300_007, height=5,
         order=8, precision="fp64_svd"),
    # The order-10 workload at the density of the 30M-particle configuration
    # (1.8 particles per leaf) and the tolerance it runs at.
    dict(name="evaluate_cube_469k_order10", path="evaluate", kind="cube", n=468_750, height=7,
         order=10, precision="mixed_svd", tol=2e-7),
    # The 1M cube's time step in the compressed mixed mode ...
    dict(name="step_cube_1m", path="step", kind="cube", n=1_000_000, height=6, order=7,
         precision="mixed_svd"),
    # ... and in the library's default mode, dense FP64.
    dict(name="step_cube_1m_fp64", path="step", kind="cube", n=1_000_000, height=6, order=7,
         precision="fp64"),
    # The sphere configuration: 10M particles on a surface, near field as
    # heavy as the far field; the largest buffers here.
    dict(name="step_sphere_10m", path="step", kind="sphere", n=10_000_000, height=8, order=7,
         precision="mixed_svd"),
    # A burst of requests of the serving mix, waited for together.
    dict(name="serve_16", path="serve", n=60_000, requests=16, precision="mixed_svd"),
    # Checking a result of the 1M cube at sampled targets.
    dict(name="direct_cube_1m", path="direct", kind="cube", n=1_000_000, targets=1024,
         kernel="inv_r"),
]

EXACT_MAX_PAIRS = 2.6e11  # pairs exact() sums within about 20 seconds


def listed():
    return [dict(c) for c in LISTED]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _height(kind, n, per_leaf):
    """The height whose leaves hold about `per_leaf` particles."""
    h = 3
    while h < 8 and n / _cells(kind, n, h) > per_leaf:
        h += 1
    return h


def draw(rng):
    top = max(_cost(c) for c in LISTED)
    path = rng.choice(["step", "step", "step", "evaluate", "evaluate", "evaluate", "serve",
                       "direct"])
    if path == "serve":
        return dict(path="serve", n=_log_int(rng, 4000, 60_000), requests=rng.randint(3, 16),
                    precision=rng.choice(["fp64", "fp64_svd", "mixed", "mixed_svd"]))
    kind = rng.choice(["cube", "sphere"])
    if path == "direct":
        return dict(path="direct", kind=kind, n=_log_int(rng, 20_000, 1_000_000),
                    targets=_log_int(rng, 64, 1024), kernel=rng.choice(["inv_r", "inv_r2"]))
    while True:
        n = _log_int(rng, 1000, 1_000_000)
        case = dict(path=path, kind=kind, n=n,
                    height=_height(kind, n, math.exp(rng.uniform(math.log(4), math.log(100)))),
                    order=rng.choice([3, 4, 5, 5, 6, 7, 7, 8, 9]),
                    precision=rng.choice(["fp64", "fp64", "mixed", "fp64_svd", "mixed_svd",
                                          "mixed_svd"]))
        if rng.random() < 0.15:
            case["kernel"] = "inv_r2"
        if path == "evaluate" and rng.random() < 0.2:
            case["graph"] = True
        if _cost(case) <= top:
            return case


# ------------------------------------------------------------------ inputs
def _particles(kind, n, gen):
    dev = gen.device
    if kind == "cube":
        pos = torch.rand(n, 3, dtype=torch.float64, device=dev, generator=gen)
    else:
        v = torch.randn(n, 3, dtype=torch.float64, device=dev, generator=gen)
        r = 1.0 + 1e-3 * (2.0 * torch.rand(n, 1, dtype=torch.float64, device=dev,
                                           generator=gen) - 1.0)
        pos = (v / v.norm(dim=1, keepdim=True) * r).contiguous()
    q = 2.0 * torch.rand(n, dtype=torch.float64, device=dev, generator=gen) - 1.0
    return pos, q


def _requests(case):
    """(kind, n, height, order) of each request: sizes spread over the mix's
    range, from a fifteenth of the largest up."""
    out = []
    for i in range(case["requests"]):
        kind = "cube" if i % 3 else "sphere"
        n = int(case["n"] * 15.0 ** (-((7 * i) % case["requests"]) / case["requests"])) | 1
        out.append((kind, n, _height(kind, n, 48), (5, 7, 3)[i % 3]))
    return out


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    if case["path"] == "serve":
        return [(*_particles(kind, n, gen), h, l) for kind, n, h, l in _requests(case)]
    pos, q = _particles(case["kind"], case["n"], gen)
    if case["path"] == "direct":
        tg = torch.randperm(case["n"], device="cuda", generator=gen)[:case["targets"]].contiguous()
        return pos, q, tg
    return pos, q


def _plan(case, pos):
    return fmm.Plan(pos, case["height"], case["order"], case["precision"],
                    kernel=case.get("kernel", "inv_r"), m2l_tolerance=case.get("tol"))


def prepare(case, seed):
    data = _inputs(case, seed)
    state = dict(case=case, data=data)
    if case["path"] == "evaluate":
        state["plan"] = _plan(case, data[0])
        if case.get("graph"):
            state["plan"].set_graph(True)
    elif case["path"] == "serve":
        state["server"] = fmm.Server(64 << 30, max_active=32)
    return state


def run(state):
    case, data = state["case"], state["data"]
    if case["path"] == "step":
        pos, q = data
        plan = _plan(case, pos)
        out = plan.evaluate(q)
        plan.release()
        return out
    if case["path"] == "evaluate":
        return state["plan"].evaluate(data[1])
    if case["path"] == "direct":
        pos, q, tg = data
        return fmm.direct_sampled(pos, q, tg, kernel=case["kernel"])
    srv = state["server"]
    reqs = [srv.submit(pos, q, h, l, case["precision"]) for pos, q, h, l in data]
    for r in reqs:
        if r.wait().status != fmm.FMM_OK:
            raise RuntimeError("request failed: " + r.error())
    return [(r.potential, r.forces) for r in reqs]


# ------------------------------------------------------------------- exact
def _direct(pos, q, rows, kernel):
    """Potentials and forces at particles `rows`: plain pairwise sums."""
    n = pos.shape[0]
    step = max(1, int(2.5e8 // n))
    phi = torch.empty(len(rows), dtype=torch.float64, device=pos.device)
    f = torch.empty(len(rows), 3, dtype=torch.float64, device=pos.device)
    for a in range(0, len(rows), step):
        i = rows[a:a + step]
        r2 = torch.zeros(len(i), n, dtype=torch.float64, device=pos.device)
        for d in range(3):
            t = pos[i, d][:, None] - pos[None, :, d]
            r2.addcmul_(t, t)
        r2.masked_fill_(r2 == 0.0, math.inf)
        w = r2.reciprocal() if kernel == "inv_r2" else r2.rsqrt()
        phi[a:a + step] = w @ q
        w.div_(r2).mul_(2.0 if kernel == "inv_r2" else 1.0)
        for d in range(3):
            t = pos[i, d][:, None] - pos[None, :, d]
            f[a:a + step, d] = q[i] * (t.mul_(w) @ q)
    return phi, f


def exact(case, seed):
    if case["path"] == "serve":
        if sum(float(n) ** 2 for _, n, _, _ in _requests(case)) > EXACT_MAX_PAIRS:
            return None
        return [_direct(pos, q, torch.arange(len(q), device=q.device), "inv_r")
                for pos, q, _, _ in _inputs(case, seed)]
    if float(case["n"]) * case.get("targets", case["n"]) > EXACT_MAX_PAIRS:
        return None
    data = _inputs(case, seed)
    rows = data[2] if case["path"] == "direct" else torch.arange(case["n"], device="cuda")
    return _direct(data[0], data[1], rows, case.get("kernel", "inv_r"))


# -------------------------------------------------------------------- work
def _cells(kind, n, height):
    """About how many leaves hold a particle."""
    side = 2 ** (height - 1)
    slots = side ** 3 if kind == "cube" else max(1.0, 4.7 * side ** 2)
    return slots * -math.expm1(-n / slots)


def _fmm_work(kind, n, height, order, precision, tol=None):
    """Algorithmic flops: 20 per near pair, 2 l^6 (dense) or 4 l^3 r
    (compressed, r the mean kept rank) per far pair of cells, and the
    interpolations; bytes: particles in, potentials and forces out."""
    l3 = float(order) ** 3
    leaves = _cells(kind, n, height)
    side = 2 ** (height - 1)
    per = 3 - 2 / side  # neighbours along an axis, the cell itself included
    near = n * max(1.0, n / leaves) * (per ** 3 if kind == "cube" else min(per ** 3, 13.0))
    rank = l3
    if precision.endswith("_svd"):
        digits = -math.log10(tol) if tol else min(order, 10)
        rank = min(l3, 0.38 * digits ** 2 + 0.65 * digits)
    far, cells = 0.0, 0.0
    for lv in range(2, height):
        c = _cells(kind, n, lv + 1)
        s = 2 ** lv
        cells += c
        full = (6 - 8 / s) ** 3 - (3 - 2 / s) ** 3
        # empty cells are no sources; a surface keeps about a fifth
        far += c * (full * c / s ** 3 if kind == "cube" else min(0.2 * full, c))
    per_pair = 4 * l3 * rank if precision.endswith("_svd") else 2 * l3 * l3
    flops = (20 * near + per_pair * far + 12 * float(order) ** 4 * cells
             + n * (6 * l3 + 9 * order ** 2))
    return {"bytes": 64.0 * n, "flops": flops}


def work(case):
    if case["path"] == "direct":
        return {"bytes": 32.0 * case["n"] + 32.0 * case["targets"],
                "flops": 20.0 * case["n"] * case["targets"]}
    if case["path"] == "serve":
        each = [_fmm_work(k, n, h, l, case["precision"]) for k, n, h, l in _requests(case)]
        return {"bytes": sum(w["bytes"] for w in each), "flops": sum(w["flops"] for w in each)}
    return _fmm_work(case["kind"], case["n"], case["height"], case["order"], case["precision"],
                     case.get("tol"))


def _cost(case):
    """Work in units of FP32 matrix flops (FP64 runs at half the rate)."""
    half = case.get("precision", "fp64").startswith("fp64")
    return work(case)["flops"] * (2.0 if half else 1.0)
