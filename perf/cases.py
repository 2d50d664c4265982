"""Performance cases: the solves that programs using this library run, over the
range of sizes, trees, orders, kernels and precisions it serves.

listed() gives the named cases, draw(rng) one more of the same ranges.  Every
case goes through the Python binding (paper_2508_02626_amd.fmm) with its inputs
on the GPU:
  solve     fmm.Plan + evaluate + close: new positions on every call (a served
            request, a time step of moving particles)
  evaluate  evaluate on a plan that is kept: fixed positions, new charges (an
            iterative solver's matrix-vector product)
  batch     fmm.plan_batch + evaluate_batch over many small problems
Points follow the repository's synthetic distributions (uniform cube, 3-D
Gaussian of unit deviation, Plummer sphere of radius 0.05 cut at 1, mixture of
8 Gaussian clusters); charges are U(-1, 1).
"""
import math

import torch

from paper_2508_02626_amd import fmm

DEVICE = "cuda:0"


def _case(name, what, dist, n, order, **kw):
    c = dict(name=name, what=what, dist=dist, n=n, order=order, leaf_size=64, depth=-1, precision="fp64",
             field=True, kernel="coulomb", softening=0.0, count=1)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest served request: the loosest accuracy (order 4, mixed
        # precision); latency and launches are all of it.
        _case("solve_1k_p4_mixed", "solve", "uniform", 1000, 4, precision="mixed"),
        # An iterative solver's product on a small fixed geometry.
        _case("evaluate_2k_p6_depth3", "evaluate", "uniform", 2000, 6, depth=3),
        # A served request of middling size on a clustered set, order 8.
        _case("solve_plummer_17k_p8", "solve", "plummer", 17389, 8),
        # The leaf-size / order sweep's 1e5 Gaussian (an odd size beside it).
        _case("solve_gaussian_100k_p6", "solve", "gaussian", 100003, 6),
        # A served request of the tightest accuracy, order 12.
        _case("solve_plummer_250k_p12", "solve", "plummer", 250007, 12),
        # Many small problems at once, orders 4, 6 and 8, mixed precision.
        _case("batch_32_mixed", "batch", "mixed", 200000, 8, precision="mixed", count=32),
        # The uniform benchmark: 1e6 points in a cube, full tree of depth 5.
        _case("solve_uniform_1m_p8", "solve", "uniform", 1000000, 8, depth=5),
        # The same through the mixed-precision path.
        _case("solve_uniform_1m_p8_mixed", "solve", "uniform", 1000000, 8, depth=5, precision="mixed"),
        # Potentials only, a kept plan, larger leaves (the sweep's order 10).
        _case("evaluate_gaussian_1m_p10_phi", "evaluate", "gaussian", 1000000, 10, leaf_size=128, field=False),
        # The softened (N-body) kernel on a full tree and on a clustered set.
        _case("solve_softened_1m_p8", "solve", "uniform", 1000000, 8, depth=5, kernel="softened",
              softening=1e-3),
        _case("solve_softened_plummer_1m_p8", "solve", "plummer", 1000000, 8, kernel="softened",
              softening=1e-4),
        # The headline benchmark: 4e6 clustered points to an error of 1e-7.
        _case("solve_plummer_4m_p14", "solve", "plummer", 4000000, 14),
    ]


def draw(rng):
    what = rng.choice(["solve", "solve", "solve", "evaluate", "batch"])
    n = int(math.exp(rng.uniform(math.log(1000), math.log(1.0e6)))) | 1
    if what == "batch":
        n = int(math.exp(rng.uniform(math.log(1.0e4), math.log(2.0e5)))) | 1
        return dict(what=what, dist="mixed", n=n, order=8, leaf_size=rng.choice([32, 64]), depth=-1,
                    precision=rng.choice(["fp64", "mixed"]), field=True, kernel="coulomb", softening=0.0,
                    count=rng.randint(8, 32))
    kernel = rng.choice(["coulomb", "coulomb", "coulomb", "softened"])
    dist = rng.choice(["uniform", "gaussian", "plummer", "clusters"])
    order = rng.choice([4, 5, 6, 7, 8] if kernel == "softened" else [2, 4, 6, 7, 8, 10, 12, 13, 14])
    depth = -1
    if dist == "uniform" and rng.random() < 0.5:  # a full tree of about 15 to 120 points a leaf
        depth = max(2, int(math.log(n / rng.uniform(15, 120)) / math.log(8) + 0.5))
    precision = "fp64" if kernel == "softened" else rng.choice(["fp64", "fp64", "fp64", "mixed"])
    return dict(what=what, dist=dist, n=n, order=order, leaf_size=rng.choice([32, 48, 64, 100, 128]), depth=depth,
                precision=precision, field=rng.random() < 0.75, kernel=kernel,
                softening=rng.choice([1e-4, 1e-3, 1e-2]) if kernel == "softened" else 0.0, count=1)


def _points(dist, n, gen):
    """n points and charges of a distribution, FP64 on the GPU."""
    opt = dict(dtype=torch.float64, device=DEVICE, generator=gen)
    if dist == "uniform":
        x = torch.rand(n, 3, **opt)
    elif dist == "gaussian":
        x = torch.randn(n, 3, **opt)
    elif dist == "plummer":
        a, rmax = 0.05, 1.0
        u = torch.rand(n, **opt).clamp_min(1e-12) * (1.0 + (a / rmax) ** 2) ** -1.5  # cut at rmax
        v = torch.randn(n, 3, **opt)
        x = v / v.norm(dim=1, keepdim=True) * (a / torch.sqrt(u ** (-2.0 / 3.0) - 1.0))[:, None]
    elif dist == "clusters":
        c = torch.rand(8, 3, **opt) * 0.8 + 0.1
        lab = torch.randint(0, 8, (n,), device=DEVICE, generator=gen)
        x = c[lab] + 0.02 * torch.randn(n, 3, **opt)
    else:
        raise ValueError(dist)
    q = torch.rand(n, **opt) * 2.0 - 1.0
    return x, q


def _problems(case):
    """(distribution, size, order) of each problem of a batch: sizes spread over
    the logarithm from 1e3 to n, half uniform cubes and half clusters."""
    m = case["count"]
    out = []
    for i in range(m):
        t = ((i * 29) % m) / max(1, m - 1)
        n = int(1000.0 * (case["n"] / 1000.0) ** t)
        out.append(("uniform" if i % 2 == 0 else "clusters", n, (4, 6, 8)[i % 3]))
    return out


def _plan_options(case):
    kw = dict(leaf_size=case["leaf_size"], precision=case["precision"], want_field=case["field"])
    if case["depth"] >= 0:
        kw.update(uniform_depth=case["depth"], root=[0.0, 0.0, 0.0, 1.0])
    if case["kernel"] != "coulomb":
        kw.update(kernel=case["kernel"], softening=case["softening"])
    return kw


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    if case["what"] == "batch":
        return [_points(d, n, gen) for d, n, _ in _problems(case)]
    return [_points(case["dist"], case["n"], gen)]


def prepare(case, seed):
    pts = _inputs(case, seed)
    state = dict(case=case, x=[x for x, _ in pts], q=[q for _, q in pts])
    if case["what"] == "batch":
        state["orders"] = [p for _, _, p in _problems(case)]
    if case["what"] == "evaluate":
        state["plan"] = fmm.Plan(state["x"][0], case["order"], **_plan_options(case))
    return state


def run(state):
    case = state["case"]
    if case["what"] == "batch":
        plans = fmm.plan_batch(state["x"], state["orders"], leaf_size=case["leaf_size"],
                               precision=case["precision"], threads=8)
        outs = fmm.evaluate_batch(plans, state["q"])
        for pl in plans:
            pl.close()
        return [v for out in outs for v in out]
    if case["what"] == "evaluate":
        phi, fld = state["plan"].evaluate(state["q"][0], want_field=case["field"])
    else:
        pl = fmm.Plan(state["x"][0], case["order"], **_plan_options(case))
        phi, fld = pl.evaluate(state["q"][0], want_field=case["field"])
        pl.close()
    return [phi, fld] if case["field"] else [phi]


def work(case):
    """Inputs read and outputs written once, and the operations of the method:
    the near-field pairs (about 20 operations each with the field, 12 without)
    and the far-field translations of the boxes (one contraction per sign class
    of source offsets: 26 full, 24 half and 6 quarter ones).  A box of an
    adaptive tree holds about 0.4 leaf sizes of points."""
    if case["what"] == "batch":
        probs = [(n, p) for _, n, p in _problems(case)]
    else:
        probs = [(case["n"], case["order"])]
    nbytes = flops = 0
    for n, p in probs:
        per = n / 8.0 ** case["depth"] if case["depth"] >= 0 else 0.4 * case["leaf_size"]
        coef = (p + 1) ** 2 if case["kernel"] == "coulomb" else (p + 1) * (p + 2) * (p + 3) // 6
        boxes = 8.0 / 7.0 * n / per
        nbytes += n * (24 + 8 + 8 + (24 if case["field"] else 0))
        flops += int(n * min(n, 27.0 * per) * (20 if case["field"] else 12) + boxes * 79.0 * coef * coef)
    return {"bytes": nbytes, "flops": flops}


def _direct(x, q, eps, field):
    """Direct sum in FP64, pairs at distance zero left out (j = i alone when
    the kernel is softened)."""
    n = x.shape[0]
    phi = torch.empty(n, dtype=torch.float64, device=x.device)
    fld = torch.empty(n, 3, dtype=torch.float64, device=x.device) if field else None
    step = max(1, (1 << 26) // n)
    for a in range(0, n, step):
        b = min(n, a + step)
        d = [x[a:b, k, None] - x[None, :, k] for k in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps * eps
        if eps > 0.0:
            r2[torch.arange(b - a, device=x.device), torch.arange(a, b, device=x.device)] = math.inf
        else:
            r2[r2 == 0.0] = math.inf
        inv = r2.rsqrt_()
        w = inv * q
        phi[a:b] = w.sum(1)
        if field:
            w.mul_(inv).mul_(inv)
            for k in range(3):
                fld[a:b, k] = d[k].mul_(w).sum(1)
    return phi, fld


def exact(case, seed):
    if case["what"] == "batch" or case["n"] > 300000:
        return None  # the direct sum over all pairs takes too long
    x, q = _inputs(case, seed)[0]
    phi, fld = _direct(x, q, case["softening"], case["field"])
    return [phi, fld] if case["field"] else [phi]
