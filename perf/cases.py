"""Workloads of the force step and its companions, for timing and comparison.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call (particles on
the GPU, a context with its workspace, output arrays), ``run(state)`` is one
pass through the public entry points, ``work(case)`` the bytes and flops a pass
cannot do without, and ``exact(case, seed)`` the outputs in float64 from direct
sums (None where that takes too long).

Kinds of case:

* ``static``    one force step on the library's own workspace (forces_static):
                the smallest calls, bound by launches and latency.
* ``step``      one force step of a single system through a context: build,
                multipoles, walk (every particle's acceleration and potential).
* ``ensemble``  one batched step of many independent systems of uneven size,
                eager or replayed from a captured graph.
* ``active``    one tick of block time steps: the tree is refitted to drifted
                positions and only the due particles are walked.
* ``leapfrog``  a few shared-time-step kick-drift-kick steps.
* ``sph``       one gas step: tree, moments and SPH density.
* ``neighbors`` one neighbour-list step: tree, moments and CSR lists, which the
                program then puts in ascending order (the library leaves the
                order inside a list open) in a buffer of its own.
* ``estimator`` one training step of the work estimator: gradient and Adam.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1204_2280_amd import estimator, mibh, workloads

DIRECT_MAX = 320_000  # particles of a direct float64 sum that takes seconds, not minutes


def listed():
    return [
        # a small cluster inside a serving or planning loop: nothing but launches and latency
        {"name": "static_1000", "kind": "static", "model": "plummer", "n": 1000, "theta": 0.75},
        # the paper's smallest sphere: a step too small to fill the chip
        {"name": "step_32768", "kind": "step", "model": "plummer", "n": 32768, "theta": 0.75,
         "precision": "plain", "eps2": 0.0, "equal_mass": True},
        # a mid-size odd-sized cuspy halo at the small opening angle
        {"name": "step_hernquist_100003", "kind": "step", "model": "hernquist", "n": 100003, "theta": 0.5,
         "precision": "plain", "eps2": 0.0, "equal_mass": True},
        # softened, unequal masses, compensated sums, wide opening angle
        {"name": "step_kahan_300007", "kind": "step", "model": "plummer", "n": 300007, "theta": 1.0,
         "precision": "kahan", "eps2": 1e-4, "equal_mass": False},
        # the paper's sphere of 2^20 bodies
        {"name": "step_1m", "kind": "step", "model": "plummer", "n": 1 << 20, "theta": 0.75,
         "precision": "plain", "eps2": 0.0, "equal_mass": True},
        # the paper's largest sphere, the headline step
        {"name": "step_4m", "kind": "step", "model": "plummer", "n": 1 << 22, "theta": 0.75,
         "precision": "plain", "eps2": 0.0, "equal_mass": True},
        # the benchmark's ensemble: 64 uneven systems in one graph-replayed step
        {"name": "ensemble_64", "kind": "ensemble", "nsys": 64, "lo": 12, "hi": 18, "theta": 0.75, "graph": True},
        # a tick of block time steps: 15% of the particles due on a refitted tree
        {"name": "active_1m", "kind": "active", "model": "plummer", "n": 1 << 20, "theta": 0.75, "share": 0.15},
        # a short run of a small cluster with the native integrator
        {"name": "leapfrog_20011", "kind": "leapfrog", "n": 20011, "theta": 0.75, "steps": 4},
        # a gas step with about 64 neighbours inside the kernel's support
        {"name": "sph_250007", "kind": "sph", "n": 250007, "ngb": 64},
        # neighbour lists of a mid-size sphere, each list in ascending order
        {"name": "neighbors_131072", "kind": "neighbors", "n": 1 << 17, "ngb": 64},
        # one training step of the work estimator at its default batch
        {"name": "estimator_1024", "kind": "estimator", "rows": 30000, "batch": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["static", "step", "step", "step", "ensemble", "active", "leapfrog", "sph", "neighbors",
                       "estimator"])
    theta = rng.choice([0.5, 0.6, 0.75, 0.75, 0.9, 1.0])
    model = rng.choice(["plummer", "hernquist"])
    if kind == "static":
        return {"kind": kind, "model": model, "n": _log_int(rng, 300, 32768), "theta": theta}
    if kind == "step":
        top = (1 << 20) if theta < 0.75 else (1 << 22)
        return {"kind": kind, "model": model, "n": _log_int(rng, 3000, top), "theta": theta,
                "precision": rng.choice(["plain", "plain", "kahan"]), "eps2": rng.choice([0.0, 1e-4]),
                "equal_mass": rng.random() < 0.5}
    if kind == "ensemble":
        return {"kind": kind, "nsys": rng.randint(2, 64), "lo": rng.randint(8, 12), "hi": rng.randint(13, 17),
                "theta": max(theta, 0.75), "graph": rng.random() < 0.5}
    if kind == "active":
        return {"kind": kind, "model": "plummer", "n": _log_int(rng, 20000, 1 << 21), "theta": max(theta, 0.75),
                "share": round(rng.uniform(0.02, 0.6), 3)}
    if kind == "leapfrog":
        return {"kind": kind, "n": _log_int(rng, 1000, 200000), "theta": max(theta, 0.75), "steps": rng.randint(1, 6)}
    if kind == "sph":
        return {"kind": kind, "n": _log_int(rng, 5000, 1 << 20), "ngb": rng.choice([32, 48, 64])}
    if kind == "neighbors":
        return {"kind": kind, "n": _log_int(rng, 5000, 1 << 18), "ngb": rng.choice([16, 32, 64])}
    return {"kind": kind, "rows": _log_int(rng, 2000, 200000), "batch": _log_int(rng, 100, 8192)}


# ---------------------------------------------------------------------------
# inputs, made on the GPU from the seed alone
# ---------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _isotropic(n, g):
    u = torch.rand((n, 2), generator=g, device="cuda", dtype=torch.float64)
    c, p = 2.0 * u[:, 0] - 1.0, 2.0 * math.pi * u[:, 1]
    s = torch.sqrt(torch.clamp(1.0 - c * c, min=0.0))
    return torch.stack([s * torch.cos(p), s * torch.sin(p), c], dim=1)


def _positions(model, n, g):
    """Sphere of the named model, centre of mass at the origin (float32 [n, 3])."""
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    if model == "plummer":
        r = 1.0 / torch.sqrt(torch.clamp(0.999 * u, min=1e-30) ** (-2.0 / 3.0) - 1.0)
        scale = 3.0 * math.pi / 16.0
    else:
        x = torch.sqrt(u) * (50.0 / 51.0)
        r, scale = x / (1.0 - x), 1.0
    p = r[:, None] * _isotropic(n, g)
    return ((p - p.mean(dim=0)) * scale).to(torch.float32).contiguous()


def _masses(n, g, equal):
    m = torch.full((n,), 1.0 / n, dtype=torch.float32, device="cuda")
    if not equal:
        m = m * (0.5 + torch.rand(n, generator=g, device="cuda", dtype=torch.float32))
    return m


def _smoothing(pos, ngb):
    return torch.from_numpy(workloads.plummer_smoothing_lengths(pos.cpu().numpy(), ngb)).cuda()


def _sizes(case):
    """System sizes of an ensemble, log-uniform in [2^lo, 2^hi] (the same for every seed)."""
    return workloads.ensemble_sizes(case["nsys"], 4, case["lo"], case["hi"])


def _inputs(case, seed):
    """The case's particles (or training rows) alone, without a context."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "estimator":
        rows, batch = case["rows"], case["batch"]
        w32, w16 = estimator.init_weights(torch.device("cuda", 0), int(seed))
        x = torch.rand((rows, mibh.MLP_FEATURES), generator=g, device="cuda")
        t = 9.0 + 3.0 * x[:, 0] + 0.5 * torch.randn(rows, generator=g, device="cuda")
        idx = torch.randint(0, rows, (batch,), generator=g, device="cuda", dtype=torch.int32)
        m = 1e-2 * torch.randn(mibh.MLP_PARAMS, generator=g, device="cuda")
        v = 1e-3 * (0.5 + torch.rand(mibh.MLP_PARAMS, generator=g, device="cuda"))
        return {"w32": w32, "w16": w16, "x": x, "t": t, "idx": idx, "m": m, "v": v}
    if kind == "ensemble":
        sizes = _sizes(case)
        half = len(sizes) // 2
        pos = torch.cat([_positions("plummer" if k < half else "hernquist", int(s), g) for k, s in enumerate(sizes)])
        mass = torch.cat([torch.full((int(s),), 1.0 / int(s), dtype=torch.float32, device="cuda") for s in sizes])
        off = np.zeros(len(sizes) + 1, dtype=np.int64)
        off[1:] = np.cumsum(sizes)
        return {"pos": pos.contiguous(), "mass": mass, "offsets": off}
    n = case["n"]
    if kind == "leapfrog":
        p, v, m = workloads.plummer(n, int(seed) + 11)
        return {"pos": torch.from_numpy(p).cuda(), "vel": torch.from_numpy(v).cuda(),
                "mass": torch.from_numpy(m).cuda()}
    pos = _positions(case.get("model", "plummer"), n, g)
    d = {"pos": pos, "mass": _masses(n, g, case.get("equal_mass", True))}
    if kind in ("sph", "neighbors"):
        d["h"] = _smoothing(pos, case["ngb"])
        d["radius"] = 2.0 * d["h"]  # the kernel's support
    if kind == "active":
        # one tick of dt_max / 16 = 1/256 with velocities of the order of the dispersion; the particles
        # nearest to the centre (the largest accelerations) are due
        vel = 0.4 * torch.randn((n, 3), generator=g, device="cuda")
        d["pos1"] = (pos + vel / 256.0).contiguous()
        r2 = (pos.double() ** 2).sum(dim=1)
        k = max(1, int(case["share"] * n))
        d["active"] = (r2 <= torch.kthvalue(r2, k).values).to(torch.uint8)
    return d


def prepare(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    s = {"case": dict(case), **d}
    if kind == "estimator":
        s["grad"] = torch.empty(mibh.MLP_PARAMS, device="cuda")
        s["loss"] = torch.empty(1, device="cuda")
        s["scratch"] = torch.empty(int(mibh.lib().mibh_mlp_scratch_bytes(case["batch"])), dtype=torch.uint8,
                                   device="cuda")
        return s
    n = int(d["mass"].shape[0])
    s["acc"] = torch.zeros((n, 3), dtype=torch.float32, device="cuda")
    s["pot"] = torch.zeros((n,), dtype=torch.float32, device="cuda")
    if kind == "static":
        mibh.lib()
        return s
    par = {}
    if kind == "step":
        par = {"eps2": case["eps2"], "precision": mibh.KAHAN if case["precision"] == "kahan" else mibh.PLAIN}
    elif kind == "leapfrog":
        par = {"eps2": 1e-4}
    elif kind == "ensemble":
        par = {"max_systems": case["nsys"]}
    stream = None
    if kind == "ensemble" and case["graph"]:
        torch.cuda.current_stream().synchronize()  # the inputs are ready before another stream reads them
        stream = torch.cuda.Stream()
    ctx = s["ctx"] = mibh.Context(n, stream=stream, **par)
    if kind == "ensemble" and case["graph"]:
        ctx.graph_capture(s["pos"], s["mass"], s["offsets"], case["theta"], s["acc"], s["pot"])
    if kind == "neighbors":
        s["ids"] = torch.arange(n, device="cuda")
        # room for the outskirts of a small sphere too, whose kernels reach into the core
        s["lists"] = torch.zeros((3 * case["ngb"] + 128) * n, dtype=torch.int32, device="cuda")
    if kind == "active":  # the tree of the last rebuild
        ctx.build_tree(s["pos"], s["mass"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "static":
        mibh.forces_static(s["pos"], s["mass"], c["theta"], s["acc"], s["pot"])
        return {"acc": s["acc"], "pot": s["pot"]}
    if kind == "step":
        s["ctx"].forces(s["pos"], s["mass"], c["theta"], s["acc"], s["pot"])
        return {"acc": s["acc"], "pot": s["pot"]}
    if kind == "ensemble":
        if c["graph"]:
            s["ctx"].graph_launch()
        else:
            s["ctx"].forces_batch(s["pos"], s["mass"], s["offsets"], c["theta"], s["acc"], s["pot"])
        return {"acc": s["acc"], "pot": s["pot"]}
    if kind == "active":
        ctx = s["ctx"]
        ctx.refit(s["pos1"], s["mass"])
        ctx.compute_multipoles()
        ctx.compute_forces_active(c["theta"], s["active"], s["acc"], s["pot"])
        return {"acc": s["acc"], "pot": s["pot"]}
    if kind == "leapfrog":
        s["ctx"].leapfrog(s["pos"], s["vel"], s["mass"], c["theta"], 1.0 / 128, c["steps"], acc=s["acc"], pot=s["pot"])
        return {"pos": s["pos"], "vel": s["vel"], "acc": s["acc"], "pot": s["pot"]}
    if kind == "sph":
        ctx = s["ctx"]
        ctx.build_tree(s["pos"], s["mass"])
        ctx.compute_multipoles()
        rho, count = ctx.sph_density(s["h"])
        return {"rho": rho, "count": count}
    if kind == "neighbors":
        ctx = s["ctx"]
        ctx.build_tree(s["pos"], s["mass"])
        ctx.compute_multipoles()
        count, offset, index = ctx.neighbor_list(s["radius"])
        total = index.shape[0]
        owner = torch.repeat_interleave(s["ids"], count, output_size=total)
        s["lists"][:total] = torch.sort((owner << 32) + index).values.to(torch.int32)  # the low word: the index
        return {"count": count, "offset": offset, "lists": s["lists"]}
    mibh.mlp_gradient(s["w16"], s["x"], s["t"], s["idx"], s["grad"], s["loss"], s["scratch"])
    mibh.mlp_adam(s["w32"], s["w16"], s["grad"], s["m"], s["v"], 500, 1e-3)
    return {"grad": s["grad"], "loss": s["loss"], "w32": s["w32"], "w16": s["w16"], "m": s["m"], "v": s["v"]}


# ---------------------------------------------------------------------------
# work and exact values
# ---------------------------------------------------------------------------


def _interactions(n, theta):
    """Particle-cell and particle-particle terms per particle: the benchmark spheres' counts at 2^22
    (theta 0.5, 0.75, 1.0), falling with the logarithm of n and never more than the particles there are."""
    ts, pcs, pps = (0.5, 0.75, 1.0), (3114.0, 1286.0, 848.0), (902.0, 385.0, 309.0)
    f = lambda ys: float(np.exp(np.interp(theta, ts, np.log(ys))))  # noqa: E731
    depth = min(1.0, math.log2(max(n, 2)) / 22.0)
    return min(f(pcs) * depth, n / 4.0), min(f(pps), 0.75 * n)


def _force_work(n, theta, share=1.0):
    pc, pp = _interactions(n, theta)
    return {"bytes": 32.0 * n, "flops": share * n * (53.0 * pc + 20.0 * pp)}


def work(case):
    kind = case["kind"]
    if kind in ("static", "step"):
        return _force_work(case["n"], case["theta"])
    if kind == "ensemble":
        parts = [_force_work(int(s), case["theta"]) for s in _sizes(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if kind == "active":
        w = _force_work(case["n"], case["theta"], case["share"])
        w["bytes"] += case["n"]
        return w
    if kind == "leapfrog":
        n, steps = case["n"], case["steps"]
        w = _force_work(n, case["theta"])
        return {"bytes": 2.0 * 24 * n + 20 * n, "flops": (steps + 1) * w["flops"] + 18.0 * n * steps}
    if kind == "sph":
        return {"bytes": 28.0 * case["n"], "flops": 20.0 * case["n"] * case["ngb"]}
    if kind == "neighbors":
        return {"bytes": case["n"] * (28.0 + 4.0 * case["ngb"]), "flops": 8.0 * case["n"] * case["ngb"]}
    params = mibh.MLP_PARAMS
    return {"bytes": 4.0 * params * 8 + 36.0 * case["batch"], "flops": 6.0 * params * case["batch"] + 12.0 * params}


def _direct(pos, mass, eps2=0.0, targets=None):
    """Direct float64 sums: (acc, pot) of the targets (all particles by default)."""
    x, m = pos.double(), mass.double()
    t = x if targets is None else x[targets]
    acc, pot = torch.empty_like(t), torch.empty(len(t), dtype=torch.float64, device=t.device)
    step = max(1, 400_000_000 // max(1, len(x)))
    for b in range(0, len(t), step):
        r2 = torch.zeros((min(step, len(t) - b), len(x)), dtype=torch.float64, device=t.device)
        for a in range(3):
            r2 += (x[None, :, a] - t[b:b + step, a, None]).square_()
        same = r2 == 0
        w = r2.add_(eps2).rsqrt_()
        w[same] = 0.0
        del same
        pot[b:b + step] = -(w @ m)
        w = w.pow_(3).mul_(m[None, :])
        acc[b:b + step] = w @ x - w.sum(dim=1)[:, None] * t[b:b + step]
        del r2, w
    return acc, pot


def exact(case, seed):
    kind = case["kind"]
    if kind == "neighbors":
        return None
    if kind == "ensemble":
        if int(_sizes(case).max()) > 100_000:
            return None
        d = _inputs(case, seed)
        parts = [_direct(d["pos"][a:b], d["mass"][a:b]) for a, b in zip(d["offsets"][:-1], d["offsets"][1:])]
        return {"acc": torch.cat([p[0] for p in parts]), "pot": torch.cat([p[1] for p in parts])}
    if kind != "estimator" and case["n"] > (DIRECT_MAX if kind != "leapfrog" else 60_000):
        return None
    d = _inputs(case, seed)
    if kind in ("static", "step"):
        acc, pot = _direct(d["pos"], d["mass"], case.get("eps2", 0.0))
        return {"acc": acc, "pot": pot}
    if kind == "active":
        due = torch.nonzero(d["active"]).flatten()
        a, p = _direct(d["pos1"], d["mass"], 0.0, due)
        acc = torch.zeros((case["n"], 3), dtype=torch.float64, device="cuda")
        pot = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        acc[due], pot[due] = a, p
        return {"acc": acc, "pot": pot}
    if kind == "leapfrog":
        dt = 1.0 / 128
        x, v = d["pos"].double(), d["vel"].double()
        acc, pot = _direct(x, d["mass"], 1e-4)
        for _ in range(case["steps"]):
            v = v + 0.5 * dt * acc
            x = x + dt * v
            acc, pot = _direct(x, d["mass"], 1e-4)
            v = v + 0.5 * dt * acc
        return {"pos": x, "vel": v, "acc": acc, "pot": pot}
    if kind == "sph":
        x, m, h = d["pos"].double(), d["mass"].double(), d["h"].double()
        n = len(x)
        rho = torch.empty(n, dtype=torch.float64, device="cuda")
        order = torch.argsort(h)  # near particles have near smoothing lengths: the far tiles stay empty
        step = max(1, 200_000_000 // n)
        for b in range(0, n, step):
            i = order[b:b + step]
            r2 = torch.zeros((len(i), n), dtype=torch.float64, device="cuda")
            for a in range(3):
                r2 += (x[None, :, a] - x[i, a, None]).square_()
            row, col = torch.nonzero(r2 < (4.0 * h[i] * h[i])[:, None], as_tuple=True)
            hi = h[i][row]
            q = torch.sqrt(r2[row, col]) / hi
            w = torch.where(q < 1.0, 1.0 - 1.5 * q * q + 0.75 * q ** 3, 0.25 * (2.0 - q) ** 3)
            w = m[col] * w / (math.pi * hi ** 3)
            rho[i] = torch.zeros(len(i), dtype=torch.float64, device="cuda").index_add_(0, row, w)
            del r2
        return {"rho": rho, "count": None}
    # one training step of the estimator: mean squared error, then Adam with bias correction
    w = d["w16"].double().requires_grad_(True)
    i = d["idx"].long()
    x, t = d["x"][i].double(), d["t"][i].double()
    W1, b1, W2 = w[:512].reshape(64, 8), w[512:576], w[576:4672].reshape(64, 64)
    b2, w3, b3 = w[4672:4736], w[4736:4800], w[4800]
    y = torch.relu(torch.relu(x @ W1.T + b1) @ W2.T + b2) @ w3 + b3
    loss = ((y - t) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, w)
    m = 0.9 * d["m"].double() + 0.1 * grad
    v = 0.999 * d["v"].double() + 0.001 * grad * grad
    w32 = d["w32"].double() - 1e-3 * (m / (1.0 - 0.9 ** 500)) / (torch.sqrt(v / (1.0 - 0.999 ** 500)) + 1e-8)
    return {"grad": grad, "loss": loss.detach().reshape(1), "w32": w32, "w16": None, "m": m, "v": v}
