"""Neighbour searches of groups whose candidates fill the first pass' list and that
stay with their wave, or almost do: counts exactly as every pair's float32 distance
decides, lists as the sets of these pairs, densities against float64 sums within
2e-6 (positive terms, each rounded a few times at 6e-8, in float32 sums of a few
lists).  Uniform spheres of influence of one and of several lists, and so wide that
the stack spills; the same with few groups of wide radii, with radii that differ, with
a dense spot, with points that coincide, in a batch, and with few waves.
"""
import math

import numpy as np
import pytest

from gpu_helpers import gpu_context

pytestmark = pytest.mark.gpu


def _input(kind, n, k):
    rng = np.random.default_rng(101)
    pos = rng.random((n, 3)).astype(np.float32)
    r = np.full(n, (0.75 * k / n / math.pi) ** (1 / 3))
    if kind == "few":
        r[np.arange(n) % 997 != 0] = 0.02
    elif kind == "spot":
        r[((pos - 0.5) ** 2).sum(1) > 0.01] = 0.02
    elif kind == "spread":
        r *= 0.8 + 0.4 * rng.random(n)
    elif kind == "dense":
        pos[: n // 10] = 0.5 + 0.1 * (pos[: n // 10] - 0.5)
    elif kind == "points":  # leaves of 40, and one of 2000
        pos = pos[rng.integers(0, n // 40, n)]
        pos[:2000] = 0.25
    return pos, r.astype(np.float32)


def _pairs(pos, r, rows):
    """(row, neighbour) by the float32 predicate, each operation rounded."""
    import torch
    out = []
    for q in torch.split(rows, max(1, 100_000_000 // len(pos))):
        d = pos[None, :, :] - pos[q, None, :]
        d2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        i, j = torch.nonzero(d2 <= (r[q] * r[q])[:, None], as_tuple=True)
        out.append(torch.stack([q[i], j]))
    return torch.cat(out, dim=1)


def _check(ctx, pos, r, mass, first, last):
    """Counts, lists and densities of the particles first .. last, a system of their own."""
    import torch
    cnt, off, idx = ctx.neighbor_list(r)
    assert torch.equal(cnt, ctx.neighbor_count(r))
    rho, dcnt = ctx.sph_density(0.5 * r)
    rho2, _ = ctx.sph_density(0.5 * r)
    assert torch.equal(dcnt, cnt) and torch.equal(rho, rho2)
    p, rad, m = pos[first:last], r[first:last], mass[first:last].double()
    n = last - first
    rows = torch.arange(0, n, max(1, n // 3000), device="cuda")
    i, j = _pairs(p, rad, rows)
    assert torch.equal(torch.bincount(i, minlength=n)[rows], cnt[first:last].long()[rows])
    o = off.long()
    got = torch.cat([torch.sort(idx[o[first + q]:o[first + q + 1]].long() - first)[0] for q in rows.tolist()])
    assert torch.equal(got, j)
    h = 0.5 * rad.double()[i]
    q = (p[i].double() - p[j].double()).norm(dim=1) / h
    w = torch.where(q < 1, 1 - 1.5 * q * q + 0.75 * q ** 3, 0.25 * torch.clamp(2 - q, min=0) ** 3) / (math.pi * h ** 3)
    ref = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, i, m[j] * w)[rows]
    assert float(((rho[first:last].double()[rows] - ref) / ref).abs().max()) <= 2e-6


@pytest.mark.parametrize("kind,n,k,params", [
    ("cube", 60000, 450, {}), ("cube", 50000, 1500, {}), ("cube", 100003, 700, {}), ("cube", 40000, 4000, {}),
    ("few", 60000, 800, {}), ("spot", 60000, 800, {}), ("spread", 60000, 500, {}), ("dense", 70000, 300, {}),
    ("points", 60000, 500, {}), ("cube", 40000, 500, {"walk_waves": 24}), ("cube", 40000, 400, {"group_cap": 16})])
def test_full_lists(kind, n, k, params):
    import torch
    pos, r = (torch.from_numpy(x).cuda() for x in _input(kind, n, k))
    mass = torch.rand(n, generator=torch.Generator().manual_seed(3)).cuda() / n
    print(f"[gpu] full lists: {kind} n={n} k={k} {params}", flush=True)
    ctx = gpu_context(n, **params)
    ctx.build_tree(pos, mass)
    ctx.compute_multipoles()
    _check(ctx, pos, r, mass, 0, n)


def test_full_lists_in_a_batch():
    import torch
    parts = [_input("cube", 40000, 500), _input("spread", 33, 5), _input("cube", 60000, 900)]
    off = np.concatenate([[0], np.cumsum([len(r) for _, r in parts])])
    pos, r = (torch.from_numpy(np.concatenate([p[q] for p in parts])).cuda() for q in range(2))
    mass = torch.rand(int(off[-1]), generator=torch.Generator().manual_seed(4)).cuda()
    print("[gpu] full lists: batch", flush=True)
    ctx = gpu_context(int(off[-1]), max_systems=3)
    ctx.build_tree_batch(pos, mass, off)
    ctx.compute_multipoles()
    for a, b in zip(off[:-1], off[1:]):
        _check(ctx, pos, r, mass, int(a), int(b))
