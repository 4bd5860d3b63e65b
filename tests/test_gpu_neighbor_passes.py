"""Neighbour search with every group on eight waves (trees of up to 32768
particles) against the two passes of larger trees (a wave per group, eight for
the heavy ones): the same systems alone and inside a batch.  Counts and lists are
compared exactly, densities within 1e-5 (float32 sums of positive terms in two
orders: each rounds by at most 6e-8 times log2(n) + n / 64 partial sums).  The
systems have groups with few candidates, with several full lists of them, with
leaves of many particles at one point, and radii that reach nothing or all.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _system(k, n):
    rng = np.random.default_rng(70 + k)
    if k % 3 == 0:  # outskirts whose radii reach the core
        pos, _, _ = W.plummer(n, 70 + k, with_velocities=False)
        r = 2.0 * W.plummer_smoothing_lengths(pos, 48)
    elif k % 3 == 1:  # points of 100 particles each, some radii hold everything
        pos = rng.random((n, 3)).astype(np.float32)
        pos[: n // 2] = pos[: n // 2][np.arange(n // 2) // 100]
        r = np.where(np.arange(n) % 997 == 0, 2.0, 0.02)
    else:
        pos = rng.random((n, 3)).astype(np.float32)
        r = np.where(np.arange(n) % 7 == 0, 0.0, 0.05)
    return pos, rng.random(n).astype(np.float32) / n, r.astype(np.float32)


@pytest.mark.parametrize("params", [{}, {"walk_waves": 24}])
def test_passes_agree(params):
    import torch
    sizes = [30000, 6000, 25000, 1, 70, 9000]
    parts = [_system(k, n) for k, n in enumerate(sizes)]
    pos, mass, r = (torch.from_numpy(np.concatenate([p[q] for p in parts])).cuda() for q in range(3))
    h = torch.clamp(0.5 * r, min=1e-3)
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] > 65536
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes), **params)
    ctx.build_tree_batch(pos, mass, off)
    ctx.compute_multipoles()
    print(f"[gpu] neighbour passes: batch {params}", flush=True)
    cnt, o, idx = (t.cpu().numpy() for t in ctx.neighbor_list(r))
    rho, dcnt = ctx.sph_density(h)
    rho2, _ = ctx.sph_density(h)
    assert torch.equal(rho, rho2)
    for k, n in enumerate(sizes):
        print(f"[gpu] neighbour passes: system {k} n={n}", flush=True)
        s = slice(off[k], off[k + 1])
        one = gpu_context(n, **params)
        one.build_tree(pos[s].contiguous(), mass[s].contiguous())
        one.compute_multipoles()
        c1, o1, i1 = (t.cpu().numpy() for t in one.neighbor_list(r[s].contiguous()))
        np.testing.assert_array_equal(cnt[s], c1)
        np.testing.assert_array_equal(o[s] - o[off[k]], o1[:-1])
        own = np.repeat(np.arange(n), c1)
        a = idx[o[off[k]]:o[off[k + 1]]] - off[k]
        np.testing.assert_array_equal(a[np.lexsort((a, own))], i1[np.lexsort((i1, own))])
        rho1, d1 = one.sph_density(h[s].contiguous())
        assert torch.equal(dcnt[s], d1)
        assert float(((rho[s] - rho1).abs() / rho1).max()) <= 1e-5


@pytest.mark.parametrize("n", [3000, 70000])
def test_fill_with_earlier_counts(n):
    import torch
    from paper_1204_2280_amd import mibh
    pos, mass, r = (torch.from_numpy(x).cuda() for x in _system(0, n))
    ctx = gpu_context(n)
    ctx.build_tree(pos, mass)
    ctx.compute_multipoles()
    cnt, off, idx = ctx.neighbor_list(r)
    total = int(off[n])
    cnt2, off2, idx2 = ctx.neighbor_list(r, capacity=total + 10)
    assert torch.equal(cnt, cnt2) and torch.equal(off, off2) and torch.equal(idx, idx2)
    short = torch.full((total,), -7, dtype=torch.int32, device="cuda")
    st = mibh.lib().mibh_neighbor_fill(ctx.handle, r.data_ptr(), cnt.data_ptr(), off.data_ptr(), short.data_ptr(),
                                       total - 5)
    assert st == 0
    ctx.sync()
    assert torch.equal(short[:-5], idx[:-5]) and bool((short[-5:] == -7).all())
    assert mibh.lib().mibh_neighbor_fill(ctx.handle, r.data_ptr(), cnt.data_ptr(), None, short.data_ptr(), 5) == -1


@pytest.mark.parametrize("n", [32768, 32769, 65537])
def test_both_sides_of_the_pass_lines(n):
    import torch
    pos, mass, r = (torch.from_numpy(x).cuda() for x in _system(0, n))
    far = (pos + 100.0).contiguous()  # a second system, to reach more particles
    one = gpu_context(n)
    one.build_tree(pos, mass)
    one.compute_multipoles()
    both = gpu_context(2 * n, max_systems=2)
    both.build_tree_batch(torch.cat([pos, far]), torch.cat([mass, mass]), np.array([0, n, 2 * n]))
    both.compute_multipoles()
    print(f"[gpu] neighbour pass lines: n={n}", flush=True)
    c1, o1, i1 = (t.cpu().numpy() for t in one.neighbor_list(r))
    c2, o2, i2 = (t.cpu().numpy() for t in both.neighbor_list(torch.cat([r, r])))
    np.testing.assert_array_equal(c1, c2[:n])
    own = np.repeat(np.arange(n), c1)
    i2 = i2[: o2[n]]
    np.testing.assert_array_equal(i1[np.lexsort((i1, own))], i2[np.lexsort((i2, own))])


@pytest.mark.parametrize("sizes", [[30000, 4000], [30000, 30000, 10000]])  # 1535 and 3006 groups, nearly all heavy
def test_many_heavy_groups(sizes):
    import torch
    pos = torch.cat([torch.from_numpy(W.uniform_cube(n, 400 + k)[0]) for k, n in enumerate(sizes)]).cuda()
    mass = torch.full((len(pos),), 1.0 / len(pos), device="cuda")
    r = torch.full((len(pos),), 0.33, device="cuda")
    off = np.concatenate([[0], np.cumsum(sizes)])
    print(f"[gpu] many heavy groups: {sizes}", flush=True)
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes))
    ctx.build_tree_batch(pos, mass, off)
    ctx.compute_multipoles()
    cnt, o, idx = ctx.neighbor_list(r)
    rho, dcnt = ctx.sph_density(r * 0.5)
    assert torch.equal(rho, ctx.sph_density(r * 0.5)[0]) and torch.equal(cnt, dcnt)
    for k, n in enumerate(sizes):
        s = slice(off[k], off[k + 1])
        one = gpu_context(n)
        one.build_tree(pos[s].contiguous(), mass[s].contiguous())
        one.compute_multipoles()
        c1, o1, i1 = one.neighbor_list(r[s].contiguous())
        assert torch.equal(cnt[s], c1)
        own = torch.repeat_interleave(torch.arange(n, device="cuda"), c1.long())
        a = idx[int(o[off[k]]):int(o[off[k + 1]])].long() - int(off[k])
        assert torch.equal(torch.sort(own * n + a)[0], torch.sort(own * n + i1.long())[0])
        assert float(((rho[s] - one.sph_density((r * 0.5)[s].contiguous())[0]).abs() / rho[s]).max()) <= 1e-5
