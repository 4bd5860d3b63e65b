"""The bucket sort at its edges against the oracle, bit for bit (keys,
permutation, moved particles, and the tree built from the shared digits): one
bucket and one particle more (4096, 4097), partial tiles, few and many buckets,
long runs of equal keys across buckets, everything at one point, input already
sorted or reversed, a bucket that the sample misses (sorted in pieces), batches of one-bucket and split systems, and the radix
sort's first size beyond it.
"""
import numpy as np
import pytest

from gpu_helpers import assert_tree_equal, gpu_context, run_gpu
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _input(kind, n):
    if kind == "plummer":
        pos, _, mass = W.plummer(n, 61, with_velocities=False)
        return pos, mass
    rng = np.random.default_rng(62)
    pos = rng.random((n, 3)).astype(np.float32)
    if kind == "clump":  # half of the particles at one point, spread over the input
        pos[1::2] = np.float32(0.37)
    elif kind == "point":
        pos[:] = np.float32(0.25)
    elif kind == "dense":  # a dense clump and one particle far away: few distinct leading digits
        pos = (1e-4 * pos).astype(np.float32)
        pos[n // 2] = 1.0
    elif kind == "missed":  # the particles the sample draws come first, so one bucket holds all the others
        nb = -(-n // 1365)
        m = min(8192, 8 * nb)
        j = np.arange(m, dtype=np.uint64)
        step = (n << 32) // m
        lo, hi = step * j >> np.uint64(32), step * (j + np.uint64(1)) >> np.uint64(32)
        v = j * 0x9e3779b9 & 0xffffffff
        for shift, mul in ((16, 0x7feb352d), (15, 0x846ca68b), (16, 1)):
            v = ((v ^ (v >> np.uint64(shift))) * mul) & 0xffffffff
        drawn = lo + (v * (hi - lo) >> np.uint64(32))
        pos[:, 0] = 0.6 + 0.4 * pos[:, 0]
        pos[drawn.astype(np.int64), 0] *= 0.1
    elif kind in ("sorted", "reversed"):
        pos = pos[np.argsort(pos[:, 0], kind="stable")]
        pos[:, 1:] = 0.5
        pos = pos[::-1].copy() if kind == "reversed" else pos
    return pos, rng.random(n).astype(np.float32)


@pytest.mark.parametrize("kind,n", [
    ("plummer", 7), ("plummer", 17), ("plummer", 2048), ("plummer", 2049), ("plummer", 4096), ("plummer", 4097),
    ("plummer", 70001), ("clump", 5000), ("clump", 60001), ("point", 20000), ("dense", 50000), ("sorted", 30000),
    ("reversed", 30001), ("missed", 30001), ("plummer", (1 << 19) + 1)])
def test_sorted_order_matches_oracle(orc, kind, n):
    pos, mass = _input(kind, n)
    print(f"[gpu] bucket sort {kind} n={n}", flush=True)
    g = run_gpu(gpu_context(n), pos, mass, 0.9, exports=("keys", "perm", "cells", "groups", "spos"))
    T = orc.Tree(pos, mass)
    assert_tree_equal(g, T)
    np.testing.assert_array_equal(g["spos"][:, :3], pos[T.perm])
    np.testing.assert_array_equal(g["spos"][:, 3], mass[T.perm])


@pytest.mark.parametrize("sizes", [[1, 4096, 3, 900], [4097, 1, 20000, 4096, 2, 60001], [50] * 200 + [9000]])
def test_batches_match_single_systems(orc, sizes):
    import torch
    parts = [_input("clump" if k % 3 == 1 else "plummer", n) for k, n in enumerate(sizes)]
    pos, mass = np.concatenate([p for p, _ in parts]), np.concatenate([m for _, m in parts])
    off = np.concatenate([[0], np.cumsum(sizes)])
    print(f"[gpu] bucket sort, batch of {len(sizes)}", flush=True)
    ctx = gpu_context(len(mass), max_systems=len(sizes))
    ctx.forces_batch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), off, 0.9)
    ctx.sync()
    keys = ctx.export("keys").cpu().numpy().view(np.uint64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    spos = ctx.export("spos").cpu().numpy()
    ncells = 0
    for k, (p, m) in enumerate(parts):
        T = orc.Tree(p, m)
        s = slice(off[k], off[k + 1])
        np.testing.assert_array_equal(keys[s], T.keys)
        np.testing.assert_array_equal(perm[s] - off[k], T.perm)
        np.testing.assert_array_equal(spos[s, :3], p[T.perm])
        ncells += T.ncells
    assert ctx.stats()["ncells"] == ncells


@pytest.mark.parametrize("n", [5_591_040, 5_600_000])
def test_last_bucket_sort_and_first_radix_sort(orc, n):
    """5591040 particles take all 4096 buckets, 5600000 more than there are: the radix sort.  One
    system and two."""
    import torch
    pos, mass = _input("plummer", n)
    print(f"[gpu] large sort n={n}", flush=True)
    ctx = gpu_context(n, max_systems=2)
    P, M = torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda()
    for off in ([0, n], [0, 700001, n]):
        ctx.build_tree_batch(P, M, off)
        ctx.sync()
        keys = ctx.export("keys").cpu().numpy().view(np.uint64)
        perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
        for a, b in zip(off[:-1], off[1:]):
            assert np.array_equal(np.sort(perm[a:b]), np.arange(a, b))
            k = keys[a:b]
            assert np.all((k[1:] > k[:-1]) | ((k[1:] == k[:-1]) & (perm[a + 1:b] > perm[a:b - 1])))
        if len(off) == 2:
            T = orc.Tree(pos, mass)
            np.testing.assert_array_equal(keys, T.keys)
            np.testing.assert_array_equal(perm, T.perm)
