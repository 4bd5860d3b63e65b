"""Builds on both sides of the sizes up to which a kernel adds up the counts of the
one before itself: 64 blocks of the tree build (32768 particles), 64 tiles and
one bucket per thread of the bucket sort (a batch with more buckets), against
the oracle, bit for bit.
"""
import numpy as np
import pytest

from gpu_helpers import assert_multipoles_equal, assert_tree_equal, gpu_context, run_gpu
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 512, 513, 32768, 32769])
def test_build_blocks(orc, n):
    pos, _, mass = W.plummer(n, 77, with_velocities=False)
    print(f"[gpu] folded scans n={n}", flush=True)
    g = run_gpu(gpu_context(n), pos, mass, 0.75)
    T = orc.Tree(pos, mass)
    assert_tree_equal(g, T)
    assert_multipoles_equal(g, T, 0.75)


@pytest.mark.parametrize("small", [190, 200])  # 249 and 259 buckets, 256 threads
def test_batch_buckets(orc, small):
    import torch
    sizes = [20] * small + [60000]
    parts = [W.plummer(n, 300 + k, with_velocities=False) for k, n in enumerate(sizes)]
    pos, mass = np.concatenate([p for p, _, _ in parts]), np.concatenate([m for _, _, m in parts])
    off = np.concatenate([[0], np.cumsum(sizes)])
    print(f"[gpu] folded scans, batch of {len(sizes)}", flush=True)
    ctx = gpu_context(len(mass), max_systems=len(sizes))
    ctx.build_tree_batch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), off)
    ctx.sync()
    keys = ctx.export("keys").cpu().numpy().view(np.uint64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    for k in (0, 1, small // 2, small - 1, small):
        a, b = off[k], off[k + 1]
        T = orc.Tree(pos[a:b], mass[a:b])
        np.testing.assert_array_equal(keys[a:b], T.keys)
        np.testing.assert_array_equal(perm[a:b] - a, T.perm)
