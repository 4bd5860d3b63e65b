"""Bucket sort at the sizes where its buckets change: a sample that misses most
particles of a split system (buckets of several pieces) with 1024 elements per
bucket on average, and the first size with 1365, which also has the thinnest
sample.  The order is checked against a stable sort of the keys.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _sampled(n, nb):
    """The particles the sample draws from one system of n in nb buckets."""
    m = min(16 * nb, 8 * 4096)
    lists = -(-m // 4096)
    m = m // lists // 8 * 8 * lists
    j = np.arange(m, dtype=np.uint64)
    step = np.uint64((n << 32) // m)
    lo, hi = step * j >> np.uint64(32), step * (j + np.uint64(1)) >> np.uint64(32)
    v = j * np.uint64(0x9e3779b9) & np.uint64(0xffffffff)
    for shift, mul in ((16, 0x7feb352d), (15, 0x846ca68b), (16, 1)):
        v = ((v ^ (v >> np.uint64(shift))) * np.uint64(mul)) & np.uint64(0xffffffff)
    return (lo + (v * (hi - lo) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("kind,n", [("missed", 30001), ("missed", 300007), ("plummer", 1 << 21),
                                    ("plummer", (1 << 21) + 1)])
def test_order_is_the_stable_sort_of_the_keys(kind, n):
    import torch
    if kind == "missed":
        rng = np.random.default_rng(63)
        pos = rng.random((n, 3)).astype(np.float32)
        mass = rng.random(n).astype(np.float32)
        pos[:, 0] = 0.6 + 0.4 * pos[:, 0]
        pos[_sampled(n, -(-n // 1024)), 0] *= 0.1
    else:
        pos, _, mass = W.plummer(n, 64, with_velocities=False)
    print(f"[gpu] bucket sort sizes {kind} n={n}", flush=True)
    ctx = gpu_context(n)
    ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    ctx.sync()
    keys = ctx.export("keys").cpu().numpy().view(np.uint64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    spos = ctx.export("spos").cpu().numpy()
    assert np.array_equal(np.sort(perm), np.arange(n))
    assert np.all(keys[:-1] <= keys[1:])
    same = keys[:-1] == keys[1:]
    assert np.all(perm[:-1][same] < perm[1:][same])
    np.testing.assert_array_equal(spos[:, :3], pos[perm])
    np.testing.assert_array_equal(spos[:, 3], mass[perm])
    # the keys are those of the particles: Morton order of the cube's 2^20 grid
    lo, hi = pos.min(0).astype(np.float64), pos.max(0).astype(np.float64)
    q = np.minimum(np.floor((pos[perm].astype(np.float64) - lo) * 2.0 ** (20 - np.frexp((hi - lo).max())[1])), 2 ** 20 - 1)
    top = (q.astype(np.uint64) >> np.uint64(19)) & np.uint64(1)
    np.testing.assert_array_equal(keys >> np.uint64(57), top[:, 0] << np.uint64(2) | top[:, 1] << np.uint64(1) | top[:, 2])
