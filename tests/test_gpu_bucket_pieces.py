"""Buckets of the sort that the sample makes too large for one piece, against the
oracle bit for bit: keys, permutation, moved particles, and cells and groups, which
are built from the shared digits that the sort leaves.  The particles that the
sample draws come first along the Morton curve, so one bucket holds all the others;
the model of the sample here has to say so, for one system and for two of a batch.
"""
import numpy as np
import pytest

from gpu_helpers import assert_tree_equal, gpu_context, run_gpu
from test_gpu_bucket_sort_sizes import _sampled

SORT_BUCKET, MEAN = 4096, 1024  # elements a workgroup sorts at once; per bucket on average


def _mix32(v):
    for shift, mul in ((16, 0x7feb352d), (15, 0x846ca68b), (16, 1)):
        v = ((v ^ (v >> np.uint64(shift))) * np.uint64(mul)) & np.uint64(0xffffffff)
    return v


def _drawn(n, system):
    """The particles the sample draws from system `system` of n."""
    m = 16 * -(-n // MEAN)
    assert m <= SORT_BUCKET  # one list
    m = m // 8 * 8
    j = np.arange(m, dtype=np.uint64)
    step = np.uint64((n << 32) // m)
    lo, hi = step * j >> np.uint64(32), step * (j + np.uint64(1)) >> np.uint64(32)
    v = _mix32((j * np.uint64(0x9e3779b9) + np.uint64(system)) & np.uint64(0xffffffff))
    return (lo + (v * (hi - lo) >> np.uint64(32))).astype(np.int64)


def _missed(n, system, equal_keys):
    rng = np.random.default_rng(90 + system)
    pos = rng.random((n, 3)).astype(np.float32)
    if equal_keys:  # runs of 40 equal keys, spread over the input
        pos = pos[rng.integers(0, n // 40, n)]
    d = _drawn(n, system)
    pos[:, 0] = 0.6 + 0.4 * pos[:, 0]
    pos[d, 0] *= 0.1
    nb, m = -(-n // MEAN), len(d)
    # bucket r starts at the sample of rank m r / nb: the last one has everything that was not drawn
    assert n - m + m // nb > 6 * SORT_BUCKET and pos[d, 0].max() < pos[np.setdiff1d(np.arange(n), d), 0].min()
    return pos, rng.random(n).astype(np.float32)


def test_the_sample_misses_the_particles():
    np.testing.assert_array_equal(np.sort(_drawn(30001, 0)), np.sort(_sampled(30001, -(-30001 // MEAN))))
    for equal in (False, True):
        _missed(30001, 0, equal)


@pytest.mark.gpu
@pytest.mark.parametrize("n,equal_keys", [(30001, False), (30001, True), (45056, False)])
def test_bucket_of_several_pieces(orc, n, equal_keys):
    pos, mass = _missed(n, 0, equal_keys)
    print(f"[gpu] bucket pieces: n={n} equal_keys={equal_keys}", flush=True)
    g = run_gpu(gpu_context(n), pos, mass, 0.9, exports=("keys", "perm", "cells", "groups", "spos"))
    T = orc.Tree(pos, mass)
    assert_tree_equal(g, T)
    np.testing.assert_array_equal(g["spos"][:, :3], pos[T.perm])
    np.testing.assert_array_equal(g["spos"][:, 3], mass[T.perm])


@pytest.mark.gpu
def test_bucket_of_several_pieces_in_a_batch(orc):
    import torch
    from paper_1204_2280_amd.mibh import Decoded
    sizes = [30001, 31000]
    parts = [_missed(n, k, k == 1) for k, n in enumerate(sizes)]
    pos, mass = np.concatenate([p for p, _ in parts]), np.concatenate([m for _, m in parts])
    off = np.concatenate([[0], np.cumsum(sizes)])
    print("[gpu] bucket pieces: batch", flush=True)
    ctx = gpu_context(len(mass), max_systems=2)
    ctx.build_tree_batch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), off)
    ctx.sync()
    keys = ctx.export("keys").cpu().numpy().view(np.uint64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    cells = Decoded.cells(ctx.export("cells"))
    groups = Decoded.groups(ctx.export("groups"))
    for k, (p, m) in enumerate(parts):
        T = orc.Tree(p, m)
        s = slice(off[k], off[k + 1])
        np.testing.assert_array_equal(keys[s], T.keys)
        np.testing.assert_array_equal(perm[s] - off[k], T.perm)
        for ours, theirs in ((cells, T.cells()), (groups, T.groups())):
            own = ours["system"] == k
            for f in ("count", "level"):
                np.testing.assert_array_equal(ours[f][own], theirs[f])
            np.testing.assert_array_equal(ours["first"][own] - off[k], theirs["first"])
