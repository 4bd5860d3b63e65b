"""The bucket sort's words that agree in their key bits, against the oracle bit for
bit (keys, permutation, records, and the tree built from the shared digits): runs
of equal keys at the longest that one thread puts in order (8) and one more, of
keys that differ only in the bits a word leaves out, one-bucket and split systems,
one and two places per thread, and systems of a batch.
"""
import numpy as np
import pytest

from gpu_helpers import assert_tree_equal, gpu_context, run_gpu

pytestmark = pytest.mark.gpu


def _input(kind, n):
    rng = np.random.default_rng(81)
    if kind == "near":  # 50 particles within a few of the grid's cells at each of n / 50 points
        pos = rng.random((-(-n // 50), 3)).repeat(50, axis=0)[:n] + rng.integers(0, 4, (n, 3)) * 2.0 ** -20
        pos[0] = 0.0  # the cube's corner and extent whatever the others are
        pos[-1] = 0.999
    elif kind == "mixed":  # runs of 1 .. 12 keys
        pos = rng.random((n, 3))[np.sort(rng.integers(0, n // 3, n))]
    else:
        k = int(kind)
        pos = rng.random((-(-n // k), 3)).repeat(k, axis=0)[:n]
    pos = pos[rng.permutation(n)].astype(np.float32)
    return pos, rng.random(n).astype(np.float32)


@pytest.mark.parametrize("n", [60, 2048, 4096, 4097, 50001, 300001])
@pytest.mark.parametrize("kind", ["2", "8", "9", "30", "near", "mixed"])
def test_runs_match_oracle(orc, kind, n):
    pos, mass = _input(kind, n)
    print(f"[gpu] bucket runs {kind} n={n}", flush=True)
    g = run_gpu(gpu_context(n), pos, mass, 0.9, exports=("keys", "perm", "cells", "groups", "spos"))
    T = orc.Tree(pos, mass)
    assert_tree_equal(g, T)
    np.testing.assert_array_equal(g["spos"][:, :3], pos[T.perm])
    np.testing.assert_array_equal(g["spos"][:, 3], mass[T.perm])


@pytest.mark.parametrize("sizes", [[3000, 4096, 17, 900], [3000, 20000, 5, 4097]])
def test_runs_in_a_batch(orc, sizes):
    import torch
    parts = [_input(kind, n) for kind, n in zip(("30", "near", "2", "9"), sizes)]
    pos, mass = np.concatenate([p for p, _ in parts]), np.concatenate([m for _, m in parts])
    off = np.concatenate([[0], np.cumsum(sizes)])
    print(f"[gpu] bucket runs, batch {sizes}", flush=True)
    ctx = gpu_context(len(mass), max_systems=len(sizes))
    ctx.build_tree_batch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), off)
    ctx.sync()
    keys = ctx.export("keys").cpu().numpy().view(np.uint64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    for k, (p, m) in enumerate(parts):
        T = orc.Tree(p, m)
        s = slice(off[k], off[k + 1])
        np.testing.assert_array_equal(keys[s], T.keys)
        np.testing.assert_array_equal(perm[s] - off[k], T.perm)
