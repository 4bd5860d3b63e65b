"""Trees on both sides of the size from which the ends of large cells are searched by
quarters instead of eighths (2^19 particles), against the oracle: cells that end
anywhere from the next wave to the end of the input, one run over most of it, and
the ends of systems.
"""
import numpy as np
import pytest

from gpu_helpers import assert_tree_equal, gpu_context
from paper_1204_2280_amd.mibh import Decoded

pytestmark = pytest.mark.gpu


def _input(kind, n):
    rng = np.random.default_rng(91)
    pos = rng.random((n, 3)).astype(np.float32)
    if kind == "clump":  # most of the particles at one point
        pos[rng.random(n) < 0.9] = np.float32(0.3)
    elif kind == "line":
        pos[:, 1:] = 0.5
    elif kind == "corner":  # all but a few in the last octant of the last octants
        pos = (1.0 - 1e-3 * pos).astype(np.float32)
        pos[:7] = 0.0
    return pos, rng.random(n).astype(np.float32)


@pytest.mark.parametrize("kind", ["cube", "clump", "line", "corner"])
@pytest.mark.parametrize("n", [1 << 19, (1 << 19) + 1, 777777])
def test_ends_match_oracle(orc, kind, n):
    import torch
    pos, mass = _input(kind, n)
    print(f"[gpu] cell ends {kind} n={n}", flush=True)
    ctx = gpu_context(n)
    ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    ctx.sync()
    g = {"keys": ctx.export("keys").cpu().numpy().view(np.uint64),
         "perm": ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64),
         "cells": Decoded.cells(ctx.export("cells")), "groups": Decoded.groups(ctx.export("groups"))}
    assert_tree_equal(g, orc.Tree(pos, mass))


def test_ends_of_systems(orc):
    import torch
    sizes = [5, 300000, 1, 64, 250000, 3]
    parts = [_input(("cube", "clump", "line")[k % 3], n) for k, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] > 1 << 19
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes))
    print("[gpu] cell ends, batch", flush=True)
    ctx.build_tree_batch(torch.from_numpy(np.concatenate([p for p, _ in parts])).cuda(),
                         torch.from_numpy(np.concatenate([m for _, m in parts])).cuda(), off)
    ctx.sync()
    cells = Decoded.cells(ctx.export("cells"))
    for k, (p, m) in enumerate(parts):
        ref, own = orc.Tree(p, m).cells(), cells["system"] == k
        np.testing.assert_array_equal(cells["first"][own] - off[k], ref["first"])
        for f in ("count", "level", "nchild"):
            np.testing.assert_array_equal(cells[f][own], ref[f])
