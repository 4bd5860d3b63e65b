"""The walk with one, two and four waves per group gives the same bits: systems
walked alone (4 waves per group up to 32768 particles of the tree, 2 up to
160000) against the same systems inside a batch too large for more than one, in
every accumulation mode, with and without shared anchor lists, and with lists
that are flushed during the traversal.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("params", [{}, {"precision": 1}, {"precision": 2}, {"anchor_up": 0},
                                    {"pc_cap": 128, "pp_cap": 128}, {"walk_waves": 24}])
def test_waves_per_group_do_not_change_the_bits(params):
    import torch
    sizes = [1, 70, 3000, 20000, 40000, 110000]
    parts = [W.plummer(n, 80 + k, with_velocities=False) for k, n in enumerate(sizes)]
    pos = torch.from_numpy(np.concatenate([p for p, _, _ in parts])).cuda()
    mass = torch.from_numpy(np.concatenate([m for _, _, m in parts])).cuda()
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] > 160000
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes), **params)
    acc, pot = ctx.forces_batch(pos, mass, off, 0.75)
    ctx.sync()
    for k, n in enumerate(sizes):
        print(f"[gpu] waves per group: n={n} {params}", flush=True)
        one = gpu_context(n, **params)
        s = slice(off[k], off[k + 1])
        a, p = one.forces(pos[s].contiguous(), mass[s].contiguous(), 0.75)
        one.sync()
        assert torch.equal(a, acc[s]) and torch.equal(p, pot[s])
