"""The walk on both sides of each line between eight, four, two and one waves per
group: systems walked alone against the same systems inside a batch large enough
for one wave, bit for bit, in every accumulation mode and with short lists.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("params", [{}, {"precision": 1}, {"precision": 2, "anchor_up": 0},
                                    {"pc_cap": 128, "pp_cap": 128, "ncrit": 64}])
@pytest.mark.parametrize("n", [64, 8192, 32768, 122880])
def test_waves_on_both_sides_of_a_line(n, params):
    import torch
    sizes = [n, n + 1, 130000]
    parts = [W.plummer(k, 90 + j, with_velocities=False) for j, k in enumerate(sizes)]
    pos = torch.from_numpy(np.concatenate([p for p, _, _ in parts])).cuda()
    mass = torch.from_numpy(np.concatenate([m for _, _, m in parts])).cuda()
    off = np.concatenate([[0], np.cumsum(sizes)])
    print(f"[gpu] wave lines: n={n} {params}", flush=True)
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes), **params)
    acc, pot = ctx.forces_batch(pos, mass, off, 0.75)
    ctx.sync()
    for k in range(2):
        one = gpu_context(sizes[k], **params)
        s = slice(off[k], off[k + 1])
        a, p = one.forces(pos[s].contiguous(), mass[s].contiguous(), 0.75)
        one.sync()
        assert torch.equal(a, acc[s]) and torch.equal(p, pot[s])
