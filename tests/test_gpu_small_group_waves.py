"""The walk of groups smaller than 64 on both sides of each line between eight,
four, two and one waves per group, which lies at fewer particles the smaller the
groups are: systems walked alone against the same systems inside a batch large
enough for one wave, bit for bit.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _lines(cap):
    """The largest n of each number of waves."""
    return [m * (cap + 3) // 67 for m in (8192, 15360 + 272 * cap, 73728 + 768 * cap)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cap", [1, 8, 32])
def test_waves_on_both_sides_of_a_line(cap, precision):
    import torch
    assert _lines(64) == [8192, 32768, 122880]
    params = {"ncrit": min(cap, 16), "group_cap": cap, "precision": precision, "anchor_up": 0 if cap == 1 else 3}
    sizes = [k + d for k in _lines(cap) for d in (0, 1)] + [130000]
    parts = [W.plummer(k, 190 + j, with_velocities=False) for j, k in enumerate(sizes)]
    pos = torch.from_numpy(np.concatenate([p for p, _, _ in parts])).cuda()
    mass = torch.from_numpy(np.concatenate([m for _, _, m in parts])).cuda()
    off = np.concatenate([[0], np.cumsum(sizes)])
    ctx = gpu_context(int(off[-1]), max_systems=len(sizes), **params)
    acc, pot = ctx.forces_batch(pos, mass, off, 0.75)
    ctx.sync()
    for k, n in enumerate(sizes[:-1]):
        print(f"[gpu] small groups: n={n} {params}", flush=True)
        one = gpu_context(n, **params)
        s = slice(off[k], off[k + 1])
        a, p = one.forces(pos[s].contiguous(), mass[s].contiguous(), 0.75)
        one.sync()
        fits = one.stats()["anchor_fallbacks"] == 0 and ctx.stats()["anchor_fallbacks"] == 0
        if fits:  # an anchor without room leaves its groups to sums in another order
            assert torch.equal(a, acc[s]) and torch.equal(p, pot[s])
        else:
            assert float((a - acc[s]).norm(dim=1).div(acc[s].norm(dim=1)).quantile(0.99)) < 1e-5
