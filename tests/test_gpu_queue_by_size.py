"""A large tree's walk takes the end of each queue by the groups' particle counts:
every group exactly once (the outputs start as NaN) and the same bits as in the
order of the previous walk's work, at the shortest sorted queue, where windows
cover whole eighths and where they do not, with one system and with many, for
full and for active walks.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _inputs(kind):
    import torch
    if kind == "plummers":
        sizes = [60000, 1, 300, 90000, 4096, 70]
        parts = [W.plummer(n, 40 + k, with_velocities=False) for k, n in enumerate(sizes)]
        pos, mass = np.concatenate([p for p, _, _ in parts]), np.concatenate([m for _, _, m in parts])
        off = np.concatenate([[0], np.cumsum(sizes)])
    else:
        name, n = kind
        pos, mass = {"plummer": lambda: W.plummer(n, 9, with_velocities=False)[::2],
                     "hernquist": lambda: W.hernquist(n, 9), "cube": lambda: W.uniform_cube(n, 9)}[name]()
        off = np.array([0, n])
    return torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), off


@pytest.mark.parametrize("share", [None, 0.5, 0.03])
@pytest.mark.parametrize("kind", [("plummer", 65537), ("cube", 65537), ("cube", 70001), ("hernquist", 140000),
                                  ("plummer", 1500000), "plummers"])
def test_queue_by_size_visits_every_group_once(kind, share):
    import torch
    pos, mass, off = _inputs(kind)
    n = int(off[-1])
    ctx = gpu_context(n, max_systems=len(off) - 1)
    acc = torch.full((n, 3), float("nan"), device="cuda")
    pot = torch.full((n,), float("nan"), device="cuda")
    print(f"[gpu] queue by size: {kind} share={share}", flush=True)
    ctx.forces_batch(pos, mass, off, 0.75, acc, pot)
    ctx.sync()
    assert not bool(torch.isnan(acc).any()) and not bool(torch.isnan(pot).any())
    counts = ctx.export("counts").clone()
    if share is None:
        ctx.set_queue_order(2)  # by the work of the walk above
        acc2, pot2 = torch.full_like(acc, float("nan")), torch.full_like(pot, float("nan"))
        ctx.compute_forces(0.75, acc2, pot2)
        ctx.sync()
        assert torch.equal(acc, acc2) and torch.equal(pot, pot2)
    else:
        on = torch.rand(n, generator=torch.Generator().manual_seed(n)).cuda() < share
        acc2, pot2 = torch.full_like(acc, float("nan")), torch.full_like(pot, float("nan"))
        ctx.compute_forces_active(0.75, on.to(torch.uint8), acc2, pot2)
        ctx.sync()
        assert torch.equal(acc[on], acc2[on]) and torch.equal(pot[on], pot2[on])
        assert bool(torch.isnan(acc2[~on]).all()) and bool(torch.isnan(pot2[~on]).all())
    assert torch.equal(counts, ctx.export("counts"))
