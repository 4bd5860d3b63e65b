"""The queue of an active walk: the groups that hold an active particle, then the
others, both in Morton order, against the groups and the permutation exported
from the same tree; with masks of none, the first, the last, a few and all of the
particles, and fewer and more groups than one workgroup handles at a time.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 70, 20000, 300007])
@pytest.mark.parametrize("pick", ["none", "first", "last", "few", "most", "all"])
def test_active_queue_is_visited_groups_first(n, pick):
    import torch
    pos, _, mass = W.plummer(n, 61, with_velocities=False)
    frac = np.random.default_rng(n).random(n)
    active = {"none": frac < 0, "first": np.arange(n) == 0, "last": np.arange(n) == n - 1,
              "few": frac < 0.01, "most": frac < 0.9, "all": frac >= 0}[pick]
    print(f"[gpu] active queue: n={n} {pick}", flush=True)
    ctx = gpu_context(n)
    P, M = torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda()
    full, fpot = ctx.forces(P, M, 0.75)
    acc = torch.full((n, 3), 7.0, device="cuda")
    pot = torch.full((n,), 7.0, device="cuda")
    ctx.compute_forces_active(0.75, torch.from_numpy(active.astype(np.uint8)).cuda(), acc, pot)
    ctx.sync()
    groups = ctx.export("groups").cpu().numpy().view(np.uint32).astype(np.int64)
    perm = ctx.export("perm").cpu().numpy().view(np.uint32).astype(np.int64)
    first, count = groups[:, 0], groups[:, 1] & 255
    before = np.concatenate([[0], np.cumsum(active[perm])])
    has = before[first + count] > before[first]
    want = np.concatenate([np.flatnonzero(has), np.flatnonzero(~has)])
    np.testing.assert_array_equal(ctx.export("queue").cpu().numpy().astype(np.int64), want)
    on = torch.from_numpy(active).cuda()
    assert torch.equal(acc[on], full[on]) and torch.equal(pot[on], fpot[on])
    assert bool((acc[~on] == 7.0).all()) and bool((pot[~on] == 7.0).all())
