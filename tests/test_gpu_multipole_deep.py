"""Multipole moments against the oracle, bit for bit, where a chunk holds more
internal cells than its list (small ncrit; chains of cells with one child above
points that coincide, and with two along a line) and at the sizes where the chunks
change: 1024, 2048, 32768 and 2^19 particles, by ncrit.
"""
import numpy as np
import pytest

from gpu_helpers import assert_multipoles_equal, assert_tree_equal, gpu_context, run_gpu
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _input(kind, n):
    rng = np.random.default_rng(71)
    if kind.startswith("dup"):  # several particles at each point, spread over the input
        k = int(kind[3:])
        pos = rng.random((-(-n // k), 3)).astype(np.float32).repeat(k, axis=0)[:n][rng.permutation(n)]
    elif kind == "line":
        pos = np.full((n, 3), 0.5, np.float32)
        pos[:, 0] = rng.random(n)
    elif kind == "massless":  # chains of massless cells take their centres
        pos = rng.random((-(-n // 24), 3)).astype(np.float32).repeat(24, axis=0)[:n]
        mass = rng.random(n).astype(np.float32)
        mass[(np.arange(n) // 24) % 2 == 0] = 0.0
        return pos, mass
    else:
        return W.plummer(n, 52, with_velocities=False)[::2]
    return pos, rng.random(n).astype(np.float32)


@pytest.mark.parametrize("kind,n,ncrit,gcap", [
    ("plummer", 1024, 2, 64), ("plummer", 1025, 2, 64), ("plummer", 1500, 3, 64), ("plummer", 2048, 1, 1),
    ("plummer", 2049, 7, 64), ("plummer", 2049, 8, 64), ("plummer", 32768, 4, 64), ("plummer", 32769, 4, 64),
    ("plummer", 32768, 16, 64), ("plummer", 32769, 16, 64), ("plummer", 70001, 2, 16), ("plummer", 1 << 19, 2, 64),
    ("plummer", (1 << 19) + 1, 1, 64), ("dup24", 3000, 16, 64), ("dup24", 50003, 16, 64), ("dup8", 1700, 4, 16),
    ("dup8", 20000, 4, 64), ("dup8", 140000, 4, 64), ("dup40", 9000, 16, 64), ("dup2", 6000, 1, 1),
    ("line", 5000, 1, 8), ("line", 140000, 1, 64), ("massless", 3000, 16, 64), ("massless", 100003, 4, 64)])
def test_moments_of_deep_trees(orc, kind, n, ncrit, gcap):
    pos, mass = _input(kind, n)
    print(f"[gpu] deep multipoles {kind} n={n} ncrit={ncrit}", flush=True)
    g = run_gpu(gpu_context(n, ncrit=ncrit, group_cap=gcap), pos, mass, 0.75)
    T = orc.Tree(pos, mass, ncrit, gcap)
    assert_tree_equal(g, T)
    assert_multipoles_equal(g, T, 0.75)


def test_many_systems(orc):
    """Cells of the last of 256 systems, listed and gathered again."""
    import torch
    from paper_1204_2280_amd.mibh import Decoded
    parts = [_input("plummer", 20 + k % 50) for k in range(253)] + [_input("dup24", 4000), _input("plummer", 3000),
                                                                    _input("massless", 2500)]
    off = np.concatenate([[0], np.cumsum([len(m) for _, m in parts])])
    ctx = gpu_context(int(off[-1]), max_systems=256)
    print("[gpu] deep multipoles, 256 systems", flush=True)
    ctx.build_tree_batch(torch.from_numpy(np.concatenate([p for p, _ in parts])).cuda(),
                         torch.from_numpy(np.concatenate([m for _, m in parts])).cuda(), off)
    ctx.compute_multipoles()
    cells = Decoded.cells(ctx.export("cells"))
    mp = ctx.export("multipoles").cpu().numpy()
    delta = ctx.export("delta").cpu().numpy()
    for k in (0, 100, 253, 254, 255):
        T = orc.Tree(*parts[k])
        own = cells["system"] == k
        np.testing.assert_array_equal(cells["first"][own] - off[k], T.cells()["first"])
        ref = T.multipoles()
        np.testing.assert_array_equal(mp[own, 0], ref["M"])
        np.testing.assert_array_equal(mp[own, 1:4], ref["com"])
        np.testing.assert_array_equal(mp[own, 4:], ref["S"])
        np.testing.assert_array_equal(delta[own], ref["delta"])
