"""Multipole moments at the edges of the pass' particle ranges (chunks of 2048
particles, 64 chunks per merge) against the oracle, bit for bit: one chunk and
one particle more or less, one and two merges, more internal cells per chunk
than its list holds (ncrit 1), leaves larger than a chunk (coincident points).
"""
import numpy as np
import pytest

from gpu_helpers import assert_multipoles_equal, assert_tree_equal, gpu_context, run_gpu
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


def _input(kind, n):
    if kind == "clump":  # a run of identical keys across chunk edges, among other particles
        rng = np.random.default_rng(51)
        pos = rng.random((n, 3)).astype(np.float32)
        pos[n // 5:n // 5 + n // 2] = pos[0]
        return pos, np.full(n, 1.0 / n, np.float32)
    pos, _, mass = W.plummer(n, 52, with_velocities=False)
    return pos, mass


@pytest.mark.parametrize("kind,n,ncrit,gcap", [
    ("plummer", 2047, 16, 64), ("plummer", 2048, 16, 64), ("plummer", 2049, 16, 64), ("plummer", 4097, 1, 1),
    ("plummer", 12001, 2, 8), ("clump", 9001, 16, 64), ("plummer", 131072, 16, 64), ("plummer", 131073, 16, 64),
    ("plummer", 300001, 4, 16)])
def test_moments_at_range_edges(orc, kind, n, ncrit, gcap):
    pos, mass = _input(kind, n)
    print(f"[gpu] multipole chunks {kind} n={n} ncrit={ncrit}", flush=True)
    g = run_gpu(gpu_context(n, ncrit=ncrit, group_cap=gcap), pos, mass, 0.75)
    T = orc.Tree(pos, mass, ncrit, gcap)
    assert_tree_equal(g, T)
    assert_multipoles_equal(g, T, 0.75)
