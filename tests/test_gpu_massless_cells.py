"""Moments of cells without mass (their centre stands for their centre of mass)
among cells with mass, in leaves, in a chunk's internal cells and in cells that
span chunks, against the oracle, bit for bit.
"""
import numpy as np
import pytest

from gpu_helpers import assert_multipoles_equal, assert_tree_equal, gpu_context, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ncrit", [(300, 16), (9001, 16), (9001, 1), (140001, 16)])
@pytest.mark.parametrize("kind", ["octants", "scattered", "one", "none"])
def test_moments_of_massless_cells(orc, n, ncrit, kind):
    rng = np.random.default_rng(n + ncrit)
    pos = rng.random((n, 3)).astype(np.float32)
    mass = rng.random(n).astype(np.float32)
    zero = {"octants": (pos[:, 0] < 0.5) ^ (pos[:, 1] < 0.5), "scattered": rng.random(n) < 0.9,
            "one": np.arange(n) != n // 2, "none": np.ones(n, bool)}[kind]
    mass[zero] = 0.0
    print(f"[gpu] massless cells {kind} n={n} ncrit={ncrit}", flush=True)
    g = run_gpu(gpu_context(n, ncrit=ncrit), pos, mass, 0.75)
    T = orc.Tree(pos, mass, ncrit, 64)
    assert_tree_equal(g, T)
    assert_multipoles_equal(g, T, 0.75)
