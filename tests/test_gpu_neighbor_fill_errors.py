"""mibh_neighbor_fill refuses a negative capacity and fills as much of a list as
fits without an error, as its header says.
"""
import pytest

from gpu_helpers import gpu_context
from paper_1204_2280_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 40000])
def test_capacity_of_a_fill(n):
    import torch
    from paper_1204_2280_amd import mibh
    pos, _, mass = W.plummer(n, 5, with_velocities=False)
    ctx = gpu_context(n)
    ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    ctx.compute_multipoles()
    r = torch.full((n,), 0.05, device="cuda")
    cnt, off, idx = ctx.neighbor_list(r)
    out = torch.full_like(idx, -7)

    def fill(capacity, index=out):
        return mibh.lib().mibh_neighbor_fill(ctx.handle, r.data_ptr(), cnt.data_ptr(), off.data_ptr(),
                                             None if index is None else index.data_ptr(), capacity)

    print(f"[gpu] neighbour fill: n={n} total={len(idx)}", flush=True)
    assert fill(-1) == -1 and b"capacity" in mibh.lib().mibh_last_error()
    assert fill(0, None) == 0
    ctx.sync()
    assert bool((out == -7).all())
    assert fill(len(idx) // 2) == 0
    ctx.sync()
    half = len(idx) // 2
    assert torch.equal(out[:half], idx[:half]) and bool((out[half:] == -7).all())
