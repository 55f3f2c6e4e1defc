"""The two compactions whose workgroups go to the XCDs in strips of consecutive blocks.

Every block of 256 rows has to be moved once whatever the number of blocks leaves of the last strip and of
the last group of eight strips: the lifecycle scatter (strips of 4 blocks: a strip ends at 1024 rows, a
group at 8192) against the oracle, and the voxel map's rebuild (strips of 16 without offloads, of 4 with)
by the rows it must keep bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import lifecycle as olc
from tests.test_gpu_lifecycle import _compare_lifecycle, _lifecycle_inputs, _run_lifecycle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ras():
    from paper_2510_26358_amd.rasterizer import Rasterizer
    return Rasterizer(0)


@pytest.mark.parametrize("n", [1, 256, 257, 1024, 1025, 8191, 8192, 8193])
def test_lifecycle_scatter_at_the_ends_of_strips(ras, n):
    lp = olc.LifecycleParams(do_reset=True)
    print("n", n, flush=True)
    params, m, v, accum, count, noise = _lifecycle_inputs(900 + n, n, 0, lp)
    ref = olc.apply({k: a.astype(np.float64) for k, a in params.items()}, m, v, accum, count,
                    noise.astype(np.float64), lp)
    _compare_lifecycle(_run_lifecycle(ras, params, m, v, accum, count, noise, lp, 0), ref, params)


def _columns(gm):
    """(rows of parameters and moments, n) of the resident set."""
    return torch.cat([t.reshape(-1, gm.n) for s in (gm.params, gm.m, gm.v) for t in s.tensors()])


@pytest.mark.parametrize("offload", [False, True])
@pytest.mark.parametrize("n_old,n_new", [(255, 1), (4095, 1), (4096, 1), (1023, 2), (32767, 1), (32768, 1),
                                         (30000, 2770)])
def test_map_rebuild_at_the_ends_of_strips(ras, n_old, n_new, offload):
    from paper_2510_26358_amd.voxel_map import VoxelMap
    n = n_old + n_new
    n_out = n_new if offload else 0  # a full map gives its oldest rows for the new ones
    print("rows", n_old, n_new, "offloaded", n_out, flush=True)
    gm = VoxelMap(ras, voxel=1.0, sh_degree=1, tau=n - n_out, max_ids=1 << 17, max_points=1 << 16, s_init=0.01,
                  o_init=0.2)
    try:
        pts = torch.zeros(n, 3, device="cuda")
        pts[:, 0] = torch.arange(n, device="cuda") + 0.5  # one voxel each
        cols = torch.rand(n, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
        first = max(n_out, 1)
        gm.insert(pts[:first], cols[:first], 0)
        if first < n_old:
            gm.insert(pts[first:n_old], cols[first:n_old], 1)
        assert gm.n == n_old
        for s in (gm.params, gm.m, gm.v):
            for t in s.tensors():
                t.copy_(torch.rand(t.shape, device="cuda"))
        before = _columns(gm).clone()
        gm.insert(pts[n_old:], cols[n_old:], 2)
        torch.cuda.synchronize()
        assert gm.n == n - n_out
        after = _columns(gm)
        assert torch.equal(after[:, :n_old - n_out], before[:, n_out:])
        assert torch.equal(after[:3, n_old - n_out:].t(), pts[n_old:])
    finally:
        gm.close()
