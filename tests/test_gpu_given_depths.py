"""Depths of given records that no projection writes: NaNs of any bits are ordered by those bits like
every other depth, and the one whose bits mark a pair without a depth (all ones) is listed nowhere,
whether the lists are sorted tile by tile or by radix sorts over all."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import saved_arrays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [70, 1100])
@pytest.mark.parametrize("rest", ["equal", "distinct"])  # equal depths leave the buckets for the merges
def test_nan_depths(n, rest):
    from paper_2510_26358_amd.rasterizer import Rasterizer, ViewSpec
    ras = Rasterizer(0)
    rng = np.random.default_rng(7200 + n)
    recs = np.zeros((n, 12), np.float32)
    recs[:, 0:2] = rng.uniform(4, 12, (n, 2))
    recs[:, 2] = recs[:, 4] = 0.5
    recs[:, 5] = 0.9
    recs[:, 7] = recs[:, 8] = np.sqrt(2 * np.log(255 * 0.9) * 2)
    zb = (np.full(n, 2.5, np.float32) if rest == "equal" else rng.permutation(np.linspace(0.3, 90.0, n, dtype=np.float32)))
    zb = zb.view(np.uint32).copy()
    odd = rng.permutation(n)[:12]
    zb[odd[:10]] = rng.permutation(np.arange(0xFFFFFFBD, 0xFFFFFFFF, dtype=np.uint32))[:10]
    zb[odd[10:]] = 0xFFFFFFFF
    recs.view(np.uint32)[:, 6] = zb
    views = ViewSpec([16], [16], [0], [n])
    want = np.lexsort((np.arange(n), zb))[:n - 2]
    for cap in (n, 1 << 22, (1 << 22) + 1):
        print("n", n, rest, "capacity", cap, flush=True)
        buf = ras.buffers(views, n, 0, cap)
        ras.bin_records(views, n, torch.from_numpy(recs).cuda(), torch.ones(n, dtype=torch.uint8).cuda(), buf)
        torch.cuda.synchronize()
        sv = saved_arrays(buf, views)
        assert (sv["K"], sv["V"], sv["overflow"], sv["n_listed"]) == (n - 2, n - 2, 0, n - 2)
        assert np.array_equal(sv["tile_pairs"], want)
        assert np.array_equal(sv["ranges"], [[0, n - 2]])
