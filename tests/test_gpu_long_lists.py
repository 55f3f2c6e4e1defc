"""Lists too long for one workgroup's LDS, sorted in segments, against the order by (depth bits, id), bit for bit.

All records lie in one tile of their view; a second view that holds none gives the launch the tiles that admit
its capacity to the tile-by-tile sort (512 entries a tile on average).  Depths are distinct, tie often, are all
equal, or lie within a few steps of each other but for one far outlier, and then the segments' sort by
buckets gives way to merges and ranges of keys are halved.
"""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import saved_arrays

pytestmark = pytest.mark.gpu


def _records(rng, n, depths):
    r = np.zeros((n, 12), np.float32)
    r[:, 0:2] = rng.uniform(5, 11, (n, 2))
    r[:, 2] = r[:, 4] = 2.0
    r[:, 5] = 0.9
    r[:, 7] = r[:, 8] = 2.3
    z = {"distinct": lambda: rng.permutation(np.linspace(0.3, 900.0, n)),
         "tie": lambda: np.round(rng.uniform(0.5, 4.0, n) * 16) / 16,
         "equal": lambda: np.full(n, 2.5),
         "skew": lambda: np.where(np.arange(n) == n // 3, 1e30, 1 + 2.0 ** -20 * rng.integers(0, 40, n))}[depths]()
    r[:, 6] = z
    return r


@pytest.mark.parametrize("depths", ["distinct", "tie", "equal", "skew"])
@pytest.mark.parametrize("lengths", [(2048, 2049), (4095, 4097, 1), (5000, 8193), (20_000, 700, 2050), (100_000,),
                                     (327_680,), (327_681, 3000)])
def test_long_lists(lengths, depths):
    from paper_2510_26358_amd.rasterizer import Rasterizer, ViewSpec
    ras = Rasterizer(0)
    rng = np.random.default_rng(7300 + sum(lengths))
    base = np.concatenate([[0], np.cumsum(lengths)])
    n, k = int(base[-1]), len(lengths)
    recs = np.concatenate([_records(rng, m, depths) for m in lengths])
    side = 16 * int(np.ceil(np.sqrt(n / 512)) + 1)
    views = ViewSpec([16] * k + [side], [16] * k + [side], [*base[:-1], n], [*base[1:], n])
    zb = recs[:, 6].view(np.uint32)
    want = np.concatenate([base[b] + np.lexsort((np.arange(m), zb[base[b]:base[b] + m]))
                           for b, m in enumerate(lengths)]).astype(np.int64)
    tiles = k + (side // 16) ** 2
    assert n <= 512 * tiles
    for cap in (n, (1 << 22) + 1):  # tile by tile; by radix sorts
        print("lengths", lengths, "depths", depths, "capacity", cap, flush=True)
        buf = ras.buffers(views, n, 0, cap)
        buf.fwd_ws.fill_(0xA5)
        buf.saved.fill_(0xA5)
        for _ in range(2):
            ras.bin_records(views, n, torch.from_numpy(recs).cuda(), torch.ones(n, dtype=torch.uint8).cuda(), buf)
        torch.cuda.synchronize()
        sv = saved_arrays(buf, views)
        assert (sv["K"], sv["V"], sv["overflow"], sv["n_listed"]) == (n, n, 0, n)
        assert np.array_equal(sv["tile_pairs"], want)
        assert np.array_equal(sv["ranges"][:k], np.stack([base[:-1], base[1:]], 1)) and not sv["ranges"][k:].any()
        assert np.array_equal(sv["tile_keys"], np.repeat(np.arange(k), lengths))
        assert sorted(w for w in sv["work"] if w != 0xFFFFFFFF) == list(range(tiles))
