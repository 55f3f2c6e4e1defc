"""Tile lists sorted tile by tile and by radix sorts over all, bit for bit.

Records whose Gaussians lie in the one tile of their view make lists of chosen lengths: at the edges of
the sort's runs of 64, of its pieces of 1024 and of their merges, with depths that tie often, never, or
always.  A launch takes the tile-by-tile sort when its capacity is at most 2^22 and its lists are
bounded (by 4096 Gaussians a view, or 512 entries a tile on average), so the same records are binned
with the exact capacity and with the capacities on both sides of that line.
"""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import saved_arrays

pytestmark = pytest.mark.gpu


def _records(rng, n, depths):
    r = np.zeros((n, 12), np.float32)
    r[:, 0:2] = rng.uniform(4, 12, (n, 2))
    r[:, 2] = r[:, 4] = 0.5                      # sigma 1.4 pixels
    r[:, 5] = 0.9
    r[:, 7] = r[:, 8] = np.sqrt(2 * np.log(255 * 0.9) * 2)
    z = {"tie": np.round(rng.uniform(0.5, 4.0, n) * 16) / 16, "equal": np.full(n, 2.5),
         "distinct": rng.permutation(np.linspace(0.3, 900.0, n))}[depths]
    r[:, 6] = z
    return r


@pytest.mark.parametrize("depths", ["tie", "equal", "distinct"])
@pytest.mark.parametrize("lengths", [(1, 63, 64, 65, 0, 129, 700), (1023, 1024, 1025, 2), (2047, 2049), (3073, 4096),
                                     (4097, 3)])
def test_list_lengths_at_the_edges(lengths, depths):
    from paper_2510_26358_amd.rasterizer import Rasterizer, ViewSpec
    ras = Rasterizer(0)
    rng = np.random.default_rng(7000 + sum(lengths))
    base = np.concatenate([[0], np.cumsum([max(n, 1) for n in lengths])])
    recs = np.concatenate([_records(rng, max(n, 1), depths) for n in lengths])
    valid = np.concatenate([np.full(max(n, 1), n > 0) for n in lengths])
    views = ViewSpec([16] * len(lengths), [16] * len(lengths), base[:-1], base[1:])
    zb = recs[:, 6].view(np.uint32)
    want = np.concatenate([base[b] + np.lexsort((np.arange(n), zb[base[b]:base[b] + n]))
                           for b, n in enumerate(lengths)]).astype(np.int64)
    ends = np.cumsum(lengths)
    ranges = np.array([[e - n, e] if n else [0, 0] for n, e in zip(lengths, ends)])
    for cap in (sum(lengths), 1 << 22, (1 << 22) + 1):
        print("lengths", lengths, "depths", depths, "capacity", cap, flush=True)
        buf = ras.buffers(views, len(recs), 0, cap)
        buf.fwd_ws.fill_(0xA5)
        buf.saved.fill_(0xA5)
        ras.bin_records(views, len(recs), torch.from_numpy(recs).cuda(),
                        torch.from_numpy(valid.astype(np.uint8)).cuda(), buf)
        torch.cuda.synchronize()
        sv = saved_arrays(buf, views)
        assert (sv["K"], sv["V"], sv["overflow"], sv["n_listed"]) == (sum(lengths), sum(lengths), 0, sum(lengths))
        assert np.array_equal(sv["tile_pairs"], want)
        assert np.array_equal(sv["ranges"], ranges)
        assert np.array_equal(sv["tile_keys"], np.repeat(np.arange(len(lengths)), lengths))
        assert sorted(w for w in sv["work"] if w != 0xFFFFFFFF) == list(range(len(lengths)))


def test_overflow_is_flagged_and_stays_in_bounds():
    from paper_2510_26358_amd.rasterizer import Rasterizer, ViewSpec
    ras = Rasterizer(0)
    rng = np.random.default_rng(7100)
    n, cap = 3000, 1300
    recs = _records(rng, n, "tie")
    views = ViewSpec([16], [16], [0], [n])
    buf = ras.buffers(views, n, 0, cap)
    ras.bin_records(views, n, torch.from_numpy(recs).cuda(), torch.ones(n, dtype=torch.uint8).cuda(), buf)
    torch.cuda.synchronize()
    sv = saved_arrays(buf, views)
    assert (sv["K"], sv["V"], sv["overflow"], sv["K_kept"], sv["n_listed"]) == (n, n, 1, cap, cap)
    assert sv["tile_pairs"].min() >= 0 and sv["tile_pairs"].max() < n and len(set(sv["tile_pairs"])) == cap
