"""The per-tile sort's lists at and beyond the most tiles and pairs that are admitted to it, against the order by
(tile, depth bits, id): few pairs in many tiles (whose counts are cleared by more workgroups than the
pairs have), and many pairs of which few are valid."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import saved_arrays

pytestmark = pytest.mark.gpu


def _check(views, recs, valid, n_gauss, cap):
    """recs: [pairs] records, each inside one tile (a 16-pixel one)."""
    from paper_2510_26358_amd.rasterizer import Rasterizer
    ras = Rasterizer(0)
    print("tiles", [((w + 15) // 16) * ((h + 15) // 16) for w, h in zip(views.widths, views.heights)], "pairs",
          len(recs), "capacity", cap, flush=True)
    buf = ras.buffers(views, n_gauss, 0, cap)
    buf.fwd_ws.fill_(0xA5)
    ras.bin_records(views, n_gauss, recs, valid, buf)
    torch.cuda.synchronize()
    on = torch.nonzero(valid)[:, 0].cpu().numpy()
    r = recs[torch.from_numpy(on).cuda()].cpu().numpy()
    starts = np.cumsum([0] + [e - b for b, e in zip(views.g_begin, views.g_end)])
    v = np.searchsorted(starts, on, side="right") - 1
    ntx = np.array([(w + 15) // 16 for w in views.widths])
    first = np.cumsum([0] + [((w + 15) // 16) * ((h + 15) // 16) for w, h in zip(views.widths, views.heights)])
    tile = first[v] + (r[:, 1] // 16).astype(np.int64) * ntx[v] + (r[:, 0] // 16).astype(np.int64)
    order = np.lexsort((on, r[:, 6].view(np.uint32), tile))
    sv = saved_arrays(buf, views)
    assert (sv["K"], sv["V"], sv["overflow"], sv["n_listed"]) == (len(on), len(on), 0, len(on))
    assert np.array_equal(sv["tile_pairs"], on[order])
    assert np.array_equal(sv["tile_keys"], tile[order])
    n = np.bincount(tile, minlength=first[-1])
    ends = np.cumsum(n)
    assert np.array_equal(sv["ranges"], np.where(n[:, None] > 0, np.stack([ends - n, ends], 1), 0))


def _records(n, width, height):
    g = torch.Generator(device="cuda").manual_seed(7400 + n)
    u = torch.rand(2, n, generator=g, device="cuda")
    size = torch.tensor([[width // 16], [height // 16]], device="cuda")
    r = torch.zeros(n, 12, device="cuda")
    r[:, 0:2] = ((u * size).floor().clamp(max=size - 1) * 16 + 8).T
    r[:, 2] = r[:, 4] = 2.0
    r[:, 5] = 0.9
    r[:, 7] = r[:, 8] = 2.3
    r[:, 6] = torch.randint(1, 40, (n,), generator=g, device="cuda") / 16
    return r


@pytest.mark.parametrize("height", [4096, 4112])  # 65,536 tiles, the most, and 65,792
@pytest.mark.parametrize("n", [1, 700, 30_000])
def test_many_tiles(n, height):
    from paper_2510_26358_amd.rasterizer import ViewSpec
    _check(ViewSpec([4096], [height], [0], [n]), _records(n, 4096, height),
           torch.ones(n, dtype=torch.uint8, device="cuda"), n, 1 << 16)


@pytest.mark.parametrize("more", [0, 1])  # 2^23 pairs, the most, and one more
def test_many_pairs(more):
    from paper_2510_26358_amd.rasterizer import ViewSpec
    n = (1 << 20) - 1
    views = ViewSpec([640] * 9, [480] * 9, [0] * 9, [n] * 8 + [8 + more])
    q = 8 * n + 8 + more
    recs = _records(1 << 16, 640, 480).repeat((q >> 16) + 1, 1)[:q].contiguous()
    valid = torch.zeros(q, dtype=torch.uint8, device="cuda")
    valid[torch.arange(0, q, 31, device="cuda")] = 1
    valid[-3:] = 1
    _check(views, recs, valid, n, 1 << 19)
