"""The first capacity guess of a render: two intersections a pair for scenes of ordinary size, and for the largest
batches that the library takes still a capacity that it takes, of bounded memory."""
import ctypes as C

import pytest


@pytest.mark.parametrize("views,n,want", [
    ([(96, 64)], 0, 1 << 16), ([(96, 64)], 50_000, 100_000), ([(1280, 800)], 1000, 512_000),
    ([(641, 397)] * 3, 150_000, 900_000), ([(64, 64)] * 2, (1 << 24) + 1, 1 << 26),
    ([(64, 64)] * 32, (1 << 26) - 1, 1 << 26), ([(65_535, 65_000)], 1000, 65_535 * 65_000 // 2)])
def test_first_capacity(views, n, want):
    from paper_2510_26358_amd import _lib as L
    from paper_2510_26358_amd.rasterizer import ViewSpec, first_capacity
    vs = ViewSpec([w for w, _ in views], [h for _, h in views], [0] * len(views), [n] * len(views))
    cap = first_capacity(vs)
    assert cap == want
    lib = L.load()
    cfg, s = L.Config(), L.Sizes()
    lib.ags_config_default(C.byref(cfg))
    rc = lib.ags_buffer_sizes(C.byref(cfg), C.byref(vs.c), n, 0, cap, C.byref(s))
    # what the pixels alone ask for is refused beyond 2^31 - 1, as it was; pairs alone never are
    assert rc == (0 if cap <= 0x7fffffff else -1)
    assert lib.ags_buffer_sizes(C.byref(cfg), C.byref(vs.c), n, 0, max(1 << 16, vs.n_pixels // 2), C.byref(s)) == rc
