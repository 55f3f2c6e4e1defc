"""Workspaces sized for a larger call have room for a smaller one: the sizes never shrink as the intersection
capacity, the Gaussians or the image grow, also across the lines where a launch changes its sort."""
import ctypes as C

import pytest


def _sizes(tile, side, n, cap):
    from paper_2510_26358_amd import _lib as L
    from paper_2510_26358_amd.rasterizer import ViewSpec
    lib = L.load()
    cfg = L.Config()
    lib.ags_config_default(C.byref(cfg))
    cfg.tile = tile
    s = L.Sizes()
    assert lib.ags_buffer_sizes(C.byref(cfg), C.byref(ViewSpec([side, 40], [side, 30], [0, 0], [n, n]).c), n, 3, cap,
                                C.byref(s)) == 0
    return s.saved_bytes, s.fwd_ws_bytes, s.bwd_ws_bytes


def _never_shrink(sizes):
    for a, b in zip(sizes, sizes[1:]):
        assert all(x <= y for x, y in zip(a, b)), (a, b)


CAPS = [0, 1, 4096, 4097, 100_000, 1 << 20, (1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 22) + 4096, 1 << 23]


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("side", [16, 500, 4096])
@pytest.mark.parametrize("n", [0, 3000, 1_000_000])
def test_sizes_grow_with_the_capacity(tile, side, n):
    _never_shrink([_sizes(tile, side, n, c) for c in CAPS])


@pytest.mark.parametrize("cap", [4000, 1 << 21, 1 << 22, 1 << 23])
def test_sizes_grow_with_the_gaussians_and_the_image(cap):
    edge = 1 << 22  # two views of each count: 2^23 pairs
    _never_shrink([_sizes(16, 500, n, cap) for n in (0, 1, 4096, 4097, 1 << 20, (1 << 20) + 1, edge, edge + 1, 2 * edge)])
    _never_shrink([_sizes(16, side, 3000, cap) for side in (1, 16, 17, 1000, 4064, 4080, 4096, 4112, 9000)])
