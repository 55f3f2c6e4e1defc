"""The D-SSIM kernel at the edges of its 44 x 30 tiles: images of one tile, a pixel less or more,
one smaller than the window, and with a mask that ends inside a tile, against the oracle at the path's
tolerances (loss 1e-5, gradients 1e-3 relative)."""
import numpy as np
import pytest

from oracle.render import loss_and_grads
from oracle.settings import RenderSettings
from tests.gpu_helpers import grad_close, run_loss_backward
from tests.oracle_helpers import random_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("w,h", [(7, 6), (44, 30), (43, 31), (45, 29), (55, 41), (89, 61)])
def test_ssim_at_tile_edges(w, h, masked):
    from paper_2510_26358_amd.rasterizer import Rasterizer
    sc = random_scene(500 + w, n=150, sh_degree=1, width=w, height=h, f=0.9 * w)
    masks = None
    if masked:
        ys, xs = np.mgrid[:h, :w]
        masks = [((xs + 2 * ys) % 5 > 1).ravel().nonzero()[0]]
    print("size", w, h, "masked", masked, flush=True)
    g = run_loss_backward(sc, Rasterizer(0), masks=masks, w_l1=0.8, lam=0.5, ssim_w=0.7)
    ref = loss_and_grads(sc, RenderSettings(), masks=masks, w_l1=0.8, lam=0.5, ssim_w=0.7)
    assert abs(g["loss"] - ref["loss"]) <= 1e-5 * max(1, abs(ref["loss"]))
    for name in ["means", "log_scales", "quats", "opacity_logits", "sh"]:
        ok, msg = grad_close(g["grads"][name], ref["grads"][name], ref["amb_gauss"])
        print(name, msg)
        assert ok, (name, msg)
    assert grad_close(g["pose"], ref["pose"])[0]
