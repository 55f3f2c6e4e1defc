"""Both block shapes of the raster kernels at the sizes where they can go wrong.

A launch of few tiles gives each wave an 8 x 8 block, one of at least 8192 8 x 16 blocks (4096 tiles of
16 pixels, 1024 of 32) gives it 8 x 16 pixels; each wave takes a tile's list 64 entries at a time.  A
small ragged view is rendered alone (8 x 8 blocks) and beside a large view that sees nothing (8 x 16
blocks), with lists that end just below, at and above one chunk and with records that need the
per-pixel tests (opacity above the alpha clamp; a conic near singular).  The two images are the same
bit for bit: every decision and every sum over a pixel's list is made in the same order.  (With several
pixels a thread the large launch takes the staged kernel, which rounds the exponent differently.)
Images, loss and gradients of every shape are each held to the oracle at the path's tolerance; not
with the near-singular conics, whose exponent cancels in single precision (an ellipse of 240 by 0.5
pixels at 45 degrees has terms of 6000, so an error of 4e-4 in its exponent and more in its gradients,
whichever way they are summed).
"""
import numpy as np
import pytest

from oracle.render import loss_and_grads, render
from oracle.settings import RenderSettings
from paper_2510_26358_amd.scenes import empty_lidar
from tests.gpu_helpers import (TOL_ALPHA, TOL_DEPTH_REL, TOL_RGB, grad_close, run_forward,
                               run_loss_backward)
from tests.oracle_helpers import camera, random_scene

pytestmark = pytest.mark.gpu

NAMES = ["means", "log_scales", "quats", "opacity_logits", "sh"]
SHAPES = [(8, 64, 1), (16, 256, 1), (16, 128, 2), (16, 64, 4), (32, 512, 2), (32, 256, 4)]
LARGE = 1024  # 4096 tiles of 16 x 16, 1024 of 32 x 32: with it a launch is just over the line
CASES = [(1, 7, 5), (64, 67, 45), (65, 33, 50), (200, 67, 45)]


def _scene(n, width, height, thin, large):
    sc = random_scene(300 + n, n=n, sh_degree=1, width=width, height=height, f=60.0)
    sc.log_scales[:] += 1.2        # about 7 pixels: most tiles list most of the Gaussians
    sc.opacity_logits[:] -= 1.0    # most pixels stay open over a whole list
    sc.opacity_logits[::7] = 7.0   # 0.999: clamped near the centre
    if thin:
        sc.log_scales[3::11] = [2.5, -6.0, -6.0]  # about 240 by 0.5 pixels
    if large:  # looks away from every Gaussian; its target is the background it renders
        away = camera(R=np.diag([-1.0, 1.0, -1.0]), f=500.0, width=LARGE, height=LARGE)
        away.g_begin, away.g_end = 0, n
        sc.cameras.append(away)
        sc.gt_rgb.append(np.zeros((3, LARGE, LARGE)))
        sc.lidar.append(empty_lidar())
    return sc


def _rasterizer(shape):
    from paper_2510_26358_amd.rasterizer import Rasterizer
    return Rasterizer(0, tile=shape[0], batch=shape[1], px_per_thread=shape[2])


@pytest.mark.parametrize("thin", [False, True])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[2] == 1], ids=str)
@pytest.mark.parametrize("n,width,height", CASES)
def test_images_do_not_depend_on_the_block_shape(shape, n, width, height, thin):
    ras = _rasterizer(shape)
    print("shape", shape, "n", n, "thin", thin, flush=True)
    a = run_forward(_scene(n, width, height, thin, False), ras, depth_var=thin)[0][0]
    b, c = run_forward(_scene(n, width, height, thin, True), ras, depth_var=thin)[0]
    assert a["alpha"].max() > 0.1
    for k in a:
        assert np.array_equal(a[k], b[k]) and not c[k].any()


_refs = {}


def _reference(*key):
    if key not in _refs:
        sc = _scene(*key, False, False)
        _refs[key] = render(sc, RenderSettings()), loss_and_grads(sc, RenderSettings(), w_l1=0.8, lam=0.5)
    return _refs[key]


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("n,width,height", CASES)
def test_both_block_shapes_match_the_oracle(shape, n, width, height, large):
    fwd, ref = _reference(n, width, height)
    print("shape", shape, "n", n, "large", large, flush=True)
    g = run_loss_backward(_scene(n, width, height, False, large), _rasterizer(shape), w_l1=0.8, lam=0.5)
    v, r = g["fwd"][0], fwd[0]
    ok = ~r["ambiguous"]
    assert np.abs(v["rgb"].reshape(3, -1)[:, r["pix"]].T - r["rgb"])[ok].max(initial=0) <= TOL_RGB
    assert np.abs(v["alpha"].reshape(-1)[r["pix"]] - r["alpha"])[ok].max(initial=0) <= TOL_ALPHA
    d = np.abs(v["depth"].reshape(-1)[r["pix"]] - r["depth"]) / np.maximum(1.0, np.abs(r["depth"]))
    assert d[ok].max(initial=0) <= TOL_DEPTH_REL
    assert abs(g["loss"] - ref["loss"]) <= 1e-5 * max(1, abs(ref["loss"]))
    for name in NAMES:
        good, msg = grad_close(g["grads"][name], ref["grads"][name], ref["amb_gauss"])
        print(name, msg)
        assert good, (name, msg)
    assert grad_close(g["pose"][:1], ref["pose"])[0]
    assert not g["pose"][1:].any()
