"""Infinite values stay with the pixels that they belong to.

A Gaussian whose colour is infinite (a diverged coefficient) makes the pixels that keep it infinite and
leaves the others as they are, whichever kernel a launch takes: a small ragged view is rendered alone
(8 x 8 blocks) and beside a large view that sees nothing (8 x 16 blocks), and both are compared with the
same scene under a finite colour of that channel.
"""
import numpy as np
import pytest
import torch

from oracle.render import render
from oracle.settings import RenderSettings
from paper_2510_26358_amd.scenes import empty_lidar
from tests.gpu_helpers import TOL_RGB, run_forward
from tests.oracle_helpers import camera, random_scene

pytestmark = pytest.mark.gpu

LARGE = 1024  # 4096 tiles of 16 x 16: with it a launch takes the 8 x 16 blocks


def _scene(value, large, opacity):
    sc = random_scene(911, n=90, sh_degree=1, width=67, height=45, f=60.0)
    sc.opacity_logits[::7] = opacity
    sc.sh[5, 0, 0] = value  # the red channel of one Gaussian
    if large:  # looks away from every Gaussian
        away = camera(R=np.diag([-1.0, 1.0, -1.0]), f=500.0, width=LARGE, height=LARGE)
        away.g_begin, away.g_end = 0, 90
        sc.cameras.append(away)
        sc.gt_rgb.append(np.zeros((3, LARGE, LARGE)))
        sc.lidar.append(empty_lidar())
    return sc


@pytest.mark.parametrize("opacity", [1.0, 7.0])  # 0.999: above the alpha clamp, tested per pixel
def test_an_infinite_colour_stays_with_its_pixels(opacity):
    from paper_2510_26358_amd.rasterizer import Rasterizer
    ras = Rasterizer(0)
    fin = _scene(1.0, False, opacity)
    ref = render(fin, RenderSettings())[0]
    base = run_forward(fin, ras, depth_var=True)[0][0]
    a = run_forward(_scene(np.inf, False, opacity), ras, depth_var=True)[0][0]
    b, empty = run_forward(_scene(np.inf, True, opacity), ras, depth_var=True)[0]
    assert np.abs(base["rgb"].reshape(3, -1)[:, ref["pix"]].T - ref["rgb"])[~ref["ambiguous"]].max() <= TOL_RGB
    hit = np.isposinf(a["rgb"][0])
    assert 0 < hit.sum() < hit.size / 2
    for k in a:
        same = a[k] == base[k]
        if k == "rgb":
            same[0] |= hit
        assert same.all(), k
        assert np.array_equal(a[k], b[k]), k
        assert not empty[k].any()


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("ppt_bwd", [1, 2])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_an_unbounded_alpha_adjoint_stays_with_its_pixel(value, ppt_bwd, large):
    """One pixel's dL/dalpha without bounds (a ratio by an alpha of zero): the Gaussians that the pixel keeps have
    unbounded gradients, the others the ones that they have with zero there."""
    from paper_2510_26358_amd.rasterizer import Rasterizer
    ras = Rasterizer(0, batch_bwd=128, px_per_thread_bwd=ppt_bwd)
    _, (p, cams, views, out, buf) = run_forward(_scene(1.0, large, 1.0), ras)
    pix = 67 * 21 + 30
    assert 0.05 < float(out[2][pix]) < 0.99

    def grads_of(at_pixel, others):
        up = torch.full((views.n_pixels,), others, device="cuda")
        up[pix] = at_pixel
        g, pose = p.zeros_like(), torch.zeros(views.n_views, 6, device="cuda")
        ras.backward_into(p, cams, views, buf, out, g, pose, upstream=(None, None, up))
        torch.cuda.synchronize()
        return [x.reshape(p.n, -1) for x in g.to_numpy_aos()]

    kept = np.any(grads_of(1.0, 0.0)[0] != 0, axis=1)
    assert 0 < kept.sum() < p.n / 2
    want, got = grads_of(0.0, 1.0), grads_of(value, 1.0)
    for a, b in zip(got, want):
        # float atomics: the order of at most a few hundred additions
        assert np.abs(a[~kept] - b[~kept]).max() <= 1e-4 * np.abs(b).max()
    assert not np.isfinite(got[0][kept]).any()
    assert not got[4].any()  # an alpha adjoint has no colour part
