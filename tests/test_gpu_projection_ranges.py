"""Projection over views whose Gaussian ranges differ, and the rows it clears for the backward.

A wave handles 64 Gaussians, skips the views whose range misses them and loads the pair counts of the
others four at a time; the lanes outside a view's range must take nothing from it.  Ranges that are
empty, hold one Gaussian, end on and beside a wave's edge and leave a wave one to nine views, at every
SH degree, against the oracle at the path's tolerance.  (The oracle takes no empty range: it is given
the last Gaussian there, which lies behind every camera.)
"""
import numpy as np
import pytest

from oracle.render import loss_and_grads
from oracle.settings import RenderSettings
from paper_2510_26358_amd.scenes import empty_lidar
from tests.gpu_helpers import grad_close, run_loss_backward
from tests.oracle_helpers import camera, random_scene

pytestmark = pytest.mark.gpu

N = 150
RANGES = [(0, 150), (70, 70), (63, 65), (64, 128), (10, 149), (149, 150), (0, 1), (128, 150), (0, 64)]


@pytest.mark.parametrize("sh_degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n_views", [1, 4, 5, 9])
def test_gradients_over_ragged_ranges_match_the_oracle(sh_degree, n_views):
    from paper_2510_26358_amd.rasterizer import Rasterizer
    sc = random_scene(700 + sh_degree, n=N + 1, sh_degree=sh_degree, width=33, height=21)
    sc.means[N] = [0.0, 0.0, -5.0]
    rng = np.random.default_rng(n_views)
    sc.cameras, sc.gt_rgb, sc.lidar = [], [], []
    for b, (g0, g1) in enumerate(RANGES[-n_views:]):
        cam = camera(t=np.array([0.05 * b, -0.03 * b, 0.1]), f=40.0 + b, width=33, height=21)
        cam.g_begin, cam.g_end = g0, g1
        sc.cameras.append(cam)
        sc.gt_rgb.append(rng.uniform(0, 1, (3, 21, 33)))
        sc.lidar.append(empty_lidar())
    print("degree", sh_degree, "views", n_views, flush=True)
    got = run_loss_backward(sc, Rasterizer(0), w_l1=0.8, lam=0.0)
    for cam in sc.cameras:
        if cam.g_begin == cam.g_end:
            cam.g_begin, cam.g_end = N, N + 1
    ref = loss_and_grads(sc, RenderSettings(), w_l1=0.8, lam=0.0)
    for name in ("means", "log_scales", "quats", "opacity_logits", "sh"):
        good, msg = grad_close(got["grads"][name], ref["grads"][name], ref["amb_gauss"])
        assert good, (name, msg)
    good, msg = grad_close(got["pose"], ref["pose"])
    assert good, ("pose", msg)


@pytest.mark.parametrize("spread", [0.2, 3.0])  # every Gaussian in sight, or about one in seven
@pytest.mark.parametrize("n", [1, 16, 17, 63, 64, 65, 130])
def test_the_forward_clears_every_kept_pairs_sums(n, spread):
    """A second step into the same buffers, whose adjoint rows hold the first step's sums: four lanes
    clear a row and a store sixteen, whatever subset of a wave is kept."""
    import torch
    from paper_2510_26358_amd.rasterizer import LossTargets, Rasterizer
    from tests.gpu_helpers import run_forward
    sc = random_scene(800 + n, n=n, sh_degree=1, width=33, height=21)
    sc.means[:] = np.random.default_rng(n).uniform(-spread, spread, (n, 3)) + [0.0, 0.0, 4.0]
    sc.means[0] = [0.0, 0.0, 3.0]
    ras = Rasterizer(0)
    print("n", n, "spread", spread, flush=True)
    _, (p, cams, views, out, buf) = run_forward(sc, ras)
    targets = LossTargets.from_scene(sc, views, w_l1=0.8, lambda_lidar=0.5)
    steps = []
    for _ in range(2):
        ras.forward_into(p, cams, views, buf, out)
        grads, pose = p.zeros_like(), torch.zeros(1, 6, device="cuda")
        ras.backward_into(p, cams, views, buf, out, grads, pose, loss=targets,
                          loss_out=torch.zeros(1, device="cuda"))
        torch.cuda.synchronize()
        steps.append([t.cpu().numpy() for t in grads.tensors()] + [pose.cpu().numpy()])
    assert np.abs(steps[0][0]).max() > 0
    for a, b in zip(*steps):
        good, msg = grad_close(b, a)
        assert good, msg
