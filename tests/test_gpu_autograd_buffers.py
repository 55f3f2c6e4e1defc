"""The differentiable render's buffers: freed with its outputs, without the garbage collector, and large
enough on the first forward for a scene of up to two intersections a pair."""
import gc
import weakref

import pytest
import torch

from tests.oracle_helpers import random_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [60, 40_000])
def test_render_outputs_are_freed_by_reference_count(n):
    from paper_2510_26358_amd.autograd import render
    from paper_2510_26358_amd.rasterizer import Rasterizer, SplatParams, ViewSpec, cameras_tensor
    sc = random_scene(811, n=n, sh_degree=1, width=96, height=64, f=60.0)
    p, views, ras = SplatParams.from_scene(sc), ViewSpec.from_scene(sc), Rasterizer(0)
    leaves = [t.requires_grad_(True) for t in p.tensors()] + [torch.zeros(1, 6, device="cuda", requires_grad=True)]
    gc.collect()
    gc.disable()
    try:
        out = render(*leaves, ras, cameras_tensor(sc.cameras), views, sc.sh_degree)
        grads = torch.autograd.grad(out, leaves, [torch.ones_like(o) for o in out], retain_graph=True)
        again = torch.autograd.grad(out, leaves, [torch.ones_like(o) for o in out])
        for a, b in zip(grads, again):  # float atomics: the order of a few thousand additions
            assert torch.linalg.vector_norm(a - b) <= 1e-4 * torch.linalg.vector_norm(a)
        refs = [weakref.ref(o) for o in out]
        del out
        assert all(r() is None for r in refs)
    finally:
        gc.enable()


def test_first_capacity():
    from paper_2510_26358_amd.rasterizer import Rasterizer, SplatParams, ViewSpec, cameras_tensor
    sc = random_scene(812, n=50_000, sh_degree=0, width=96, height=64, f=60.0)
    p, views, ras = SplatParams.from_scene(sc), ViewSpec.from_scene(sc), Rasterizer(0)
    _, buf = ras.render(p, cameras_tensor(sc.cameras), views)
    k = int(buf.counters()[0])
    assert not buf.counters()[2] and buf.capacity == (100_000 if k <= 100_000 else int(k * 1.25) + 1024)
    assert ras.render(p, cameras_tensor(sc.cameras), views, capacity=k)[1].capacity == k
