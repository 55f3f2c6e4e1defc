"""The autotuner's report: shapes that run the same kernels have one time, and the pick names the first of them."""
import pytest

from paper_2510_26358_amd.rasterizer import LossTargets, Rasterizer, SplatParams, ViewSpec, cameras_tensor
from tests.oracle_helpers import random_scene

pytestmark = pytest.mark.gpu

ALIKE = [["T8_M64_P1", "T8_M128_P1"], ["T16_M128_P1", "T16_M256_P1"], ["T32_M256_P4", "T32_M512_P2"]]
FEW = ["T16_M64_P2", "T16_M128_P2", "T16_M256_P2", "T16_M64_P4"]  # one kernel each way below 4096 tiles of 16


@pytest.mark.parametrize("width,height,alike", [(160, 120, ALIKE + [FEW]), (1280, 832, ALIKE[:2])])
def test_shapes_of_one_kernel_have_one_time(width, height, alike):
    from paper_2510_26358_amd.tune import tune
    sc = random_scene(991, n=3000, sh_degree=0, width=width, height=height, f=width)
    views, p = ViewSpec.from_scene(sc), SplatParams.from_scene(sc)
    ras = Rasterizer(0)
    res = tune(ras, p, cameras_tensor(sc.cameras), views, LossTargets.from_scene(sc, views), steps=3, warmup=1,
               use_cache=False)
    for names in alike:
        assert all(res["ms"][n] == res["ms"][names[0]] for n in names), names
    b = res["best"]
    fwd, bwd = (f"T{b['tile']}_M{b[x]}_P{b[y]}" for x, y in (("batch", "ppt"), ("batch_bwd", "ppt_bwd")))
    for names in alike:
        assert fwd not in names[1:]
    assert bwd in ("T8_M64_P1", "T16_M128_P1", "T16_M64_P2", "T32_M256_P4")
