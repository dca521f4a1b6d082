"""The update by cells, and its march over segments of 1, 2, 4, 8 and 16 cells
(B only, after the fused x sweep; the segment length follows the box): the
whole-box right-hand side and a stage equal, bit for bit, those of 3-plane
slabs, whose launches march one cell at a time."""
import numpy as np
import pytest

from gpu_helpers import random_smooth, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import wombat as W  # noqa: E402


@pytest.mark.parametrize("dims,prec", [((20, 12, 9), W.WW_FP64),          # 1 cell per segment
                                       ((70, 130, 31), W.WW_FP64),        # 2, ragged in x, y and the last segment
                                       ((64, 256, 64), W.WW_FP32_MIXED),  # 4
                                       ((64, 256, 130), W.WW_FP64),       # 8, last segment of 2
                                       ((64, 256, 258), W.WW_FP32_MIXED),  # 16, last segment of 2
                                       # rows long enough for the fused x sweep: B only
                                       ((90, 12, 9), W.WW_FP64),          # 1
                                       ((90, 130, 31), W.WW_FP64),        # 2
                                       ((150, 130, 37), W.WW_FP32_MIXED),  # 4
                                       ((128, 256, 65), W.WW_FP64),       # 8, last segment of 1
                                       ((128, 256, 258), W.WW_FP32_MIXED)])  # 16, last segment of 2
def test_segments_equal_single_planes(dims, prec):
    say(f"[update segments] {dims} precision {prec}")
    u0 = torch.tensor(random_smooth(*dims, seed=7), device="cuda")
    h = 1.0 / dims[0]
    out = []
    for slab in (0, 3):
        ctx = W.Context(*dims, dx=h, dy=h, dz=h, precision=prec, slab_planes=slab)
        u = u0.to(ctx.dtype).contiguous()
        d, acc, us = ctx.new_state(), ctx.new_state(), ctx.new_state()
        ctx.rhs(u, d)
        ctx.stage(0, 1e-3 * h, u, u, acc, us)
        torch.cuda.synchronize()
        out.append([t[:, 3:-3, 3:-3, 3:-3].cpu().numpy() for t in (d, acc, us)])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all()
        assert np.array_equal(a, b)
