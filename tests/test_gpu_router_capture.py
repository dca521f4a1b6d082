"""Right-hand sides and stages of the learned form captured in a HIP graph: every
replay, with eager work and synchronisations between, equals the eager call
(the troubled queue's counters are cleared by each replay)."""
import math

import pytest

from gpu_helpers import random_smooth, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import router as R  # noqa: E402
from paper_1808_10633_amd import wombat as W  # noqa: E402


@pytest.mark.parametrize("dims", [(90, 12, 10), (20, 18, 9), (70, 40, 1)])
@pytest.mark.parametrize("mode", [0, 1])
def test_captured_learned_rhs_and_stage(dims, mode):
    say(f"[learned capture] {dims} mode {mode}")
    stream = torch.cuda.Stream()
    h = 1.0 / dims[0]
    with torch.cuda.stream(stream):
        ctx = W.Context(*dims, dx=h, dy=h, dz=h, precision=W.WW_FP32_MIXED, learned=1, stream=stream.cuda_stream)
        theta = R.init_params(7).cuda()
        u = torch.from_numpy(random_smooth(*dims, seed=9, amp=0.15)).cuda().float().contiguous()
        where = torch.stack([torch.randint(0, m, (2000,)) for m in ((3 if dims[2] > 1 else 2), *dims)], 1)
        z = W.mlp_forward(theta, ctx.router_sample(u, where.to(torch.int32).cuda().contiguous())[0])
        ctx.set_router(theta, 1.0 / (1.0 + math.exp(-float(z.median()))), mode)
        want, acc0, us0, got, acc, us = (ctx.new_state() for _ in range(6))
        dt = 1e-3 * h
        ctx.rhs(u, want)
        ctx.stage(0, dt, u, u, acc0, us0)
        stream.synchronize()
        counts = ctx.router_stats()[:2]
        if mode == 0:
            assert 0 < counts[0] < counts[1]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
            ctx.rhs(u, got)
            ctx.stage(0, dt, u, u, acc, us)
        for replay in range(4):
            for t in (got, acc, us):
                t.fill_(float("nan"))
            graph.replay()
            stream.synchronize()
            sl = tuple(slice(3, -3) if n > 1 else slice(None) for n in dims[::-1])
            for a, b in ((got, want), (acc, acc0), (us, us0)):
                assert torch.isfinite(a[(slice(None),) + sl]).all()
                assert torch.equal(a[(slice(None),) + sl], b[(slice(None),) + sl]), replay
            assert ctx.router_stats()[:2] == counts
            ctx.rhs(u, torch.empty_like(u))          # eager work between the replays
            stream.synchronize()
    ctx.close()
