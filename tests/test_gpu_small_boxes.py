"""Small boxes run their sweeps in one launch that takes ghost cells from
interior images; larger boxes, and boxes with user faces, run one sweep after
another on filled ghosts.  The same box with its first active axis given to a
user hook that fills the same values takes the second route: right-hand side
and ghosts agree bit for bit.  A box beyond the limit with long rows takes the
fused x sweep: equal to slabs with the separate update, bit for bit."""
import numpy as np
import pytest

from gpu_helpers import random_smooth, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import wombat as W  # noqa: E402

DIMS = [(3, 3, 3), (4, 7, 5), (33, 32, 31), (84, 3, 6), (85, 4, 5), (86, 5, 3), (97, 6, 4), (3, 1, 1), (17, 1, 1), (300, 1, 1),
        (1, 9, 1), (1, 1, 40), (5, 1, 9), (40, 33, 1), (130, 1, 7), (1, 20, 30), (25, 3, 70)]


def hook(u, dims, axis, periodic):
    """A user boundary hook that fills one face of `axis` of the tensor u."""
    ax, n = 3 - axis, dims[axis]

    def fill(_ctx, _ptr, face, _stream):
        with torch.cuda.stream(torch.cuda.current_stream()):
            # later axes of u are unfilled then, as for the built-in faces
            if face % 2 == 0:
                src = u.narrow(ax, n, 3) if periodic else u.narrow(ax, 3, 1).expand_as(u.narrow(ax, 0, 3))
                u.narrow(ax, 0, 3).copy_(src.clone())
            else:
                src = u.narrow(ax, 3, 3) if periodic else u.narrow(ax, n + 2, 1).expand_as(u.narrow(ax, 0, 3))
                u.narrow(ax, n + 3, 3).copy_(src.clone())
        return 0

    return W.USER_BC_FN(fill)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("periodic", [True, False])
def test_one_launch_equals_separate_sweeps(dims, periodic):
    axis = next(a for a in range(3) if dims[a] > 1)
    for prec in (W.WW_FP64, W.WW_FP32_MIXED):
        say(f"[small boxes] {dims} {'periodic' if periodic else 'outflow'} precision {prec}")
        u0 = torch.tensor(random_smooth(*dims, seed=sum(dims)), device="cuda")
        h = 0.02
        got = []
        for user in (False, True):
            u = u0.to(torch.float64 if prec == W.WW_FP64 else torch.float32, copy=True)
            bc = [0 if periodic else 1] * 6
            kw = {}
            if user:
                bc[2 * axis] = bc[2 * axis + 1] = 2
                kw["user_bc"] = hook(u, dims, axis, periodic)
            ctx = W.Context(*dims, dx=h, dy=h, dz=h, precision=prec, bc=bc, **kw)
            d = ctx.new_state()
            ctx.rhs(u, d)
            torch.cuda.synchronize()
            got.append((d.cpu().numpy(), u.cpu().numpy()))
            ctx.close()
        assert np.isfinite(got[0][0]).all()
        assert np.array_equal(got[0][0], got[1][0])
        assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("prec", [W.WW_FP64, W.WW_FP32_MIXED])
def test_fused_x_sweep_beyond_the_limit(prec):
    dims = (100, 71, 66)                 # 5.7 k tiles of 256 faces; rows of 101 faces
    say(f"[small boxes] fused x sweep {dims} precision {prec}")
    u0 = torch.tensor(random_smooth(*dims, seed=3), device="cuda")
    out = []
    for slab in (0, 16):
        ctx = W.Context(*dims, dx=0.01, dy=0.01, dz=0.01, precision=prec, slab_planes=slab)
        u = u0.to(ctx.dtype, copy=True)
        dts = [ctx.step(u) for _ in range(2)]
        torch.cuda.synchronize()
        out.append((u[:, 3:-3, 3:-3, 3:-3].cpu().numpy(), dts))
        ctx.close()
    assert out[0][1] == out[1][1]
    assert np.isfinite(out[0][0]).all()
    assert np.array_equal(out[0][0], out[1][0])
