"""Boxes beyond the one-launch form, with rows for the fused x sweep: they are
made of periodic copies, along y and z, of a box that the oracle steps, and have
to equal the copies of its result.  The copies change the length of the update's
march segments (1, 4 and 16 cells, the last one ragged) and the places of the
x tiles.  RK4 and SSP-RK3 steps, right-hand sides, FP64 and FP32; for the
learned form the small box's own step, bit for bit, and with every interface
troubled the plain FP32 step."""
import math

import pytest

from gpu_helpers import random_smooth, say, scaled_rhs_error, scaled_state_error
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import router as R  # noqa: E402
from paper_1808_10633_amd import wombat as W  # noqa: E402

BASE = (90, 12, 10)
H = 1.0 / BASE[0]
COPIES = [(5, 6), (16, 7), (32, 21)]      # 4.2 k, 15 k and 89 k tiles; segments of 1, 4 and 16 cells
STEPS = 2


def base_state(seed):
    return random_smooth(*BASE, seed=seed, amp=0.15)


def tiled(u, copies, dtype):
    """The padded box of copies of the interior of u along y and z."""
    a = u[:, 3:-3, 3:-3, 3:-3].to("cuda", dtype).repeat(1, copies[1], copies[0], 1)
    out = torch.zeros((8,) + tuple(n + 6 for n in a.shape[1:]), dtype=dtype, device="cuda")
    out[:, 3:-3, 3:-3, 3:-3] = a
    return out


def context(u, precision, **kw):
    n = [m - 6 for m in u.shape[:0:-1]]
    return W.Context(*n, dx=H, dy=H, dz=H, precision=precision, **kw)


def each_copy(u, base, copies):
    """The interior of u as [copies, 8, nz, ny, nx], on the host in FP64."""
    a = u[:, 3:-3, 3:-3, 3:-3]
    for k in range(copies[1]):
        for j in range(copies[0]):
            yield a[:, k * base[2]:(k + 1) * base[2], j * base[1]:(j + 1) * base[1]]


ORACLE = {}


def oracle_result(integrator):
    if integrator not in ORACLE:
        g, u = O.Grid(*BASE, H, H, H), base_state(31)
        rhs, dts = O.rhs(g, u.copy()), []
        for _ in range(STEPS):
            dts.append(O.cfl_dt(g, u))
            (O.rk4_step if integrator == W.RK4 else O.ssprk3_step)(g, u, dts[-1])
        ORACLE[integrator] = g, base_state(31), u, rhs, dts
    return ORACLE[integrator]


@pytest.mark.parametrize("precision", [W.WW_FP64, W.WW_FP32_MIXED])
@pytest.mark.parametrize("integrator", [W.RK4, W.SSPRK3])
@pytest.mark.parametrize("copies", COPIES)
def test_large_box_against_the_oracle(copies, integrator, precision):
    say(f"[large boxes] {BASE} x {copies}, integrator {integrator}, precision {precision}")
    g, u0, ref, rhs, dts = oracle_result(integrator)
    dtype = torch.float64 if precision == W.WW_FP64 else torch.float32
    u = tiled(torch.from_numpy(u0), copies, dtype)
    ctx = context(u, precision, integrator=integrator)
    d = ctx.new_state()
    ctx.rhs(u, d)
    for dt in dts:
        if precision == W.WW_FP64:
            assert abs(ctx.cfl_dt(u) - dt) <= 1e-13 * dt
        ctx.step(u, dt)
    torch.cuda.synchronize()
    copies_u, copies_d = list(each_copy(u, BASE, copies)), list(each_copy(d, BASE, copies))
    # the tolerances of the parity tests of these forms on single boxes
    err = max(scaled_state_error(a.double().cpu().numpy(), g.interior(ref))[0] for a in (copies_u[0], copies_u[-1]))
    err_d, _ = scaled_rhs_error(copies_d[-1].double().cpu().numpy(), g.interior(rhs), g.interior(u0), H)
    say(f"  steps {err:.2e}, right-hand side {err_d:.2e}")
    assert err < (1e-11 if precision == W.WW_FP64 else 1e-5)
    assert err_d < (1e-11 if precision == W.WW_FP64 else 2e-6)
    # a face's and a cell's arithmetic does not depend on their place
    assert all(torch.equal(a, copies_u[0]) for a in copies_u)
    assert all(torch.equal(a, copies_d[0]) for a in copies_d)
    ctx.close()


def test_learned_large_box():
    copies = (8, 6)
    say(f"[large boxes] learned, {BASE} x {copies}")
    u0 = torch.from_numpy(base_state(32))
    theta = R.init_params(7).cuda()
    small, big = u0.cuda().float().contiguous(), tiled(u0, copies, torch.float32)
    cs = context(small, W.WW_FP32_MIXED, learned=1)
    cb = context(big, W.WW_FP32_MIXED, learned=1)
    dt = cs.cfl_dt(small)
    # a threshold that routes interfaces both ways
    gen = torch.Generator().manual_seed(5)
    where = torch.stack([torch.randint(0, m, (4000,), generator=gen) for m in (3, *BASE)], 1).to(torch.int32).cuda()
    z = W.mlp_forward(theta, cs.router_sample(small, where.contiguous())[0])
    thr = 1.0 / (1.0 + math.exp(-float(z.median())))
    cs.set_router(theta, thr, 0)
    cs.rhs(small, cs.new_state())
    sm, tot, _ = cs.router_stats()
    say(f"  {100 * sm / tot:.1f} % smooth")
    assert 0.02 < sm / tot < 0.98
    cb.set_router(theta, thr, 0)
    for _ in range(STEPS):
        cs.step(small, dt)
        cb.step(big, dt)
    torch.cuda.synchronize()
    assert cs.router_stats()[2] == 0 and cb.router_stats()[2] == 0
    want = small[:, 3:-3, 3:-3, 3:-3]
    assert torch.isfinite(want).all()
    assert all(torch.equal(a, want) for a in each_copy(big, BASE, copies))
    # every interface troubled: the plain step up to the contraction of products
    hi = theta.clone()
    hi[-1] = 1e4
    a, b = tiled(u0, copies, torch.float32), tiled(u0, copies, torch.float32)
    cb.set_router(hi, 0.5, 0)
    plain = context(b, W.WW_FP32_MIXED)
    for _ in range(STEPS):
        cb.step(a, dt)
        plain.step(b, dt)
    torch.cuda.synchronize()
    sl = (slice(None),) + (slice(3, -3),) * 3
    scale = b[sl].abs().amax(dim=(1, 2, 3))
    err = float(((a[sl] - b[sl]).abs().amax(dim=(1, 2, 3)) / scale).max())
    say(f"  all troubled against the plain fused step: {err:.2e}")
    assert err < 1e-6
    for c in (cs, cb, plain):
        c.close()
