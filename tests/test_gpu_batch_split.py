"""Batched form with patches shared between blocks: patches that exceed half an
even share of the work are split into items of several blocks.  Each patch must
equal the single-box step with the same time step (1e-13 of the state scale in
FP64, 1e-6 in FP32: the same expressions), and a split patch with a
non-physical cell stays as it is."""
import numpy as np
import pytest

from gpu_helpers import random_smooth, say, scaled_state_error
from paper_1808_10633_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import wombat as W  # noqa: E402

DX = 1.0 / 64
CASES = {
    # one patch, every phase split, odd edges
    "one": ([(40, 33, 47)], [0]),
    # long x rows (the flattened tile's upper limit) and rows of 4 cells
    "rows": ([(258, 12, 9), (4, 50, 61), (261, 5, 9)], [0, 1, 2]),
    # large ones among small whole patches
    "mixed": ([(4, 5, 6), (64, 48, 40), (5, 5, 5)] * 2 + [(4, 4, 4)] * 40, [0, 1, 2, 4, 45]),
    # more equal patches than blocks
    "equal": ([(16, 16, 16)] * 1100, [0, 1, 500, 1023, 1024, 1060, 1099]),
}


@pytest.mark.parametrize("precision", [W.WW_FP64, W.WW_FP32_MIXED])
@pytest.mark.parametrize("name", list(CASES))
def test_split_patches_equal_single_box_steps(name, precision):
    dims, checked = CASES[name]
    say(f"[batch split] {name}, {len(dims)} patches, precision {precision}")
    bt = W.Batch(dims, DX, precision=precision)
    ar = bt.new_arena()
    states = {}
    for p, d in enumerate(dims):
        key = (d, p % 7)
        if key not in states:
            states[key] = torch.from_numpy(random_smooth(*d, seed=700 + p % 7, amp=0.2)).to("cuda")
        bt.view(ar, p).copy_(states[key].to(bt.dtype))
    before = {p: bt.view(ar, p).clone() for p in checked}
    bt.step(ar)
    dts, flags = bt.dt()
    assert (flags == 0).all()
    worst = 0.0
    for p in checked:
        nx, ny, nz = dims[p]
        ctx = W.Context(nx, ny, nz, dx=DX, dy=DX, dz=DX, precision=precision)
        u = before[p].clone()
        assert abs(ctx.cfl_dt(u) - dts[p]) <= 1e-14 * dts[p]
        ctx.step(u, float(dts[p]))
        torch.cuda.synchronize()
        sl = I.interior_slices(nx, ny, nz)
        err, _ = scaled_state_error(bt.view(ar, p)[sl].double().cpu().numpy(), u[sl].double().cpu().numpy())
        worst = max(worst, err)
    say(f"  worst scaled difference {worst:.3e}")
    assert worst < (1e-13 if precision == W.WW_FP64 else 1e-6)
    # equal patches give equal results, whichever blocks worked on them
    seen = {}
    for p, d in enumerate(dims):
        v = bt.view(ar, p)[I.interior_slices(*d)]
        key = (d, p % 7)
        assert key not in seen or torch.equal(v, seen[key])
        seen.setdefault(key, v)
    bt.close()


def test_split_patch_with_a_bad_cell_is_left_alone():
    dims = [(32, 30, 28), (30, 32, 24)]
    bt = W.Batch(dims, DX, precision=W.WW_FP64)
    ar = bt.new_arena()
    for p, d in enumerate(dims):
        bt.view(ar, p).copy_(torch.from_numpy(random_smooth(*d, seed=40 + p, amp=0.2)))
    bt.view(ar, 0)[7, 3 + 9, 3 + 8, 3 + 7] = -1.0      # negative energy
    before = ar.clone()
    bt.step(ar)
    dts, flags = bt.dt()
    assert flags[0] == 1 and dts[0] == 0.0
    assert flags[1] == 0 and dts[1] > 0.0
    sl = I.interior_slices(*dims[0])
    assert torch.equal(bt.view(ar, 0)[sl], bt.view(before, 0)[sl])
    sl = I.interior_slices(*dims[1])
    assert not torch.equal(bt.view(ar, 1)[sl], bt.view(before, 1)[sl])
