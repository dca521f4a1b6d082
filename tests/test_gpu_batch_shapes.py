"""Launch shapes of the batched form: a batch that was never tuned runs 12 faces
per tile at two blocks per CU (FP64: the one that fits), many small patches 4
faces at two blocks (FP32: 8 at three), and every shape, taken from a cache
file, gives the same bits for whole and for split patches."""
import json

import pytest

from gpu_helpers import random_smooth, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import wombat as W  # noqa: E402

SETS = {"one": [(4, 4, 4)], "even": [(8, 6, 5)] * 12, "split": [(40, 33, 27), (5, 4, 7), (300, 4, 6)],
        "small": [(4, 5, 4)] * 1020 + [(16, 16, 16)] * 4, "larger": [(4, 4, 4)] * 1023 + [(16, 16, 17)]}
DEFAULT = {False: {W.WW_FP64: (12, 1), W.WW_FP32_MIXED: (12, 2)}, True: {W.WW_FP64: (4, 2), W.WW_FP32_MIXED: (8, 3)}}


@pytest.mark.parametrize("precision", [W.WW_FP64, W.WW_FP32_MIXED])
@pytest.mark.parametrize("name", list(SETS))
def test_default_and_every_shape(name, precision, tmp_path):
    dims = SETS[name]
    b = W.Batch(dims, 1.0 / 64, precision=precision)
    default = b.shape()
    assert default[:2] == DEFAULT[name == "small"][precision]
    ar = b.new_arena()
    states = {d: torch.from_numpy(random_smooth(*d, seed=sum(d), amp=0.1)).cuda() for d in set(dims)}
    for p, d in enumerate(dims):
        b.view(ar, p).copy_(states[d])
    start, got = ar.clone(), []
    b.step(ar)
    got.append((default[:2], ar.clone()))
    ar.copy_(start)
    cache = tmp_path / "tune.jsonl"
    b.autotune(ar, str(cache))
    key = json.loads(cache.read_text().splitlines()[-1])["key"]
    for ft in (4, 8, 12, 16):
        for bpc in (1, 3):
            cache.write_text(json.dumps({"key": key, "ft": ft, "bpc": bpc, "ms": 1.0}) + "\n")
            assert b.autotune(ar, str(cache)) == -1.0 and b.shape()[0] == ft
            say(f"[batch shapes] {name} precision {precision} shape {b.shape()}")
            ar.copy_(start)
            b.graph_steps(ar, 1)
            got.append((b.shape()[:2], ar.clone()))
    assert (b.dt()[1] == 0).all()
    for shape, a in got[1:]:
        assert torch.equal(a, got[0][1]), shape
    b.close()


def test_cache_entries_of_earlier_kernels_are_not_taken(tmp_path):
    # a key without the kernels' version names a shape that was best for others
    dims = [(6, 5, 4)] * 3
    h = 1469598103934665603
    for d in dims:
        for v in d:
            h = ((h ^ v) * 1099511628211) % 2 ** 64
    old = {"key": f"gfx950|fp32|{len(dims)}|{h:016x}", "ft": 4, "bpc": 1, "ms": 0.001}
    cache = tmp_path / "tune.jsonl"
    cache.write_text(json.dumps(old) + "\n")
    b = W.Batch(dims, 1.0 / 64)
    ar = b.new_arena()
    for p, d in enumerate(dims):
        b.view(ar, p).copy_(torch.from_numpy(random_smooth(*d, seed=p, amp=0.1)))
    say("[batch shapes] cache of an earlier version")
    assert b.autotune(ar, str(cache)) > 0.0
    lines = [json.loads(x) for x in cache.read_text().splitlines()]
    assert len(lines) == 2 and lines[0] == old and lines[1]["key"] != old["key"]
    assert b.autotune(ar, str(cache)) == -1.0
    assert b.shape()[:2] == (lines[1]["ft"], lines[1]["bpc"])
    b.close()
