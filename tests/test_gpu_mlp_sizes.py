"""The gradient of the router's MLP at the edges of its blocks (128 samples,
16 per wave) and of the reduction over blocks (16 partials at a time, four in
flight), on features that start at any float, against the FP64 oracle with
the operands rounded as the kernel rounds them."""
import numpy as np
import pytest

from oracle import mlp as M
from gpu_helpers import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1808_10633_amd import wombat as W  # noqa: E402
from test_gpu_router import bf16, grad_bf16  # noqa: E402


@pytest.mark.parametrize("n,shift", [(1, 0), (17, 1), (127, 0), (128, 2), (129, 0), (2048, 3), (2049, 0), (8193, 0),
                                     (8321, 1)])
def test_mlp_grad_sizes(n, shift):
    say(f"[mlp grad sizes] n {n} shift {shift}")
    rng = np.random.default_rng(n)
    theta = M.init_params(3)
    theta[M.NH * M.NIN:M.NH * M.NIN + M.NH] = rng.normal(size=M.NH) * 0.1
    theta[-1] = -0.2
    theta = theta.astype(np.float32).astype(np.float64)
    X = bf16(rng.uniform(-1, 1, size=(2 * n + 64, 48)).astype(np.float32))
    _, _, _, (z1, z2) = grad_bf16(theta, X, np.zeros(len(X)))
    # no ReLU argument near zero: FP32 and FP64 then take the same masks
    X = X[(np.abs(z1).min(1) > 1e-3) & (np.abs(z2).min(1) > 1e-3)][:n]
    assert len(X) == n
    t = (rng.uniform(size=n) < 0.4).astype(np.float64)
    buf = torch.zeros(48 * n + 4, dtype=torch.float32, device="cuda")
    Xg = buf[shift:shift + 48 * n].view(n, 48)
    Xg.copy_(torch.tensor(X, dtype=torch.float32))
    th = torch.tensor(theta, dtype=torch.float32, device="cuda")
    tg = torch.tensor(t, dtype=torch.float32, device="cuda")
    g, loss = W.mlp_grad(th, Xg, tg)
    g2, loss2 = W.mlp_grad(th, Xg, tg)
    assert torch.equal(g, g2) and torch.equal(loss, loss2)
    g = g.double().cpu().numpy()
    ge, le, absd, _ = grad_bf16(theta, X, t)
    # per parameter: operands that FP32 and FP64 round to neighbouring BF16
    # values (2^-7 of a term, once more from D2 into D1) and FP32 sums of n
    # terms (n 2^-24 < 2^-10): 2^-6 of the sum of absolute terms, and a floor
    bound = 2.0 ** -6 * absd + 1e-9
    err = np.abs(g - ge)
    assert (err <= bound).all(), float((err / bound).max())
    # the loss: FP32 logits (1e-6 of their scale) and an FP32 mean
    assert abs(float(loss) - le) < 1e-5
