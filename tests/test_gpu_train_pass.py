"""The fused training pass [in, 256, 256, 256, out] at the edges of its tiles:
sample counts around 16-sample blocks, 256-sample slices and the 64-slice
limit, input widths 1..16, output widths 1..32, in a workspace that starts as
NaN bytes, against the oracle's loss and gradient.

Bars: a gradient passes through at most eight roundings to bf16 (weights,
activations and gradients of four layers), each within 2^-9: 8 x 2^-9 = 1.6%
even if all agreed in sign; per layer |d| <= 2% of the layer's gradient (2-norm).
Loss 2% for the same reason. One train_step = loss_grad + adam_step, bit for
bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


def poisoned(nbytes):
    return torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n,in0,out", [(1, 9, 11), (15, 1, 1), (16, 16, 32), (17, 5, 16), (257, 9, 17), (511, 3, 6),
                                       (4097, 9, 11), (16391, 2, 31)])
def test_pass_against_oracle(orc, n, in0, out):
    sizes = [in0, 256, 256, 256, out]
    rng = np.random.default_rng(n + out)
    net = mdgmi.MLP(sizes, seed=n)
    x = rng.normal(0.0, 0.6, (n, in0)).astype(np.float32)
    t = rng.normal(0.0, 6.0, (n, out)).astype(np.float32)
    print(f"[train] n={n} sizes={sizes}", flush=True)
    net._ws = poisoned(net.workspace(n).numel())
    loss = net.loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()).item()
    g = net.grad().astype(np.float64)
    p = 1.0 / (1.0 + np.exp(-t.astype(np.float64)))   # the oracle takes probabilities
    rl, rg = orc.mlp_loss_grad(net.params().astype(np.float64), sizes, x.astype(np.float64), p)
    assert abs(loss - rl) <= 0.02 * abs(rl)
    o = 0
    for a, b in zip(sizes[:-1], sizes[1:]):
        for cnt in (a * b, b):
            d, r = g[o:o + cnt] - rg[o:o + cnt], rg[o:o + cnt]
            assert np.linalg.norm(d) <= 0.02 * np.linalg.norm(r) + 1e-12, (a, b, cnt)
            o += cnt
    assert np.all(np.isfinite(g))


@pytest.mark.parametrize("n", [33, 4096])
def test_step_is_gradient_then_adam(n):
    sizes = [9, 256, 256, 256, 11]
    rng = np.random.default_rng(n)
    y = torch.from_numpy(rng.normal(0.0, 0.5, (n, 8)).astype(np.float32)).cuda()
    snr = torch.from_numpy(rng.choice(np.arange(2.0, 17.25, 0.25), n).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(0.0, 6.0, (n, 11)).astype(np.float32)).cuda()
    a, b = mdgmi.MLP(sizes, seed=3), mdgmi.MLP(sizes, seed=3)
    x = torch.cat([y, ((snr.double() - 9.5) / 4.5).float()[:, None]], dim=1).contiguous()
    print(f"[train] step n={n}", flush=True)
    ws = poisoned(a.train_workspace_size(n))
    for _ in range(3):
        la = a.train_step(y, snr, t, 1e-3, ws=ws)
        lb = b.loss_grad(x, t)
        b.adam_step(1e-3)
    assert la.item() == lb.item()
    assert a.params().tobytes() == b.params().tobytes() and a.grad().tobytes() == b.grad().tobytes()
    # every copy of the weights followed: the fused kernel and the layer-by-layer path on the trained weights
    c = mdgmi.MLP(sizes, seed=4)
    c.set_params(a.params())
    assert torch.equal(a.llr(y, snr), c.llr(y, snr)) and torch.equal(a.forward(x), c.forward(x))
    assert a.loss_grad(x, t).item() == c.loss_grad(x, t).item() and a.grad().tobytes() == c.grad().tobytes()
