"""Searches that go on past the passes launched ahead, several at once on
streams of their own (so that blocks of one start late, behind another's): the
same bits as each by itself."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


def test_searches_side_by_side():
    m, n = 6, 300_001
    rng = np.random.default_rng(12)
    f = w.Format("any", rng.standard_normal((1 << m, 2)), rng.permutation(1 << m).astype(np.uint32))
    gf = mdgmi.Format.of(f)
    tx = rng.integers(0, 1 << m, n).astype(np.uint32)
    sign = 2.0 * ((f.labels[tx][:, None] >> np.arange(m)) & 1) - 1.0
    mu = np.linspace(1.0, 6.0, m)
    lam = sign * (mu + np.sqrt(2.0 * mu) * rng.standard_normal((n, m)))
    txd = torch.from_numpy(tx.view(np.int32)).cuda()
    size = mdgmi.mdgmi_gmi_sopt_workspace_size(n)
    calls = []
    for scale, dt in [(1e-3, torch.float32), (900.0, torch.float64), (1e-4, torch.float64), (0.9, torch.float32)]:
        calls.append((torch.from_numpy(lam * scale).to("cuda", dt), mdgmi.workspace(size),
                      torch.empty(9, dtype=torch.float64, device="cuda"), torch.cuda.Stream()))
    print("[sopt] four streams", flush=True)
    alone = [mdgmi.mdgmi_gmi_sopt(gf, llr, txd).cpu().numpy() for llr, _, _, _ in calls]
    assert max(a[8] for a in alone) > 6
    torch.cuda.synchronize()
    for _ in range(3):
        for llr, ws, out, st in calls:
            mdgmi.mdgmi_gmi_sopt(gf, llr, txd, out=out, ws=ws, stream=st)
        torch.cuda.synchronize()
        for a, (_, _, out, _) in zip(alone, calls):
            assert out.cpu().numpy().tobytes() == a.tobytes()
