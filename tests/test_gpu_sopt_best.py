"""What an s search reports: never less than the GMI at s = 1 that it has
evaluated, and for LLRs without an error, whose cost falls for ever, the first
scale at which the GMI is m, in one pass where nothing is left to gain."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402

GMI1, S, GMI, NGMI, ITERS = 0, 2, 3, 5, 8


def case(m, n, seed):
    rng = np.random.default_rng(seed)
    f = w.Format("any", rng.standard_normal((1 << m, 2)), rng.permutation(1 << m).astype(np.uint32))
    tx = rng.integers(0, 1 << m, n).astype(np.uint32)
    sign = 2.0 * ((f.labels[tx][:, None] >> np.arange(m)) & 1) - 1.0
    return rng, mdgmi.Format.of(f), torch.from_numpy(tx.view(np.int32)).cuda(), sign


@pytest.mark.parametrize("m,n", [(1, 100), (4, 1000), (11, 20_001), (12, 300)])
def test_not_below_a_point_evaluated(m, n):
    print(f"[sopt best] m={m} n={n}", flush=True)
    for seed in range(24):
        rng, gf, tx, sign = case(m, n, seed)
        mu = np.linspace(1.0, 6.0, m)
        lam = (sign * (mu + np.sqrt(2.0 * mu) * rng.standard_normal((n, m)))).astype(np.float32)
        lamd = torch.from_numpy(lam).cuda()
        a = mdgmi.mdgmi_gmi_sopt(gf, lamd, tx).cpu().numpy()
        assert a[GMI] >= a[GMI1] and a[NGMI] == a[GMI] / m
        # the search from its own optimum: the GMI found there stands
        b = mdgmi.mdgmi_gmi_sopt(gf, (lamd * float(a[S])).contiguous(), tx).cpu().numpy()
        assert b[GMI] >= b[GMI1]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("lo,hi", [(50.0, 50.0), (50.0, 90.0), (60.0, 600.0), (800.0, 1e4), (1e5, 1e9)])
def test_without_errors(dtype, lo, hi):
    m, n = 4, 2001
    rng, gf, tx, sign = case(m, n, 3)
    lam = torch.from_numpy(sign * rng.uniform(lo, hi, (n, m))).to("cuda", dtype)
    print(f"[sopt best] no errors {dtype} {lo} {hi}", flush=True)
    a = mdgmi.mdgmi_gmi_sopt(gf, lam, tx).cpu().numpy()
    assert a[GMI1] == m and a[GMI] == m and a[S] == 1.0
    if lo >= 800.0:  # every exponential is 0: so is the slope
        assert a[ITERS] == 1
