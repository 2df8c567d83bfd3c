"""LLRs and max-log LLRs with the path left to the library and the workspace of
the size asked for it, from the smallest formats on (and at the edges of the
rules that choose the path), against the oracle. Bar: 1e-3 max(|lambda|, 1)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("fmt", [lambda: w.pam(1), lambda: w.pam(2), lambda: w.pam(3), lambda: w.pam(4),
                                 lambda: w.square_qam(2), lambda: w.square_qam(4), lambda: w.qam_product(4, 4),
                                 lambda: w.qam_product(8, 4), lambda: w.square_qam(6),
                                 lambda: w.random_shells(8, 64, 87)])
@pytest.mark.parametrize("n", [1, 1000])
def test_auto_with_its_own_workspace(orc, fmt, n):
    f = fmt()
    gf = mdgmi.Format.of(f)
    s2 = float(w.sigma2_from_snr_db(9.0, f.dim))
    y = w.channel_samples(f, s2, seed=7, snr_slot=0, n=n)[0].astype(np.float32)
    yd = torch.from_numpy(y).cuda()
    print(f"[auto] {f.name} n={n}", flush=True)
    ref = orc.llr(y.astype(np.float64), f.X, f.labels, s2)
    lam = mdgmi.mdgmi_llr(gf, yd, s2).cpu().numpy()
    assert np.all(np.abs(lam - ref) <= 1e-3 * np.maximum(np.abs(ref), 1.0))
    ref = orc.llr_maxlog(y.astype(np.float64), f.X, f.labels, s2)
    lam = mdgmi.mdgmi_llr_maxlog(gf, yd, s2).cpu().numpy()
    assert np.all(np.abs(lam - ref) <= 1e-3 * np.maximum(np.abs(ref), 1.0))
