"""Exact LLRs of samples beyond the fp16 split's range (finite y with s ||y||^2
above 65504, or a coordinate above it): the FP32 per-class values, also where
other samples of the same 32 are merely far, or not finite, in the launch shape
that splits a tile's points and in the one that does not.

Bar: 1e-3 max(|lambda|, 1) as elsewhere, plus the rounding of the FP32 distances,
relative to the nearest point, that the fallback takes: dim + 2 roundings of
|x_r - x_j| |2 y - x_r - x_j| <= 2 R (2 |y| + 2 R), for each of two classes."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("fmt,snr", [(w.format_8d2048, 14.0), (lambda: w.random_shells(4, 1024, 84), 16.0),
                                     (lambda: w.random_shells(8, 4096, 85), 12.0), (lambda: w.pam(9), 26.0)])
@pytest.mark.parametrize("variant", [-1, 4])   # as the call chooses (points split), and whole tiles
def test_beyond_fp16(orc, fmt, snr, variant):
    f = fmt()
    gf = mdgmi.Format.of(f)
    s2 = float(w.sigma2_from_snr_db(snr, f.dim))
    s = 1.4426950408889634 / (2.0 * s2)
    n = 5 * 32 + 7
    y = w.channel_samples(f, s2, seed=6, snr_slot=0, n=n)[0].astype(np.float32)
    reach = np.sqrt(66000.0 / s)                    # |y| from which K leaves fp16
    far = lambda i, k: (y[i] / np.linalg.norm(y[i]) * reach * k).astype(np.float32)
    y[3] = far(3, 1.05)                             # alone in its tile
    y[33], y[40] = far(33, 2.0), y[40] * 8.0        # with a sample beyond the exponent window
    y[65], y[70, 0] = far(65, 30.0), np.nan         # with a NaN
    y[99], y[100], y[101, -1] = far(99, 1.3), y[100] * 8.0, np.inf
    y[n - 1] = far(n - 1, 1e3)
    y[130, 0] = 70000.0                             # a coordinate past 65504
    bad = [70, 101]
    keep = np.setdiff1d(np.arange(n), bad)
    print(f"[range] {f.name} variant {variant}", flush=True)
    mdgmi.mdgmi_set_tuning(variant)
    try:
        lam = mdgmi.mdgmi_llr(gf, torch.from_numpy(y).cuda(), s2, path="mfma").cpu().numpy()
    finally:
        mdgmi.mdgmi_set_tuning(-1)
    assert np.all(np.isnan(lam[bad]))
    ref = orc.llr(y[keep].astype(np.float64), f.X, f.labels, s2)
    R, yn = np.linalg.norm(f.X, axis=1).max(), np.linalg.norm(y[keep].astype(np.float64), axis=1)[:, None]
    bar = 1e-3 * np.maximum(np.abs(ref), 1.0) + 2 * (f.dim + 2) * 2.0**-24 * 2 * R * (2 * yn + 2 * R) / (2 * s2)
    assert np.all(np.abs(lam[keep] - ref) <= bar), keep[np.any(~(np.abs(lam[keep] - ref) <= bar), axis=1)]
