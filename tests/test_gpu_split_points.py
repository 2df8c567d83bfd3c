"""Short calls of large formats, where a column tile's points are split over
the waves of a block: LLRs, GMI / MI, hard decisions against the oracle at 2,
4, 8 and 16 groups of eight tiles, one and several column tiles per block, up to
and past the size at which calls are split, with far, near-zero and
non-finite samples.

Bars: LLR 1e-3 max(|lambda|, 1); GMI / MI 1e-4; BER and SER within the decisions
the oracle calls within 2e-3 nats (the LLR bar at zero, twice)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("fmt,snrs,n", [(lambda: w.random_shells(8, 512, 81), [3.0, 15.0], 65),
                                        (lambda: w.random_shells(2, 1024, 82), [25.0], 999),
                                        (lambda: w.format_8d2048(), [2.0, 9.0, 17.0], 33),
                                        (lambda: w.random_shells(4, 4096, 83), [12.0, 20.0], 31),
                                        (lambda: w.pam(10), [30.0], 97)])
def test_split_against_oracle(orc, fmt, snrs, n):
    f = fmt()
    gf = mdgmi.Format.of(f)
    s2 = w.sigma2_from_snr_db(np.array(snrs), f.dim)
    ys, txs = zip(*[w.channel_samples(f, float(v), seed=77, snr_slot=q, n=n) for q, v in enumerate(s2)])
    y, tx = np.stack(ys).astype(np.float32), np.stack(txs)
    print(f"[split] {f.name} {snrs} n={n}", flush=True)
    yd, txd = torch.from_numpy(y).cuda(), torch.from_numpy(tx.view(np.int32)).cuda()
    ref = orc.gmi_per_snr(y.astype(np.float64), tx, f.X, f.labels, s2)
    g = mdgmi.mdgmi_gmi(gf, yd, txd, s2, path="mfma").cpu().numpy()
    h = mdgmi.mdgmi_gmi_hd(gf, yd, txd, s2, path="mfma").cpu().numpy()
    assert np.max(np.abs(g[:, :2] - ref[:, :2])) <= 1e-4 and np.max(np.abs(h[:, :2] - ref[:, :2])) <= 1e-4
    for q in range(len(snrs)):
        lam = mdgmi.mdgmi_llr(gf, yd[q], float(s2[q]), path="mfma").cpu().numpy()
        lr = orc.llr(y[q].astype(np.float64), f.X, f.labels, float(s2[q]))
        assert np.all(np.abs(lam - lr) <= 1e-3 * np.maximum(np.abs(lr), 1.0))
        bits = (f.labels[tx[q]][:, None] >> np.arange(f.m)) & 1
        assert abs(h[q, 6] * n * f.m - np.sum((lr > 0) != (bits > 0))) <= np.sum(np.abs(lr) < 2e-3) + 0.5


def test_split_far_and_non_finite(orc):
    f = w.format_8d2048()
    gf = mdgmi.Format.of(f)
    s2 = float(w.sigma2_from_snr_db(14.0, 8))
    y, tx = w.channel_samples(f, s2, seed=5, snr_slot=0, n=70)
    y32 = y.astype(np.float32)
    y32[3] *= 8.0   # classes beyond the exponent window
    y32[40, 2] = np.nan
    print("[split] far, non-finite", flush=True)
    lam = mdgmi.mdgmi_llr(gf, torch.from_numpy(y32).cuda(), s2, path="mfma").cpu().numpy()
    keep = np.arange(70) != 40
    lr = orc.llr(y32[keep].astype(np.float64), f.X, f.labels, s2)
    assert np.all(np.isnan(lam[40])) and np.all(np.abs(lam[keep] - lr) <= 1e-3 * np.maximum(np.abs(lr), 1.0))
    g = mdgmi.mdgmi_gmi(gf, torch.from_numpy(y32).cuda(), torch.from_numpy(tx.view(np.int32)).cuda(), [s2],
                        path="mfma").cpu().numpy()[0]
    assert np.isnan(g[0]) and g[5] == 1


@pytest.mark.parametrize("n", [256 * 64 - 31, 256 * 64, 256 * 64 + 1])
def test_split_and_whole_agree(n):
    """Around the size where calls stop being split (two column tiles per CU),
    and against a launch shape asked for by mdgmi_set_tuning, which is never
    replaced: the same sums in another order."""
    f = w.format_8d2048()
    gf = mdgmi.Format.of(f)
    s2 = [float(w.sigma2_from_snr_db(11.0, 8))]
    y, tx = mdgmi.mdgmi_generate(gf, 9, s2, n, dtype=torch.float32)
    print(f"[split] n={n}", flush=True)
    a = mdgmi.mdgmi_gmi(gf, y, tx, s2, path="mfma").cpu().numpy()
    mdgmi.mdgmi_set_tuning(4)
    try:
        b = mdgmi.mdgmi_gmi(gf, y, tx, s2, path="mfma").cpu().numpy()
    finally:
        mdgmi.mdgmi_set_tuning(-1)
    assert np.max(np.abs(a[:, :2] - b[:, :2])) <= 1e-6
