"""Ragged ends: sample counts that leave lanes of the last batch or column
tile without a sample, at noise levels where the stand-in those lanes work on
(y = 0) is far from the points; and ragged batches whose instances are cut
into items of every size.

Bars: LLR 1e-3 max(|lambda|, 1), GMI / MI 1e-4 against the oracle; a batch
against one call per instance 1e-6 (the tuner may have given the batch another
kernel's arithmetic; the bar that tests hold the FP32 kernels to among
themselves)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("fmt,snr_db", [(lambda: w.square_qam(4), 27.0), (lambda: w.qam_product(4, 7), 24.0),
                                        (lambda: w.qam_product(8, 9), 22.0), (lambda: w.format_8d2048(), 17.0)])
@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 191])
def test_tail_lanes(orc, fmt, snr_db, n):
    f = fmt()
    gf = mdgmi.Format.of(f)
    s2 = float(w.sigma2_from_snr_db(snr_db, f.dim))
    y, tx = w.channel_samples(f, s2, seed=31, snr_slot=2, n=n)
    y32 = y.astype(np.float32)
    yd = torch.from_numpy(y32).cuda()
    txd = torch.from_numpy(tx.view(np.int32)).cuda()
    print(f"[tails] {f.name} n={n}", flush=True)
    ref = orc.llr(y32.astype(np.float64), f.X, f.labels, s2)
    lam = mdgmi.mdgmi_llr(gf, yd, s2, path="mfma").cpu().numpy()
    assert np.all(np.abs(lam - ref) <= 1e-3 * np.maximum(np.abs(ref), 1.0))
    refm = orc.llr_maxlog(y32.astype(np.float64), f.X, f.labels, s2)
    lamm = mdgmi.mdgmi_llr_maxlog(gf, yd, s2, path="mfma").cpu().numpy()
    assert np.all(np.abs(lamm - refm) <= 1e-3 * np.maximum(np.abs(refm), 1.0))
    g = mdgmi.mdgmi_gmi_hd(gf, yd, txd, [s2], path="mfma").cpu().numpy()[0]
    r = orc.gmi(y32.astype(np.float64), tx, f.X, f.labels, s2)
    assert np.all(np.abs(g[:2] - r[:2]) <= 1e-4) and g[4] == n and g[5] == 0


def test_batch_items_of_every_size():
    """One instance that dominates its kind, tiny ones and middling ones, both
    MFMA kinds and the direct one."""
    rng = np.random.default_rng(4)
    fmts = [w.square_qam(2), w.pam(1), w.qam_product(4, 7), w.random_shells(8, 512, 71), w.format_8d2048(),
            w.qam_product(2, 9)]
    counts = [400_003, 70_001, 1, 4097, 20_011, 511]
    items = []
    for f, n in zip(fmts, counts):
        gf = mdgmi.Format.of(f)
        for snr in (3.0, 19.0):
            s2 = float(w.sigma2_from_snr_db(snr, f.dim))
            y, tx = mdgmi.mdgmi_generate(gf, int(rng.integers(1, 1000)), [s2], n, dtype=torch.float32)
            items.append((gf, y[0], tx[0], s2))
    print("[tails] batch", counts, flush=True)
    plan = mdgmi.Batch(items, path="auto")
    a = plan.run().cpu().numpy()
    b = plan.run(use_graph=False).cpu().numpy()
    c = mdgmi.mdgmi_gmi_batched(mdgmi.instances(items), path="auto").cpu().numpy()
    assert a.tobytes() == b.tobytes() == c.tobytes()
    mdgmi.mdgmi_tune_clear()
    for q, (gf, y, tx, s2) in enumerate(items):
        one = mdgmi.mdgmi_gmi(gf, y[None], tx[None], [s2], path="auto").cpu().numpy()[0]
        assert np.all(np.abs(one[:2] - a[q, :2]) <= 1e-6) and a[q, 4] == y.shape[0], (q, one, a[q])
