"""The FP64 path's one-exponential walk and its per-class evaluation against
the oracle: chunk sizes 2, 4, 8 and 16, one and many chunks, noise levels at
which no, some and all samples have a class beyond the walk's window, far
and non-finite samples.

Bars (the FP64 path's): LLR 1e-9 max(|lambda|, 1), GMI / MI 1e-10, error
rates exact up to decisions the oracle calls within 1e-12 nats."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402

FORMATS = {"pam2": lambda: w.pam(1), "pam4": lambda: w.pam(2), "8psk": lambda: w.psk(3), "16qam": lambda: w.square_qam(4),
           "sh4d-32": lambda: w.random_shells(4, 32, 61), "sh8d-64": lambda: w.random_shells(8, 64, 62),
           "sh8d-4096": lambda: w.random_shells(8, 4096, 63)}


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("snr_db", [-5.0, 20.0, 28.0, 33.0, 50.0])
def test_walk_and_per_class(orc, name, snr_db):
    f = FORMATS[name]()
    gf = mdgmi.Format.of(f)
    s2 = float(w.sigma2_from_snr_db(snr_db, f.dim))
    n = 67 if f.M > 1000 else 515
    y, tx = w.channel_samples(f, s2, seed=7, snr_slot=1, n=n)
    y[3] *= 40.0        # far sample
    print(f"[f64] {name} {snr_db} dB n={n}", flush=True)
    yd = torch.from_numpy(y).cuda()
    txd = torch.from_numpy(tx.view(np.int32)).cuda()
    lam = mdgmi.mdgmi_llr(gf, yd, s2, path="f64").cpu().numpy()
    ref = orc.llr(y, f.X, f.labels, s2)
    assert np.all(np.abs(lam - ref) <= 1e-9 * np.maximum(np.abs(ref), 1.0))
    keep = np.arange(n) != 3
    g = mdgmi.mdgmi_gmi_hd(gf, yd[keep].contiguous(), txd[keep].contiguous(), [s2], path="f64").cpu().numpy()[0]
    r = orc.gmi_per_snr(y[keep][None], tx[keep][None], f.X, f.labels, np.array([s2]))[0]
    assert abs(g[0] - r[0]) <= 1e-10 and abs(g[1] - r[1]) <= 1e-10 and abs(g[2] - r[2]) <= 1e-10
    bits = (f.labels[tx[keep]][:, None] >> np.arange(f.m)) & 1
    lk = ref[keep]
    assert np.abs(g[6] * (n - 1) * f.m - np.sum((lk > 0) != (bits > 0))) <= np.sum(np.abs(lk) < 1e-12) + 0.5


def test_non_finite_rows():
    f = w.square_qam(4)
    gf = mdgmi.Format.of(f)
    y, tx = w.channel_samples(f, 0.05, seed=9, snr_slot=0, n=300)
    y[5, 0] = np.nan
    y[64, 1] = np.inf
    print("[f64] non-finite", flush=True)
    lam = mdgmi.mdgmi_llr(gf, torch.from_numpy(y).cuda(), 0.05, path="f64").cpu().numpy()
    bad = np.isin(np.arange(300), [5, 64])
    assert np.all(np.isnan(lam[bad])) and np.all(np.isfinite(lam[~bad]))
    g = mdgmi.mdgmi_gmi(gf, torch.from_numpy(y).cuda(), torch.from_numpy(tx.view(np.int32)).cuda(), [0.05],
                        path="f64").cpu().numpy()[0]
    assert np.isnan(g[0]) and np.isnan(g[1]) and g[5] == 2


def test_workspace_holds_fewer_samples_and_points():
    """A workspace sized for n samples at several points serves every call
    over fewer samples or points (host-side sizes only)."""
    gf = mdgmi.Format.of(w.square_qam(4))
    top = mdgmi.mdgmi_gmi_workspace_size(gf, 500_000, 11, "f64")
    for n in (1, 255, 70_000, 99_999, 196_608, 400_001, 500_000):
        for q in (1, 2, 3, 7, 11):
            assert mdgmi.mdgmi_gmi_workspace_size(gf, n, q, "f64") <= top


def test_stream_buffers_shorter_than_the_longest():
    """Buffers of fewer samples may take more blocks than the longest one:
    each row still equals mdgmi_gmi on the same samples."""
    f = w.square_qam(4)
    gf = mdgmi.Format.of(f)
    top = 6 * 256 * 256 + 1  # one stride more than the blocks of 6 per CU take (256 CUs)
    y, tx = mdgmi.mdgmi_generate(gf, 5, [0.05], top, dtype=torch.float64)
    st = mdgmi.Stream(gf, 0.05, top, n_lanes=2, path="f64")
    sizes = [top, top - 1, 1000, 200_000]
    print("[f64] stream", sizes, flush=True)
    idx = [st.push(y[0, :k].contiguous(), tx[0, :k].contiguous()) for k in sizes]
    for q, k in zip(idx, sizes):
        g = mdgmi.mdgmi_gmi(gf, y[0, :k].contiguous(), tx[0, :k].contiguous(), [0.05], path="f64").cpu().numpy()[0]
        assert np.array_equal(st.result(q), g)
