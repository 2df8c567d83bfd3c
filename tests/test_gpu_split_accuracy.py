"""Calls short enough that a column tile's points are split over a block's waves are
no further from the FP64 values than the same samples in a launch shape that walks
whole tiles: root mean square over thirty sets of samples, from many errors to
few. Bar: 1.05 times, plus 2e-9 bit (the spread of a mean of thirty)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("fmt", [w.format_8d2048, lambda: w.random_shells(8, 512, 81),
                                 lambda: w.random_shells(4, 4096, 83), lambda: w.random_shells(2, 1024, 82)])
@pytest.mark.parametrize("snr", [0.0, 4.0, 9.0, 14.0])
@pytest.mark.parametrize("fn", ["mdgmi_gmi", "mdgmi_gmi_hd"])
def test_no_further_from_64_bits(fmt, snr, fn):
    f = fmt()
    gf = mdgmi.Format.of(f)
    s2 = [float(w.sigma2_from_snr_db(snr, f.dim))]
    call = getattr(mdgmi, fn)
    off = {-1: [], 4: []}
    print(f"[split accuracy] {f.name} {snr} {fn}", flush=True)
    for seed in range(30):
        y, tx = mdgmi.mdgmi_generate(gf, seed, s2, 1500, dtype=torch.float32)
        ref = mdgmi.mdgmi_gmi(gf, y.double().contiguous(), tx, s2, path="f64").cpu().numpy()[0, :2]
        for variant in off:
            mdgmi.mdgmi_set_tuning(variant)   # 4: sixteen waves, a tile each; never split
            try:
                off[variant].append(call(gf, y, tx, s2, path="mfma").cpu().numpy()[0, :2] - ref)
            finally:
                mdgmi.mdgmi_set_tuning(-1)
    split, whole = (np.sqrt(np.mean(np.square(off[v]), axis=0)) for v in (-1, 4))
    print(f"[split accuracy] GMI, MI: split {split}, whole {whole}", flush=True)
    assert np.all(split <= 1.05 * whole + 2e-9), (split, whole)
