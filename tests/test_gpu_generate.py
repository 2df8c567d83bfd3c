"""The sample generator's deviates against the host generator: a single point at
the origin leaves y = sqrt(sigma2) z, so every deviate is compared by itself,
over words whose angles come near the multiples of pi / 2 and whose radii come
near their ends.

Bar: logarithm, root, sine and cosine within about 1 ulp on either side and
three roundings each: 2e-15 of the value (9 ulp)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2011_13695_amd import mdgmi  # noqa: E402


@pytest.mark.parametrize("dim,n", [(1, 1), (1, 100003), (2, 400009), (4, 65), (4, 100000), (8, 50001)])
def test_deviates(dim, n):
    f = w.Format(name="origin", X=np.zeros((2, dim)), labels=np.arange(2, dtype=np.uint32))
    s2 = np.array([0.25, 1.0])
    print(f"[generate] {dim} {n}", flush=True)
    y, tx = mdgmi.mdgmi_generate(mdgmi.Format.of(f), 12, s2, n, snr_slot0=1, dtype=torch.float64)
    y32, _ = mdgmi.mdgmi_generate(mdgmi.Format.of(f), 12, s2, n, snr_slot0=1, dtype=torch.float32)
    idx = np.arange(n)
    for q in range(2):
        z = w.normals(12, 1 + q, idx, dim) * np.sqrt(s2[q])
        np.testing.assert_allclose(y[q].cpu().numpy(), z, rtol=2e-15, atol=0.0)
        assert torch.equal(y[q].float(), y32[q])
        np.testing.assert_array_equal(tx[q].cpu().numpy().view(np.uint32), w.symbol_indices(12, 1 + q, idx, 1))
