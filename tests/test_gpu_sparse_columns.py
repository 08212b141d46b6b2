"""The product over the nonzeros of S*A at the edges of its column layout (two
lanes a column, 512 or 1024 columns a workgroup), and the FP64 normals it
draws, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import U64, rel_fro, to_device
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [1, 2, 255, 256, 257, 511, 512, 513, 1000, 1023])
@pytest.mark.parametrize("prec", ["f64", "bf16", "fp8"])
def test_sparse_product_columns(d, prec):
    from paper_2203_02798_amd import api
    n, m, r = 6000, 37, 4001
    print(f"sparse product d={d} {prec}", flush=True)
    a = synth.csr_uniform(n, d, min(0.2, 40.0 / (d + 40) / 8) / 16, seed=d)
    c = api.sketch_gcs(to_device(a), m, r, seed=3, prec=prec).cpu().numpy()
    ref = {"f64": osk.sketch_gcs, "bf16": osk.sketch_gcs_bf16_reference,
           "fp8": osk.sketch_gcs_fp8_reference}[prec](a, m, r, 3)
    assert rel_fro(c, ref) <= (1e-12 if prec == "f64" else 1e-4)


def test_device_normals():
    """G itself, as G I: every normal to eight roundings of the largest
    radius (sqrt(66 ln 2) < 6.77) against NumPy's."""
    from paper_2203_02798_amd import api
    n, m = 512, 300
    g = api.sketch_g(torch.eye(n, dtype=torch.float64, device="cuda"), m, seed=9)
    z = g.cpu().numpy() * np.sqrt(m)
    ref = osk.gaussian_normals(m, 0, n, 9)
    assert np.abs(z - ref).max() <= 8 * U64 * 6.77 + 2 * U64 * np.abs(ref).max()
