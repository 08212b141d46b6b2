"""The bfloat16 Gaussian product at the edges of its column and row tiles: a
column's sums do not depend on the columns beside it, to the bit, and a wide
product is the reference's."""
import numpy as np
import pytest

import synth
from helpers import to_device
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("m", [1, 63, 64, 65, 129, 300])
@pytest.mark.parametrize("r", [300, 5000])
def test_columns_alone(m, r):
    from paper_2203_02798_amd import api
    n = 6000
    a = synth.dense_gaussian(n, 400, seed=m + r)
    full = api.sketch_gcs(to_device(a), m, max(r, m), 7, prec="bf16").cpu().numpy()
    ref = osk.sketch_gcs_bf16_reference(a, m, max(r, m), 7)
    # FP32 accumulation over the buckets: r u32 of the sum of magnitudes at
    # most, far below in practice
    assert np.abs(full - ref).max() <= 2.0 ** -24 * max(r, m) ** 0.5 * 40 * np.abs(ref).max()
    for d in (1, 16, 127, 128, 129, 201, 255, 256, 257):
        print(f"bf16 m={m} r={r} d={d}", flush=True)
        part = api.sketch_gcs(to_device(np.ascontiguousarray(a[:, :d])), m, max(r, m), 7,
                              prec="bf16").cpu().numpy()
        np.testing.assert_array_equal(part, full[:, :d])
