"""Gram matrix of a wide dense A whose last 64-column tile is one to four
16-column blocks wide."""
import numpy as np
import pytest

import synth
from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n,d", [(3001, 836), (700, 849), (2000, 321), (5000, 452)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_gram_narrow_last_tile(n, d, dt):
    from paper_2203_02798_amd import api
    print(f"gram n={n} d={d} {dt}", flush=True)
    a = synth.dense_gaussian(n, d, seed=d, dtype=np.float32 if dt == "f32" else np.float64)
    g = api.gram(to_device(a)).cpu().numpy().astype(np.float64)
    a = a.astype(np.float64)
    ref = a.T @ a
    bar = 2 * gamma(n + 2, U64) * (np.abs(a).T @ np.abs(a))
    if dt == "f32":
        bar = bar + 2.0 ** -24 * np.abs(ref)
    assert (np.abs(g - ref) <= bar).all() and (g == g.T).all()
