"""Gram matrix of a dense A at the edges of its 64-column tiles and 16-column
blocks, with row counts around a wavefront's and a workgroup's slab, rows of
any stride and base alignment, and a NaN that may reach its own column only."""
import numpy as np
import pytest

import synth
from helpers import U64, gamma

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [1, 15, 16, 17, 33, 48, 49, 63, 64, 65, 80, 97, 113, 127, 129, 200])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_gram_tile_edges(d, dt):
    from paper_2203_02798_amd import api
    dtype = np.float32 if dt == "f32" else np.float64
    for n in (1, 3, 15, 17, 127, 128, 129, 1023, 4099):
        for pad, shift in ((0, 0), (3, 1)):
            ld = d + pad
            print(f"gram d={d} n={n} {dt} ld={ld}", flush=True)
            flat = synth.dense_gaussian(1, n * ld + shift, seed=7 * n + d, dtype=dtype).ravel()
            flat_t = torch.from_numpy(flat).cuda()
            view = flat_t[shift:].view(n, ld)[:, :d]
            a = flat[shift:].reshape(n, ld)[:, :d].astype(np.float64)
            g = api.gram(view).cpu().numpy().astype(np.float64)
            ref = a.T @ a
            bar = 2 * gamma(n + 2, U64) * (np.abs(a).T @ np.abs(a))
            if dt == "f32":
                bar = bar + 2.0 ** -24 * np.abs(ref)
            assert (np.abs(g - ref) <= bar).all()
            assert (g == g.T).all()
    flat_t[shift:].view(n, ld)[n - 1, d - 1] = float("nan")
    g = api.gram(view).cpu().numpy()
    bad = np.isnan(g)
    assert bad[d - 1].all() and bad[:, d - 1].all() and not bad[:d - 1, :d - 1].any()
