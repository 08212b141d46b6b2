"""Row norms of rows whose length is a multiple of 4 but not of 32: the last
chunk's groups of four are loaded whole or not at all, whatever the rows'
stride and alignment, and what follows a row (NaN here) is not used."""
import numpy as np
import pytest

import synth
from helpers import U64, gamma

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d", [4, 8, 12, 16, 20, 28, 36, 60, 100, 252, 260, 316, 572])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rownorms_fours(d, dt):
    from paper_2203_02798_amd import api
    dtype = np.float32 if dt == "f32" else np.float64
    for n, pad, shift in ((1, 0, 0), (33, 5, 1), (700, 1, 3)):
        for k in {1, min(d, 33), d}:
            print(f"rownorms fours d={d} n={n} k={k} {dt}", flush=True)
            ld = d + pad
            flat = np.full(n * ld + shift, np.nan, dtype=dtype)
            a = synth.dense_gaussian(n, d, seed=n + d, dtype=dtype)
            flat[shift:].reshape(n, ld)[:, :d] = a
            view = torch.from_numpy(flat).cuda()[shift:].view(n, ld)[:, :d]
            b = synth.dense_gaussian(d, k, seed=d + k)
            x = api.rownorms_sq(view, torch.from_numpy(b).cuda()).cpu().numpy()
            a64 = a.astype(np.float64)
            ref, mag = ((a64 @ b) ** 2).sum(1), ((np.abs(a64) @ np.abs(b)) ** 2).sum(1)
            assert (np.abs(x - ref) <= 3 * gamma(2 * d + 4, U64) * mag).all()
