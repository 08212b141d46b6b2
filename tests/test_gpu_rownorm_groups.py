"""Row norms of few rows with an odd number of column-tile pairs: every row
is visited whatever the number of row groups (3 and 5 pairs, 80 and 48
groups, used to leave rows unwritten below about 4600 and 2300 rows)."""
import numpy as np
import pytest

import synth
from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n,d", [(1, 130), (33, 130), (1000, 130), (4000, 129), (3000, 192),
                                 (1000, 160), (1000, 320), (2000, 300)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rownorms_few_rows(n, d, dt):
    from paper_2203_02798_amd import api
    a = synth.dense_gaussian(n, d, seed=n + d, dtype=np.float32 if dt == "f32" else np.float64)
    b = np.triu(synth.dense_gaussian(d, d, seed=d))
    x = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    x = api.rownorms_sq(to_device(a), torch.from_numpy(b).cuda(), x=x).cpu().numpy()
    a64 = a.astype(np.float64)
    ref = ((a64 @ b) ** 2).sum(1)
    mag = ((np.abs(a64) @ np.abs(b)) ** 2).sum(1)
    assert (np.abs(x - ref) <= 3 * gamma(2 * d + 4, U64) * mag).all()


@pytest.mark.parametrize("d,k", [(1, 1), (31, 31), (32, 32), (33, 33), (63, 40), (64, 64), (65, 65),
                                 (96, 96), (97, 97), (97, 20), (127, 64), (130, 8), (256, 256),
                                 (288, 288), (289, 289), (300, 50), (352, 352)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rownorms_tile_edges(d, k, dt):
    """Widths at the edges of the 32-column tiles and chunks, triangular and
    full B, rows of any stride and base alignment, and a NaN that stays in
    its own row."""
    from paper_2203_02798_amd import api
    dtype = np.float32 if dt == "f32" else np.float64
    for n in (1, 15, 33, 300, 4099):
        for pad, shift, tri in ((0, 0, True), (3, 1, False)):
            print(f"rownorms d={d} k={k} n={n} {dt} pad={pad}", flush=True)
            ld = d + pad
            flat = synth.dense_gaussian(1, n * ld + shift, seed=3 * n + d, dtype=dtype).ravel()
            a = flat[shift:].reshape(n, ld)[:, :d].astype(np.float64)
            b = synth.dense_gaussian(d, k, seed=d + k)
            b = np.triu(b) if tri else b
            bad = n // 2
            flat_t = torch.from_numpy(flat).cuda()
            view = flat_t[shift:].view(n, ld)[:, :d]
            view[bad, d - 1] = float("nan")
            x = api.rownorms_sq(view, torch.from_numpy(b).cuda()).cpu().numpy()
            ref = ((a @ b) ** 2).sum(1)
            mag = ((np.abs(a) @ np.abs(b)) ** 2).sum(1)
            ok = np.arange(n) != bad
            assert (np.abs(x - ref)[ok] <= (3 * gamma(2 * d + 4, U64) * mag)[ok]).all()
            # (zero rows of B past a tile's last nonzero are not multiplied)
            assert np.isnan(x[bad]) or (tri and k < d)
