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
