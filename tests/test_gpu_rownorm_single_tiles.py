"""Row norms past 256 columns, where a workgroup takes one or two column tiles
in turn: both give every row the same sums, at the row counts where the number
of tiles taken changes."""
import numpy as np
import pytest

import synth
from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,k", [(257, 32), (257, 33), (320, 64), (320, 65), (320, 320),
                                 (576, 100), (576, 576), (321, 400)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rownorms_single_tiles(d, k, dt):
    from paper_2203_02798_amd import api
    a = synth.dense_gaussian(70000, d, seed=d, dtype=np.float32 if dt == "f32" else np.float64)
    b = synth.dense_gaussian(d, k, seed=k)
    dev, bd = to_device(a), torch.from_numpy(b).cuda()
    a64 = a[:2049].astype(np.float64)
    ref, mag = ((a64 @ b) ** 2).sum(1), ((np.abs(a64) @ np.abs(b)) ** 2).sum(1)
    bar = 3 * gamma(2 * d + 4, U64) * mag
    want = api.rownorms_sq(dev, bd).cpu().numpy()
    assert (np.abs(want[:2049] - ref) <= bar).all()
    for n in (1, 2049, 6145, 12289, 20000, 32769, 65537):
        print(f"rownorms single tiles d={d} k={k} n={n} {dt}", flush=True)
        x = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
        x = api.rownorms_sq(dev[:n], bd, x=x).cpu().numpy()
        assert (x == want[:n]).all()
