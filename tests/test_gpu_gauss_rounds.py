"""The FP64 Gaussian product with as many tiles as the chip holds workgroups in
a round and more: whole K up to two full rounds, halved where three half
rounds are shorter (read off the partial products that are planned), against
the oracle."""
import pytest

import synth
from helpers import rel_fro, to_device
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("m,splits", [(2048, 2), (2100, 2), (3072, 2), (3073, 1)])
def test_tiles_past_a_round(m, splits):
    """d = 4000 is 16 column tiles: 256, 272, 384 and 400 tiles of 128 rows."""
    from paper_2203_02798_amd import _lib as L
    from paper_2203_02798_amd import api
    n, d, r = 2500, 4000, 2048
    print(f"sketch_gcs m={m} d={d} r={r}", flush=True)
    a = synth.dense_gaussian(n, d, seed=5)
    dev = to_device(a)
    sa = api.workspace_size(L.PSK_OP_SKETCH_CS, dev, r=r) + r * d * 8
    scratch = api.workspace_size(L.PSK_OP_SKETCH_GCS, dev, m=m, r=r) - sa
    assert round(scratch / (m * d * 8)) == splits
    c = api.sketch_gcs(dev, m, r, seed=4).cpu().numpy()
    assert rel_fro(c, osk.sketch_gcs(a, m, r, 4)) <= 1e-12
