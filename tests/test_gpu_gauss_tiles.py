"""The FP64 Gaussian product at the edges of its column tiles (32, 64, 128
and 256 columns) and K splits, and with a workspace that holds only the lean
plan, against the oracle (1e-12 normwise: each entry sums r products of
magnitude at most |G| |S A|, in any grouping)."""
import ctypes

import numpy as np
import pytest

import synth
from helpers import rel_fro, to_device
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n,d,m,r", [
    (500, 1, 3, 15), (2000, 31, 129, 1024), (2000, 32, 256, 1025), (1500, 33, 64, 63),
    (1500, 64, 200, 2500), (1500, 65, 130, 4096), (1500, 128, 128, 65), (1500, 129, 300, 700),
    (1200, 256, 257, 1111), (1200, 257, 516, 1300), (1200, 300, 600, 1201)])
def test_sketch_gcs_column_tiles(n, d, m, r):
    from paper_2203_02798_amd import api
    print(f"sketch_gcs n={n} d={d} m={m} r={r}", flush=True)
    a = synth.dense_gaussian(n, d, seed=d)
    c = api.sketch_gcs(to_device(a), m, r, seed=4).cpu().numpy()
    assert rel_fro(c, osk.sketch_gcs(a, m, r, 4)) <= 1e-12


def test_sketch_gcs_lean_workspace():
    """The smallest workspace accepted (found from the host-side check alone,
    by halving) is below the planned one and gives the same product."""
    from paper_2203_02798_amd import _lib as L
    from paper_2203_02798_amd import api
    n, d, m, r = 2000, 32, 256, 1024
    a = synth.dense_gaussian(n, d, seed=1)
    ad = to_device(a)
    full = api.workspace_size(L.PSK_OP_SKETCH_GCS, ad, m=m, r=r)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    c = torch.empty((m, d), dtype=torch.float64, device="cuda")
    mat = api._mat(ad)

    def call(nbytes):
        return L.lib().sketch_gcs(ctypes.byref(mat), m, r, 4, L.PSK_PREC_F64, c.data_ptr(),
                                  ws.data_ptr(), nbytes, api._stream(ad.device))

    lo, hi = 0, full
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if call(mid) == L.PSK_OK:
            hi = mid
        else:
            lo = mid
    c.zero_()
    assert call(hi) == L.PSK_OK and hi < full - 4 * m * d * 8
    assert rel_fro(c.cpu().numpy(), osk.sketch_gcs(a, m, r, 4)) <= 1e-12
    assert call(hi - 1) == -3  # PSK_ENOMEM
