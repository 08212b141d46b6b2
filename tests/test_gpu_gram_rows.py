"""Gram matrix of a narrow dense A on both sides of the row count from which
four wavefronts share an item, and with the smallest workspace."""
import ctypes

import numpy as np
import pytest

import synth
from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n", [1, 47, 49, 1000, 2000, 2001, 24000, 50007])
@pytest.mark.parametrize("d,dt", [(1, "f64"), (49, "f32"), (64, "f64"), (65, "f64"), (97, "f32"),
                                  (112, "f64"), (113, "f64")])
def test_gram_rows(n, d, dt):
    from paper_2203_02798_amd import _lib as L
    from paper_2203_02798_amd import api
    print(f"gram n={n} d={d} {dt}", flush=True)
    a = synth.dense_gaussian(n, d, seed=n + d, dtype=np.float32 if dt == "f32" else np.float64)
    dev = to_device(a)
    mat = api._mat(dev)
    full = api.workspace_size(L.PSK_OP_GRAM, dev)
    ws = torch.empty(full + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    a = a.astype(np.float64)
    ref = a.T @ a
    bar = 2 * gamma(n + 2, U64) * (np.abs(a).T @ np.abs(a))
    if dt == "f32":
        bar = bar + 2.0 ** -24 * np.abs(ref)
    # half the full plan's partials hold the lean plan of few rows (128 rows a slab, not 48)
    for size in (full, full // 2 if d <= 112 and n == 2000 else full):
        c = torch.zeros(d, d, dtype=dev.dtype, device="cuda")
        rc = L.lib().gram(1.0, ctypes.byref(mat), 0.0, c.data_ptr(), base, size,
                          torch.cuda.current_stream().cuda_stream)
        g = c.cpu().numpy().astype(np.float64)
        assert rc == 0 and (np.abs(g - ref) <= bar).all() and (g == g.T).all()
