"""Row norms of a CSR A where B holds a NaN and infinities in its first row:
only the rows of A with an entry in that column may show them, whatever their
length and with or without room for the rows' first nonzeros."""
import ctypes

import numpy as np
import pytest
import scipy.sparse as sp

from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,k,tri", [(140, 140, False), (140, 140, True), (140, 300, False),
                                     (600, 600, True), (150, 2100, False)])
@pytest.mark.parametrize("lean", [False, True])
def test_untouched_rows_stay_finite(d, k, tri, lean):
    from paper_2203_02798_amd import _lib as L
    from paper_2203_02798_amd import api
    print(f"non-finite B d={d} k={k} tri={tri} lean={lean}", flush=True)
    rng = np.random.default_rng(d + k)
    lens = np.array([1, 3, 4, 5, 16, 17, 31, 32] + list(range(33, 50)) + [64, 65, 79, 80, 81, 139])
    lens = np.concatenate([lens, lens])
    n = lens.size
    touch = np.arange(n) >= n // 2  # the second half has an entry in column 0
    ptr = np.concatenate([[0], np.cumsum(lens)])
    ind = np.concatenate([np.sort(np.concatenate([[0], 1 + rng.permutation(d - 1)[:x - 1]]) if t
                                  else 1 + rng.permutation(d - 1)[:x])
                          for x, t in zip(lens, touch)]).astype(np.int32)
    a = sp.csr_matrix((rng.standard_normal(ptr[-1]), ind, ptr), shape=(n, d))
    b = rng.standard_normal((d, k))
    b = np.triu(b) if tri else b
    b[0] = np.inf
    b[0, k // 2] = np.nan
    dev, bd = to_device(a), torch.from_numpy(b).cuda()
    mat = api._mat(dev)
    # without the 4 d bytes of the first nonzeros the lean plan still fits
    size = api.workspace_size(L.PSK_OP_ROWNORMS, dev, k=k) - (512 if lean and k <= 2048 else 0)
    ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    rc = L.lib().rownorms_sq(1.0, ctypes.byref(mat), bd.data_ptr(), k, 0.0, x.data_ptr(), base,
                             size, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    x = x.cpu().numpy()
    a64, b0 = a.toarray()[~touch], b.copy()
    b0[0] = 0.0
    ref = ((a64 @ b0) ** 2).sum(1)
    mag = ((np.abs(a64) @ np.abs(b0)) ** 2).sum(1)
    assert np.isfinite(x[~touch]).all()
    assert (np.abs(x[~touch] - ref) <= 3 * gamma(2 * d + k + 4, U64) * mag).all()
    assert not np.isfinite(x[touch]).any()
