"""Row norms of CSR rows of every length around the row classes (one lane, a
sixteenth of a wavefront, a wavefront, a workgroup), full and triangular B,
and entries that are not finite."""
import numpy as np
import pytest
import scipy.sparse as sp

from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,k,tri", [(140, 140, True), (140, 9, False), (300, 600, False),
                                     (600, 600, True), (1100, 1100, True), (150, 2100, False)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_row_lengths(d, k, tri, dt):
    from paper_2203_02798_amd import api
    print(f"csr row norms d={d} k={k} {dt}", flush=True)
    rng = np.random.default_rng(d + k)
    lens = [0, 1, 2, 3, 4, 5, 6, 15, 16, 17, 31, 32, 33, 34, 63, 64, 65, 75, 76, 127, 128, 129,
            137, 138, 139, d]
    lens = np.array([x for x in lens if x <= d] * 9)
    rng.shuffle(lens)
    n = lens.size
    ptr = np.concatenate([[0], np.cumsum(lens)])
    ind = np.concatenate([np.sort(rng.permutation(d)[:x]) for x in lens]).astype(np.int32)
    val = rng.standard_normal(ptr[-1]).astype(np.float32 if dt == "f32" else np.float64)
    a = sp.csr_matrix((val, ind, ptr), shape=(n, d))
    b = rng.standard_normal((d, k))
    b = np.triu(b) if tri else b
    bad = {}
    for what, length in ((np.nan, 3), (np.inf, 16), (np.nan, 64), (np.inf, d)):
        row = int(np.flatnonzero(lens == length)[0])
        a.data[ptr[row]] = what
        bad[row] = what
    x0 = rng.standard_normal(n)
    x = torch.from_numpy(x0.copy()).cuda()
    x = api.rownorms_sq(to_device(a), torch.from_numpy(b).cuda(), alpha=2.0, beta=-1.0,
                        x=x).cpu().numpy()
    a64 = a.toarray().astype(np.float64)
    ok = np.array([i not in bad for i in range(n)])
    ref = 2.0 * ((a64[ok] @ b) ** 2).sum(1) - x0[ok]
    mag = 2.0 * ((np.abs(a64[ok]) @ np.abs(b)) ** 2).sum(1) + np.abs(x0[ok])
    assert (np.abs(x[ok] - ref) <= 3 * gamma(2 * d + k + 4, U64) * mag).all()
    assert not np.isfinite(x[~ok]).any()
