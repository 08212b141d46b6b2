"""CSR row norms where a wavefront has few or many rows of 5 to 9 entries,
among empty, shorter and longer ones, against the product; the rows that are
not finite are those whose entries are not."""
import numpy as np
import pytest
import scipy.sparse as sp

from helpers import U64, gamma, to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# a full wavefront's worth of rows, and 2.5 rows an entry of the longest
@pytest.mark.parametrize("waves,longest,count", [
    (9, 5, 12), (9, 5, 13), (9, 7, 18), (9, 9, 22), (9, 9, 23), (9, 9, 64), (4100, 6, 15),
    (4100, 8, 20), (4100, 9, 30)])
@pytest.mark.parametrize("d,dt,tri", [(9, "f64", False), (200, "f64", True), (300, "f32", False)])
def test_rows_in_a_wavefront(waves, longest, count, d, dt, tri):
    from paper_2203_02798_amd import api
    print(f"csr row norms waves={waves} longest={longest} count={count} d={d} {dt}", flush=True)
    rng = np.random.default_rng(count + d)
    tail = 37  # the last wavefront has fewer rows than lanes
    lens = []
    for w in range(waves):
        rest = rng.choice([0, 1, 4, 10, 16, 17, 33], size=64 - count)
        x = np.concatenate([[longest], rng.integers(5, longest + 1, count - 1), np.minimum(rest, d)])
        lens.append(rng.permutation(x))
    lens = np.concatenate(lens + [rng.integers(5, longest + 1, tail)])
    n = lens.size
    ptr = np.concatenate([[0], np.cumsum(lens)])
    # distinct columns of a row: a random start and a stride prime to d
    which = np.repeat(np.arange(n), lens)
    at = np.arange(ptr[-1]) - ptr[:-1][which]
    strides = np.array([q for q in range(1, d) if np.gcd(q, d) == 1])
    ind = ((rng.integers(0, d, n)[which] + at * rng.choice(strides, n)[which]) % d).astype(np.int32)
    a = sp.csr_matrix((rng.standard_normal(ptr[-1]).astype(np.float32 if dt == "f32" else
                                                           np.float64), ind, ptr), shape=(n, d))
    bad = rng.choice(np.flatnonzero((lens >= 5) & (lens <= 9)), 4, replace=False)
    a.data[ptr[bad]] = [np.nan, np.inf, -np.inf, np.nan]
    b = rng.standard_normal((d, d))
    b = np.triu(b) if tri else b
    x0 = rng.standard_normal(n)
    x = api.rownorms_sq(to_device(a), torch.from_numpy(b).cuda(), alpha=2.0, beta=-1.0,
                        x=torch.from_numpy(x0.copy()).cuda()).cpu().numpy()
    ok = np.ones(n, bool)
    ok[bad] = False
    some = np.flatnonzero(ok)
    some = some[np.arange(0, some.size, 1 + some.size // 9000)]
    a64 = a[some].toarray().astype(np.float64)
    ref = 2.0 * ((a64 @ b) ** 2).sum(1) - x0[some]
    mag = 2.0 * ((np.abs(a64) @ np.abs(b)) ** 2).sum(1) + np.abs(x0[some])
    assert (np.abs(x[some] - ref) <= 3 * gamma(3 * d + 4, U64) * mag).all()
    assert np.isfinite(x[ok]).all() and not np.isfinite(x[bad]).any()
