"""Binning at the edges of the radix sort: bucket counts around one, two and
three digits, key counts around a 2048-key tile and around the one- and
two-launch scans, OSNAP's pairs, and CSR matrices whose rows are mostly empty."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from helpers import to_device
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _check(a, r, seed):
    """Integer data: every sum exact.  Real data where a bucket is summed by
    one wavefront (r >= 8192 or fewer than 64 rows a bucket): the bits of the
    sums in increasing row order."""
    from paper_2203_02798_amd import api
    sa = api.sketch_cs(to_device(a), r, seed=seed).cpu().numpy()
    np.testing.assert_array_equal(sa, osk.sketch_cs(a, r, seed))


@pytest.mark.parametrize("r", [1, 2, 255, 1023, 1024, 1025, 8192, 65536, (1 << 20) - 1, 1 << 20,
                               (1 << 20) + 1])
@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 32768, 40000])
def test_dense_rows(n, r):
    print(f"sort dense n={n} r={r}", flush=True)
    _check(synth.dense_integer(n, 2, seed=n + r, lo=-4, hi=4), r, 5)
    if r >= 8192 or n < 64 * r:
        _check(synth.dense_gaussian(n, 2, seed=n + r), r, 6)


@pytest.mark.parametrize("n,r,every", [
    (5000, 300, 3), (70000, 1024, 1), (70000, 5000, 700), (1 << 16, 1 << 18, 2),
    ((1 << 24) + 4097, 1 << 19, 4099), (9000, 64, 0)])
def test_csr_rows(n, r, every):
    print(f"sort csr n={n} r={r} every={every}", flush=True)
    rows = np.arange(0, n, every) if every else np.zeros(0, dtype=np.int64)
    vals = np.random.default_rng(r).integers(-4, 5, size=2 * rows.size).astype(np.float64)
    vals[vals == 0] = 1.0
    a = sp.csr_matrix((vals, (np.repeat(rows, 2), np.tile([0, 2], rows.size))), shape=(n, 3))
    _check(a, r, 7)


@pytest.mark.parametrize("n,s,r", [(1, 4, 64), (511, 4, 1024), (513, 4, 1028), (10007, 8, 1 << 16)])
def test_osnap_pairs(n, s, r):
    from paper_2203_02798_amd import api
    print(f"sort osnap n={n} s={s} r={r}", flush=True)
    a = synth.dense_integer(n, 3, seed=n, lo=-4, hi=4)
    sa = api.sketch_osnap(to_device(a), s, 0, r, seed=3).cpu().numpy()
    h, sg = (t.cpu().numpy() for t in api.osnap_hash(n, s, r, seed=3))
    ref = np.zeros((r, 3))
    for k in range(s):
        np.add.at(ref, h[:, k].astype(np.int64), sg[:, k][:, None].astype(np.float64) * a)
    np.testing.assert_allclose(sa, ref / np.sqrt(s), rtol=4e-16, atol=0)
