"""CSR least squares keeps the sketch's own preconditioner where the Gram
matrix would cost more than the passes it saves (read off the iteration
count: a sharpened solve takes a handful): few columns under many rows, and
a full column among sparse ones."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg  # noqa: F401

from helpers import to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _sparse(n, d, per_row, full, seed):
    rng = np.random.default_rng(seed)
    ind = np.sort(rng.integers(1 if full else 0, d, (n, per_row)), axis=1)
    keep = np.ones((n, per_row), bool)
    keep[:, 1:] = ind[:, 1:] != ind[:, :-1]
    if full:
        ind, keep = np.column_stack([np.zeros(n, int), ind]), np.column_stack([np.ones(n, bool), keep])
    ptr = np.concatenate([[0], np.cumsum(keep.sum(1))])
    a = sp.csr_matrix((rng.standard_normal(ptr[-1]), ind[keep].astype(np.int32), ptr), shape=(n, d))
    return a, a @ rng.standard_normal(d) + 1e-3 * rng.standard_normal(n)


@pytest.mark.parametrize("n,d,per_row,full,caller,few", [
    (400000, 10, 1, False, False, False), (400000, 10, 1, False, True, False),
    (300000, 40, 3, True, False, False), (300000, 40, 3, True, True, False),
    (100000, 300, 1, False, True, True), (150000, 300, 3, True, True, False)])
def test_preconditioner_chosen_by_cost(n, d, per_row, full, caller, few):
    from paper_2203_02798_amd import api
    print(f"csr n={n} d={d} per_row={per_row} full={full} caller={caller}", flush=True)
    a, b = _sparse(n, d, per_row, full, seed=n + d)
    dev, bd = to_device(a), torch.from_numpy(b).cuda()
    m, r = 8 * d, max(d * d, 8 * d, 2000)
    if caller:
        _, ri = api.sketch_qr(api.sketch_gcs(dev, m, r, 2))
        x, info = api.lsq_solve(dev, bd, Rinv=ri, refine=0)
    else:
        x, info = api.lsq_solve(dev, bd, m=m, r=r, seed=2, refine=0)
    x = x.cpu().numpy()
    res = b - a @ x
    ne = np.linalg.norm(a.T @ res) / (sp.linalg.norm(a) * np.linalg.norm(res))
    print(f"iters {info['iters']} normal eq {ne:.2e}", flush=True)
    assert info["status"] == "PSK_OK" and ne <= 1e-10
    assert (info["iters"] <= 6) == few
