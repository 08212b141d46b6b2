"""LSQR on few columns, where one workgroup runs both halves of an iteration
after the pass: widths at the edges of its two sizes and of the general
kernels, dense and CSR, one and several refinement passes, and right-hand
sides that stop it at once."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from helpers import to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

U64 = 2.0 ** -53


@pytest.mark.parametrize("d", [1, 2, 31, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("kind,refine", [("dense", 1), ("csr", 0), ("csr", 2)])
def test_solves(d, kind, refine):
    from paper_2203_02798_amd import api
    n = 3000
    a = synth.dense_gaussian(n, d, seed=d) * np.logspace(0, -2, d)
    if kind == "csr":
        a[np.random.default_rng(d).random((n, d)) < 0.5] = 0.0
    b = synth.dense_gaussian(n, 1, seed=d + 1).ravel()
    am = sp.csr_matrix(a) if kind == "csr" else a
    for rhs, what in ((b, "general"), (a @ np.ones(d), "consistent"), (np.zeros(n), "zero")):
        print(f"small lsq d={d} {kind} refine={refine} {what}", flush=True)
        x, info = api.lsq_solve(to_device(am), torch.from_numpy(rhs).cuda(), m=8 * d + 8,
                                r=64 * d, seed=3, refine=refine)
        x = x.cpu().numpy()
        if what == "zero":
            assert (x == 0.0).all() and info["iters"] == 0
            continue
        ref = np.linalg.lstsq(a, rhs, rcond=None)[0]
        # kappa <= 1e3 here: the normal equations' residual at the solver's
        # tolerance (1e-12 of |A| |r|) moves x by kappa^2 of it at most
        resid = np.linalg.norm(rhs - a @ ref)
        s = np.linalg.svd(a, compute_uv=False)
        bar = 1e-12 * s[0] * resid / s[-1] ** 2 + 64 * n * U64 * (s[0] / s[-1]) ** 2 \
            * np.linalg.norm(ref)
        assert np.linalg.norm(x - ref) <= bar
