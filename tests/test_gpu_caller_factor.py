"""A caller's R^{-1} of an ill-conditioned dense A: the Gram matrix that its
rounding bound would throw away is not formed, and the one that helps is."""
import numpy as np
import pytest

import synth
from helpers import to_device
from oracle import lsq as olsq

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n,d,cond,dt,heavy,formed", [
    (3000, 200, 1e7, "f64", False, False), (3000, 200, 1e7, "f64", True, False),
    (2000, 129, 3e7, "f64", False, False),
    (5000, 400, 1e6, "f64", False, False), (5000, 400, 1e6, "f64", True, False), (6000, 300, 1e7, "f32", False, False),
    (3000, 200, 1e3, "f64", False, True), (3000, 200, 1e3, "f64", True, True),
    (20000, 128, 1e3, "f32", False, True), (1000, 129, 1e2, "f64", False, True)])
def test_gram_formed_where_it_is_kept(n, d, cond, dt, heavy, formed):
    from paper_2203_02798_amd import api
    print(f"caller's factor n={n} d={d} cond={cond} {dt} heavy={heavy}", flush=True)
    a, b, _ = synth.lsq_problem(n, d, cond, seed=d)
    if heavy:  # a sampled row 1e4 times the others
        a[n // 2] *= 1e4
    a = a.astype(np.float32 if dt == "f32" else np.float64)
    dev, bd = to_device(a), torch.from_numpy(b).cuda()
    _, ri = api.sketch_qr(api.sketch_gcs(dev, 4 * d, min(n, 40 * d), 2))
    with api.kernel_timing() as kt:
        x, info = api.lsq_solve(dev, bd, Rinv=ri)
        torch.cuda.synchronize()
        grams = kt.stats().get("gram", (0.0, 0))[1]
    a = a.astype(np.float64)
    rn, _ = olsq.lsq_quality(a, b, x.cpu().numpy())
    rs, _ = olsq.lsq_quality(a, b, olsq.lstsq(a, b))
    print(f"iters {info['iters']} grams {grams} excess {(rn - rs) / rs:.1e}", flush=True)
    assert info["status"] == "PSK_OK" and (rn - rs) / rs <= 1e-10
    assert (grams == 1) == formed and (info["iters"] <= 12) == formed
