"""A pool of psk_workspace_size bytes (in whole 256) for each slot runs as many
requests at once as there are slots; one that holds less than a single request's
runs it with the smaller workspace that the call accepts."""
import numpy as np
import pytest

import synth
from helpers import to_device

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def test_pool_per_slot():
    from paper_2203_02798_amd import _lib as L
    from paper_2203_02798_amd import api
    a, b, _ = synth.lsq_problem(20000, 50, 10.0, seed=1)
    dev, rhs = to_device(a), torch.from_numpy(b).cuda()
    m, r = 400, 2500
    one = -(-api.workspace_size(L.PSK_OP_LSQ, dev, m=m, r=r) // 256) * 256
    solutions = []
    for pool, slots, most in ((4 * one, 4, 4), (one, 4, 1), (one // 256 * 128 // 256 * 256, 4, 1)):
        print(f"server pool {pool} of {one} a request", flush=True)
        with api.Server(pool, slots=slots) as srv:
            pend = [srv.submit_lsq(dev, rhs, m=m, r=r, seed=3) for _ in range(12)]
            for ticket, x in pend:
                assert srv.wait(ticket)["status"] == "PSK_OK"
                solutions.append(x.cpu().numpy())
            st = srv.stats()
        assert st["pool_peak"] <= pool and st["completed"] == 12
        assert st["inflight_peak"] <= most and st["pool_peak"] % one in (0, st["pool_peak"])
    norm = np.linalg.norm(a)
    for x in solutions:
        res = b - a @ x
        assert np.linalg.norm(a.T @ res) <= 1e-12 * norm * np.linalg.norm(res)
    for x in solutions[1:24]:
        assert (x == solutions[0]).all()
