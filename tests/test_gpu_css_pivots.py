"""Column selection at the edges of the pivot search in the Gram matrix: its
panels of 16 pivots, its workgroup sizes and LDS rows, and inputs that it
hands to the QR steps (equal columns, columns near nothing)."""
import numpy as np
import pytest

import synth
from helpers import to_device
from oracle import css as ocss
from oracle import sketch as osk

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,k,kind", [
    (2, 2, ""), (17, 16, ""), (17, 17, ""), (63, 33, ""), (64, 32, ""), (65, 65, ""),
    (130, 48, "equal"), (130, 40, "scales"), (300, 100, ""), (300, 90, "tiny"), (1100, 50, ""),
    (2100, 30, "")])
def test_pivots_match_the_qr(d, k, kind):
    from paper_2203_02798_amd import api
    n = 4 * d + 100
    a = synth.dense_gaussian(n, d, seed=d + k)
    order = np.random.default_rng(d).permutation(d)
    spread = {"": 1e2, "equal": 1e2, "scales": 1e9, "tiny": 1e2}[kind]
    a = a * np.logspace(0, -np.log10(spread), d)[order]
    if kind == "equal":  # pairs of equal columns: exact ties from the first step on
        a[:, order[1]] = a[:, order[0]]
        a[:, order[31]] = a[:, order[30]]
    if kind == "tiny":   # squared norms below the normal range
        a = a * 1e-160
    m, r = 2 * d + 2, 3 * d + 5
    dev = api.css_select(to_device(a), m, r, k, seed=9).cpu().numpy().astype(np.int64)
    b = osk.sketch_gcs(a, m, r, 9)
    if kind == "tiny":
        b = b * 2.0 ** 531  # the same pivots, at a scale that squares hold
    ref, _ = ocss.qrcp_pivots(b, k)
    assert len(set(dev.tolist())) == k and dev.min() >= 0 and dev.max() < d
    if kind == "tiny":  # only that the call ends with distinct columns
        return
    if not np.array_equal(dev, ref):
        took, best = ocss.qrcp_replay(b, dev)
        assert np.all(took >= best * (1 - 1e-10))
