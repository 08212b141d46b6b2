"""How many partial results the Gram matrix of a wide dense A is cut into: a
last diagonal tile of one 16-column block does little work a row step but waits
as long as any, so its slabs have to be as short as its steps are slow."""
import ctypes

import pytest

from paper_2203_02798_amd import _lib as L


@pytest.mark.parametrize("d,items", [
    # tiles x slabs: off-diagonal, off-diagonal in the last column, diagonal, last
    (836, 78 * 21 + 13 * 13 + 13 * 13 + 5), (849, 78 * 21 + 13 * 15 + 13 * 13 + 7),
    (870, 78 * 20 + 13 * 18 + 13 * 13 + 10), (896, 91 * 20 + 14 * 12)])
def test_partials_planned(d, items):
    m = L.PskMat(format=L.PSK_DENSE, dtype=L.PSK_F64, n=120000, d=d, ld=d)
    out = ctypes.c_size_t()
    assert L.lib().psk_workspace_size(L.PSK_OP_GRAM, ctypes.byref(m), 0, 1, 1, 0,
                                      ctypes.byref(out)) == 0
    assert out.value == items * 64 * 64 * 8 + 256
