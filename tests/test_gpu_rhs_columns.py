"""The right-hand side where a thread takes a column of 16 planes (from 16384 planes of 64 x 4 nodes on), on a box that is
ragged along every axis and whose last column has one plane. Tolerance as in test_gpu_stencil_chunks.py: FP64 sums of at
most 27 terms, 1e-12 of the largest value."""
import numpy as np
import pytest

from oracle import operators as op
from test_gpu_parity import H, _h3, dev, host, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,complex_k2", [(4, False), (6, False), (6, True)])
def test_columns_of_16(order, complex_k2):
    shape = (257, 66, 260)                        # 5 x 17 column tiles, 16 columns of 16 planes and one of 1
    h3, k0 = _h3(shape, order), 21.0
    k2 = medium(shape, h3, k0, 3)
    if complex_k2:
        k2 = k2 * (1 + 0.05j)
    rng = np.random.default_rng(6)
    f = rng.standard_normal([s + 4 for s in shape]) + 1j * rng.standard_normal([s + 4 for s in shape])
    ctx = H().helm_setup(dev(k2), h3, order, "abc", k0)
    F = host(H().helm_rhs(ctx, dev(f)))
    fields = op.derived_fields(k2, h3[0]) if order == 6 else None
    ref = op.rhs(order, f, h3, k2[2:-2, 2:-2, 2:-2], fields).ravel()
    assert np.abs(F - ref).max() <= 1e-12 * np.abs(ref).max()
