"""The right-hand side where a thread takes a column of 16 planes (order 4: from 16384 planes of 256 nodes on) or 4, on a box that is
ragged along every axis and whose last column has one plane. Tolerance as in test_gpu_stencil_chunks.py: FP64 sums of at
most 27 terms, 1e-12 of the largest value."""
import numpy as np
import pytest

from oracle import operators as op
from test_gpu_parity import H, _h3, dev, host, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,complex_k2", [(4, False), (6, False), (6, True)])
def test_columns_of_16(order, complex_k2):
    shape = (257, 66, 260)                        # 9 x 9 column tiles; 257 = 16 x 16 + 1 = 64 x 4 + 1
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


@pytest.mark.parametrize("complex_k2", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("shape", [(61, 70, 250), (101, 60, 88), (257, 256, 250)])
def test_sixth_order_columns(shape, complex_k2):
    """Columns of 4 planes in blocks 64 and 32 nodes wide, and of 16 planes (from 65536 planes on): the first and the last
    planes against the oracle on these planes alone, which every value depends on."""
    h3, k0 = _h3(shape, 6), 21.0
    k2 = medium(shape, h3, k0, 3)
    if complex_k2:
        k2 = k2 * (1 + 0.05j)
    rng = np.random.default_rng(7)
    f = rng.standard_normal([s + 4 for s in shape]) + 1j * rng.standard_normal([s + 4 for s in shape])
    F = host(H().helm_rhs(H().helm_setup(dev(k2), h3, 6, "abc", k0), dev(f))).reshape(shape)
    for a, b in ((0, 18), (shape[0] - 18, shape[0])):
        k2p = k2[a:b + 4]
        ref = op.rhs(6, f[a:b + 4], h3, k2p[2:-2, 2:-2, 2:-2], op.derived_fields(k2p, h3[0]))
        assert np.abs(F[a:b] - ref.reshape(F[a:b].shape)).max() <= 1e-12 * np.abs(ref).max()
