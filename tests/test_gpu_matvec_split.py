"""A x and F - A x cut their planes into chunks of their own lengths, by the blocks of each that a CU holds: both forms
compared on boxes where the two lengths differ at order 4 and the last chunks are short, A x with the oracle's rows
(tolerance as in test_gpu_stencil_chunks.py), F - A x with it through the norm of the whole residual."""
import numpy as np
import pytest

from oracle import operators as op
from test_gpu_parity import H, _h3, cvec, dev, host, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [2, 4, 6])
@pytest.mark.parametrize("shape", [(100, 150, 130), (31, 130, 310)])
def test_both_forms(shape, order):
    h3, k0 = _h3(shape, order), 21.0
    k2 = medium(shape, h3, k0, 3)
    n = int(np.prod(shape))
    rng = np.random.default_rng(8)
    ctx = H().helm_setup(dev(k2), h3, order, "abc", k0)
    x, F = cvec(n, 4), cvec(n, 5)
    gs = [op.gamma_abc(k0, h) for h in h3]
    plane = shape[1] * shape[2]
    nodes = np.unique(np.concatenate([rng.integers(0, n, 4000), np.arange(7, n, plane), np.arange(plane - 1, n, plane)]))
    ref = op.sampled_matvec(order, k2, h3, gs, x, nodes)
    y = host(H().helm_matvec(ctx, dev(x)))
    assert np.abs(y[nodes] - ref).max() <= 2e-12 * np.abs(ref).max()
    # the solve reports the norm of its first residual, F - A x at the guess, and is content with it
    _, info = H().helm_gmres_solve(ctx, dev(F), x=dev(x), m=1, maxit=1, rtol=1e30)
    assert info["iters"] == 0
    assert abs(info["relres_true"] - np.linalg.norm(F - y) / np.linalg.norm(F)) <= 1e-12 * info["relres_true"]
