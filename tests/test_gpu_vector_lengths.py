"""Inner products and orthogonalisation at vector lengths on both sides of each line of their launch rules (elements per
thread 1, 4, 16), with a last block that is not full."""
import numpy as np
import pytest

from test_gpu_parity import H, _h3, cvec, dev, host, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 5, 7), (63, 64, 65), (64, 64, 64), (127, 128, 64), (128, 128, 64), (101, 103, 105)],
                         ids=lambda s: "x".join(map(str, s)))
def test_inner_products_and_update(shape):
    h, h3 = H(), _h3(shape, 4)
    k0 = 0.5 / max(h3)
    k2 = medium(shape, h3, k0, 7)
    n = int(np.prod(shape))
    ctx = h.helm_setup(dev(k2), h3, 4, "abc", k0)
    x = cvec(n, 3)
    y = host(h.helm_matvec(ctx, dev(x)))
    F = (0.7 - 1.1j) * y + 0.3 * cvec(n, 4) * np.abs(y).max()
    # |x^H y| of n terms: FP64 sums in any order agree to n eps of sum |terms| at most, far less in blocks
    ref = np.vdot(y, F) / np.vdot(y, y).real
    alpha = h.helm_scale_guess(ctx, dev(F), dev(x))
    assert abs(alpha - ref) <= 1e-12 * abs(ref)
    # five steps without a restart: the residual estimate is that of the returned iterate only if every inner product
    # and every update was right (they agree to a few eps times ||A|| ||x|| / ||F||, some hundreds here)
    xs, info = h.helm_gmres_solve(ctx, dev(F), m=8, rtol=1e-30, maxit=5, flexible=True, raise_on_noconv=False)
    assert info["iters"] == 5
    r = F - host(h.helm_matvec(ctx, xs))
    true = np.linalg.norm(r) / np.linalg.norm(F)
    assert abs(true - info["relres_est"]) <= 1e-11
    h.helm_destroy(ctx)


@pytest.mark.parametrize("reorth", [None, "0.9"], ids=["one_pass", "two_passes"])
def test_batch_steps_match_single_solves(reorth, monkeypatch):
    """Batched steps whose inner products come from more blocks than a wave reads in one round (537) and are more in
    number than the reducing block's waves (16), next to a problem of one block; the same with a second Gram-Schmidt pass
    at nearly every step. Both solves stop at 1e-10, so their solutions agree to that times the operator's condition."""
    if reorth:
        monkeypatch.setenv("HELM_CGS_REORTH", reorth)
    h = H()
    ctxs, Fs = [], []
    for shape, seed in (((130, 130, 130), 1), ((9, 11, 10), 2)):
        h3 = _h3(shape, 6)
        k0 = 0.5 / max(h3)
        ctxs.append(h.helm_setup(dev(medium(shape, h3, k0, seed)), h3, 6, "abc", k0))
        Fs.append(dev(cvec(int(np.prod(shape)), seed)))
    xs, infos = h.helm_batch_solve(h.helm_batch_create(ctxs, m=40, prec_fp32=False), Fs, rtol=1e-10)
    assert infos[0]["iters"] > 16
    for ctx, F, x, info in zip(ctxs, Fs, xs, infos):
        x1, single = h.helm_gmres_solve(ctx, F, m=40, rtol=1e-10, flexible=True)
        assert info["converged"] and abs(info["iters"] - single["iters"]) <= 1
        assert (info["cancellations"] > 0) == bool(reorth)
        a, b = host(x), host(x1)
        assert np.linalg.norm(a - b) <= 1e-8 * np.linalg.norm(b)
