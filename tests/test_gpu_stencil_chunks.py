"""The matvec and the right-hand side where a launch is cut into z-chunks of several planes with a shorter last one (the
small boxes of test_gpu_parity.py get one plane per block), and batches whose runs of right-hand sides on one medium are
longer than a pair. Tolerances: FP64 sums of at most 27 terms, 1e-12 of the largest value, as in test_gpu_parity.py."""
import numpy as np
import pytest

import synth
from oracle import operators as op
from test_gpu_parity import H, _h3, cvec, dev, host, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("complex_k2", [False, True], ids=["real", "complex"])
@pytest.mark.parametrize("order", [2, 4, 6])
def test_long_chunks(order, complex_k2):
    shape = (151, 70, 200)                        # 36 column tiles: 7 chunks of 22 planes, the last of 19
    h3, k0 = _h3(shape, order), 21.0
    k2 = medium(shape, h3, k0, 3)
    if complex_k2:
        k2 = k2 * (1 + 0.05j)
    n = int(np.prod(shape))
    rng = np.random.default_rng(5)
    f = rng.standard_normal([s + 4 for s in shape]) + 1j * rng.standard_normal([s + 4 for s in shape])
    ctx = H().helm_setup(dev(k2), h3, order, "abc", k0)
    x = cvec(n, 4)
    y = host(H().helm_matvec(ctx, dev(x)))
    gs = [op.gamma_abc(k0, h) for h in h3]
    nodes = np.unique(np.concatenate([rng.integers(0, n, 4000), np.arange(0, n, 70 * 200), np.arange(70 * 200 - 1, n, 70 * 200)]))
    ref = op.sampled_matvec(order, k2, h3, gs, x, nodes)
    assert np.abs(y[nodes] - ref).max() <= 2e-12 * np.abs(ref).max()    # the largest of the sampled rows
    F = host(H().helm_rhs(ctx, dev(f)))
    k2i = k2[2:-2, 2:-2, 2:-2]
    fields = op.derived_fields(k2, h3[0]) if order == 6 else None
    Fr = op.rhs(order, f, h3, k2i, fields).ravel()
    assert np.abs(F - Fr).max() <= 1e-12 * np.abs(Fr).max()


def test_batch_runs_of_one_medium():
    """Three right-hand sides, one and two on three media in one batch, each against its own solve."""
    h = H()
    ctxs, Fs = [], []
    for n, seed, count in ((14, 1, 3), (18, 2, 1), (16, 3, 2)):
        k0, hh = 0.45 * (n + 1), 1.0 / (n + 1)
        k2 = synth.inclusions_k2(n, k0, seed=seed)
        ctx = h.helm_setup(dev(k2), hh, 6, k0=k0)
        for f in synth.plane_wave_sources(k2, k0, synth.unit_directions(count, seed=seed)):
            ctxs.append(ctx)
            Fs.append(h.helm_rhs(ctx, dev(f)))
    xs, infos = h.helm_batch_solve(h.helm_batch_create(ctxs, m=20, prec_fp32=False), Fs, rtol=1e-10)
    for ctx, F, x, info in zip(ctxs, Fs, xs, infos):
        x1, single = h.helm_gmres_solve(ctx, F, m=20, rtol=1e-10, flexible=True)
        assert info["converged"] and abs(info["iters"] - single["iters"]) <= 1
        a, b = host(x), host(x1)
        assert np.linalg.norm(a - b) <= 1e-8 * np.linalg.norm(b)
