"""The folded transforms where the two halves of an axis need different numbers of 16-wide mode blocks (129: 65 and 64,
33: 17 and 16), where the last tile of modes is short (97: 49, 200: 100) and where a tile of columns spans several slices,
with complex and real blocks and every tile configuration. Bounds of test_gpu_parity.py."""
import numpy as np
import pytest

from oracle import operators as op
from oracle import precond as pc
from test_gpu_parity import H, TOL32_PFFT, cvec, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(5, 33, 129), (4, 129, 33), (6, 97, 200), (3, 200, 97), (3, 3, 4)])
def test_mode_blocks(shape, fp32):
    hh = 1.0 / (max(shape) + 1)
    h3, k0 = (hh,) * 3, 0.47 / hh
    ctx = H().helm_setup(dev(np.full(tuple(s + 4 for s in shape), k0 * k0)), h3, 4, k0=k0, shape=shape)
    y = cvec(int(np.prod(shape)), 31)
    ref = pc.EigT(shape, h3, k0, (op.gamma_abc(k0, hh),) * 3).solve(y)
    for kind, tol in (("eigt", 1e-5 if fp32 else 1e-11), ("pfft", TOL32_PFFT if fp32 else 1e-11)):
        for cfg in range(4) if kind == "eigt" else (0,):
            for k in ("x32", "y32") if fp32 else ("x64", "y64"):
                H().helm_gemm_config(ctx, k, cfg)
            z = host(H().helm_precond_apply(ctx, dev(y), kind=kind, fp32=fp32))
            err = np.linalg.norm(z - ref) / np.linalg.norm(ref)
            assert err <= tol, (kind, cfg, err)
