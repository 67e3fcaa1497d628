"""The 1D eigen-decomposition never hands out a NaN: corner entries whose squares leave the range of a double either give
a decomposition that holds or are refused by its checks (HELM_ENUMERIC). Runs on the CPU."""
import math

import numpy as np
import pytest

from paper_2602_07711_amd import helm

GAMMAS = [0.0, 1e-300, 1e-160j, 1e80, 1e150j, 1e200, 1e200j, complex(1e300, 1e300), math.inf, complex(0, math.inf), math.nan]


@pytest.mark.parametrize("zeta", [1.0, 2.0])
@pytest.mark.parametrize("n", [2, 3, 5, 8, 16])
def test_extreme_corners(n, zeta):
    for gamma in GAMMAS:
        try:
            d, V, Vinv = (np.asarray(a) for a in helm.helm_eig1d(n, complex(gamma), zeta))
        except helm.HelmError as e:
            assert "ENUMERIC" in str(e) and not abs(gamma) < 1e70, gamma
            continue
        assert all(np.isfinite(a).all() for a in (d, V, Vinv)), gamma
        L = np.diag(np.ones(n - 1), 1).astype(complex) + np.diag(np.ones(n - 1), -1)
        L[0, 0] += gamma
        L[-1, -1] += gamma
        L[0, 1] = L[-1, -2] = zeta
        assert np.abs(L @ V - V * d).max() <= 1e-10 * np.abs(L).max() * np.abs(V).max(), gamma
        assert np.abs(Vinv @ V - np.eye(n)).max() <= 1e-8, gamma
