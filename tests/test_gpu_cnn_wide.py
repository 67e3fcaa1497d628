"""The network at the sizes whose convolutions take the tiles of 512 voxels (from 2^18 voxels of 16 channels on): a width
below a row of 64 voxels, with a short last tile along every axis, and one above it, whose rows take two tiles and their
halo columns from each other. Bounds as in test_gpu_cnn.py (FP32 and BF16 operands against the FP64 oracle)."""
import pytest
import torch

from oracle import cnn as ocnn
from test_gpu_cnn import H, _inputs, _layer_slices, _params, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("S,B", [(56, 2), (72, 1)])
def test_wide_tiles(S, B, bf16):
    print(f"cnn wide tiles S={S} B={B} bf16={bf16}", flush=True)
    net = H().Cnn(S, max_batch=B, bf16=bf16, seed=2)
    p = _params(31)
    net.set_params(torch.from_numpy(p))
    x, t = _inputs(32, B, S)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y = net.forward(xd).cpu().numpy()
    assert _rel(y, ocnn.forward(p, x)) < (3e-2 if bf16 else 1e-5)
    net.loss_grad(xd, td)
    g = net.grads().numpy()
    _, ref_g = ocnn.loss_and_grad(p, x, t)
    for sl in _layer_slices():
        assert _rel(g[sl], ref_g[sl]) < (1e-1 if bf16 else 1e-3), sl
    net.close()
