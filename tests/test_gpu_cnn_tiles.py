"""The network's kernels at the edges of their tiles: a volume whose levels (40, 20, 10, 5) are no multiple of a tile and
cover every tile width, with rows that cannot be loaded four values at a time (10, 5), and an input that is not aligned
to 16 bytes. Bounds as in test_gpu_cnn.py (FP32 and BF16 operands against the FP64 oracle)."""
import numpy as np
import pytest
import torch

from oracle import cnn as ocnn
from test_gpu_cnn import H, _inputs, _layer_slices, _params, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("S,B", [(40, 1), (40, 3)])
def test_ragged_levels(S, B, bf16):
    print(f"cnn tiles S={S} B={B} bf16={bf16}", flush=True)
    net = H().Cnn(S, max_batch=B, bf16=bf16, seed=2)
    p = _params(21)
    net.set_params(torch.from_numpy(p))
    x, t = _inputs(22, B, S)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y = net.forward(xd).cpu().numpy()
    assert _rel(y, ocnn.forward(p, x)) < (3e-2 if bf16 else 1e-5)
    net.loss_grad(xd, td)
    g = net.grads().numpy()
    _, ref_g = ocnn.loss_and_grad(p, x, t)
    for sl in _layer_slices():
        assert _rel(g[sl], ref_g[sl]) < (1e-1 if bf16 else 1e-3), sl
    # the same input at an odd address: other loads, the same arithmetic
    shifted = torch.empty(xd.numel() + 1, dtype=torch.float32, device="cuda")[1:].view(xd.shape)
    shifted.copy_(xd)
    assert shifted.data_ptr() % 16 == 4
    assert np.array_equal(net.forward(shifted).cpu().numpy(), y)
    net.loss_grad(shifted, td)
    assert np.array_equal(net.grads().numpy(), g)
    net.close()
