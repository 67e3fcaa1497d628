"""Write what the network's training steps give (stored expected values): gradients of the first step, and gradients and
parameters after three Adam steps, every 211th value, for widths below, at and above a row of 64 voxels and both operand
types.

Adam's step is the gradient over its own size, so gradients near zero whose last bit changes become another step, and
the next step's gradients differ by 1e-3 and more, although each is as near to the 64-bit values as before. A training
run is therefore only reproduced when every sum is made in the same order; no oracle can say which. The stored values are
those of the network's first weight-gradient kernel (commit ef00809, 8 x 8 x 4 tiles strided over the tile groups).
Regenerate, on an MI355X, from the root of a tree with that kernel built:
    PYTHONPATH=<tree> python tests/golden/make_cnn_training.py OUT.npz
"""
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.append(ROOT)

CASES = [(24, 1, 0), (24, 3, 1), (56, 2, 0), (64, 1, 1), (72, 1, 1)]   # width, batch, BF16 operands
STRIDE, STEPS, LR = 211, 3, 1e-3


def run(S, B, bf16):
    import torch

    import paper_2602_07711_amd as H
    rng = np.random.default_rng(100 * S + B)
    x, t = (torch.from_numpy(rng.standard_normal((B, 2, S ** 3)).astype(np.float32)).cuda() for _ in range(2))
    net = H.Cnn(S, max_batch=B, bf16=bool(bf16), seed=3)
    loss = net.loss_grad(x, t)
    out = {"loss": np.array([loss]), "first": net.grads().numpy()[::STRIDE].copy()}
    for _ in range(STEPS):
        net.train_step(x, t, LR)
    out["later"] = net.grads().numpy()[::STRIDE].copy()
    out["params"] = net.params().numpy()[::STRIDE].copy()
    net.close()
    return out


if __name__ == "__main__":
    res = {}
    for case in CASES:
        print("training", case, flush=True)
        for k, v in run(*case).items():
            res["%d_%d_%d_%s" % (*case, k)] = v
    np.savez_compressed(sys.argv[1], **res)
    print("wrote", sys.argv[1])
