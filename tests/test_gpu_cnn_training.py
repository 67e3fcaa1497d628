"""Training is reproduced beyond its first step: the sums of the gradients are made in the order they always had, so
that the same inputs give the same parameters to the bit. The stored values and the reason are described in
golden/make_cnn_training.py."""
import os

import numpy as np
import pytest

from golden import make_cnn_training as gold

pytestmark = pytest.mark.gpu
STORED = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "cnn_training.npz")


@pytest.mark.parametrize("S,B,bf16", gold.CASES)
def test_training_reproduces_the_stored_run(S, B, bf16):
    print(f"cnn training S={S} B={B} bf16={bf16}", flush=True)
    with np.load(STORED) as ref:
        for k, v in gold.run(S, B, bf16).items():
            assert np.array_equal(v, ref["%d_%d_%d_%s" % (S, B, bf16, k)]), k
