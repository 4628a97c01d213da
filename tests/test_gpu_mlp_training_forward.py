"""GPU: the training forward (lb_mlp_forward_layered, the forward half of the training kernel) against
the inference kernels of every batch size, bit for bit; it leaves gradients as they are.
"""
import numpy as np
import pytest

from test_gpu_mlp_batches import S, inputs  # noqa: F401

pytestmark = pytest.mark.gpu


def test_training_forward_matches_every_inference_kernel(S):  # noqa: F811
    # inference: 16 samples per block to 4096, 32 to 24576, 128 above; training: 32, padded to 64
    x = inputs(24640, 9)
    net = S.MLP(max_batch=24640, seed=4)
    for n in (1, 31, 33, 64, 4096, 4097, 24576, 24577, 24640):
        print(f"batch {n}", flush=True)
        y = net.predict(x[:n])
        assert np.any(y != 0) and np.array_equal(net.predict(x[:n], layered=True), y)
    t = np.sin(3 * x[:200, 0]).astype(np.float32)
    before = net.grad(x[:200], t)
    net.predict(x, layered=True)
    after = net.grad(x[:200], t)
    assert before[0] == after[0] and np.array_equal(before[1], after[1])
    net.close()
