"""GPU: the network's kernels at the batch sizes where they change.

Inference runs 16, 32 or 128 samples per block by batch size: a sample's output must not depend on
which.  Gradients at batches around the 32- and 64-sample blocks and the chunks of the weight
gradients, against the FP64 oracle (same bound as the other gradient tests: a few BF16 roundings
of 2^-8 through five layers, 2e-2 in the 2-norm).
"""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_02346_amd import surrogate as S
    return S


def inputs(n, seed):
    return np.random.Generator(np.random.PCG64(seed)).uniform(-1, 1, (n, 4)).astype(np.float32)


def test_outputs_do_not_depend_on_the_batch_size(S):
    x = inputs(24600, 5)
    net = S.MLP(max_batch=4100, seed=3)
    whole = net.predict(x)                      # 128 samples per block
    assert np.isfinite(whole).all()
    for n in (1, 15, 16, 17, 31, 33, 4096, 4097, 24576, 24577):
        print(f"batch {n}", flush=True)
        assert np.array_equal(net.predict(x[:n]), whole[:n])
        if n <= 4100:
            assert np.array_equal(net.predict(x[:n], layered=True), whole[:n])
    net.close()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 129, 1000])
def test_gradients_at_block_edges(S, n):
    print(f"gradients of {n} samples", flush=True)
    x = inputs(n, 7)
    t = (1.0 + 0.5 * np.sin(3 * x[:, 0])).astype(np.float32)  # well away from the outputs near 0
    p = S.init_params(11)
    net = S.MLP(max_batch=1000, params=p)
    loss, g = net.grad(x, t)
    net.close()
    pr, off = p.astype(np.float64), 0   # the oracle takes the BF16-rounded weights and inputs
    for k, m in zip(M.DIMS[:-1], M.DIMS[1:]):
        pr[off: off + m * k] = M.bf16_round(pr[off: off + m * k])
        off += m * k + m
    lref, gref = M.loss_and_grad(pr, M.bf16_round(x), t)
    assert loss == pytest.approx(lref, rel=2e-2)
    assert np.linalg.norm(g - gref) < 2e-2 * np.linalg.norm(gref)
