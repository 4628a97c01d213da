"""GPU: lb_wave_autotune times what a long call runs, and leaves a handle at rest.

2D boxes that run many steps per launch in long calls: the reported time per step is that of such a
call (a launch per step takes more than twice as long), for trials of any length.  Handles with
instances that stop within the trial, and with graph replay switched on before, are tuned too and
then give the results of an untuned handle bit for bit.
"""
import time

import numpy as np
import pytest

from test_gpu_launch_plans import BOXES, problem
from test_gpu_resident import problem as problem2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_02346_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n_trial", [2, 6, 40])
def test_reported_time_is_that_of_a_long_call(P, n_trial):
    import torch
    h = P.LBWave([problem2((128, 64))], storage="f64")
    ms = h.autotune(n_trial)
    h.step(1280)
    torch.cuda.synchronize()
    t = time.perf_counter()
    h.step(6400)
    torch.cuda.synchronize()
    per = (time.perf_counter() - t) / 6400 * 1e3
    h.close()
    print(f"autotune({n_trial}): {1e3 * ms:.2f} us, 6400 steps: {1e3 * per:.2f} us per step")
    assert 0.6 * per < ms < 1.6 * per


@pytest.mark.parametrize("dim,storage", [(2, "f64"), (2, "f16"), (3, "f32"), (3, "f16")])
@pytest.mark.parametrize("graph", [0, 12])
def test_results_after_tuning(P, dim, storage, graph):
    stops = (0, 9, 21)
    if dim == 2:
        probs = [problem2(s, stop) for s, stop in zip([(128, 64), (70, 33), (64, 128)], stops)]
    else:
        probs = [problem(*b, stop) for b, stop in zip(BOXES[:3], stops)]
    out = []
    for tuned in (False, True):
        h = P.LBWave(probs, storage=storage, trace_steps=64)
        if tuned:
            h.set_graph(graph)
            assert h.autotune(8) > 0 and h.t == 0
            for i in range(h.n):
                assert not h.get_state(i).any() and not h.trace(i, 64).any()
        for n in (3, 40):
            h.step(n)
        out.append([h.get_state(i) for i in range(h.n)] + [h.trace(i, 43) for i in range(h.n)]
                   + list(h.force(allow_empty=True)))
        h.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)
