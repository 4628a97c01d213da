"""GPU: run_batch without tuning takes several steps per launch where the boxes allow it, with the
same forces as one step per launch; where they do not (2D, rows that no row block divides) it runs as
before."""
import numpy as np
import pytest

from test_gpu_march import P, problem  # noqa: F401
from test_gpu_resident import problem as problem2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,steps", [([(60, 16, 12)], 2), ([(60, 16, 12), (33, 32, 14)], 2),
                                          ([(60, 16, 12), (33, 20, 14)], 1),
                                          ([(60, 17, 12)], 1), ([(40, 30, 1)], 1)])
def test_untuned_batch(P, shapes, steps):  # noqa: F811
    from paper_2404_02346_amd import surrogate
    probs = []
    for n, s in zip((70, 41), shapes):
        p = problem(s) if s[2] > 1 else problem2(s[:2])
        probs.append(dict(p, n_steps=n))
    r = surrogate.run_batch(probs, autotune=False)
    assert r["variant"][3] == steps
    h = P.LBWave(probs, storage="f32", freeze_at_n_steps=True)
    h.step(70)
    F, n = h.force(allow_empty=True)
    h.close()
    assert np.array_equal(r["F"], F, equal_nan=True) and np.array_equal(r["n_acc"], n)
