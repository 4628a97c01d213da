"""GPU: 2D boxes held in one block's registers for up to 64 steps (resident_kernel) at the edges of
its tiling.

Boxes that fill the wavefronts and lanes and boxes that do not (fewer columns than wavefronts, a share
that does not divide, one row more and less than 64 and 128 lanes), all storage types, calls that are
split unevenly over launches and mixed with single steps, instances that stop inside a launch:
state, per-step force and time average equal calls of one step each, which take the other kernel (the
one that the oracle tests of short runs cover), bit for bit.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_02346_amd as P
    P.lib()
    return P


def problem(shape, stop=0):
    nx, ny = shape
    c0 = 0.5
    p = {"dim": 2, "nx": nx, "ny": ny, "nz": 1, "xbc": "driven", "c0": c0, "rho0": 1.0,
         "center": (0.55 * nx, 0.5 * ny + 0.3), "radius": 1.5, "cp": 0.55, "d": 3.0,
         "rho_a": 1.0, "omega": 2 * np.pi * c0 / nx, "wall_phi": 0.99, "avg_start": 3,
         "max_steps": stop}
    a = 2 * np.pi * (np.arange(96) + 0.5) / 96
    n = np.stack([np.cos(a), np.sin(a), 0.0 * a], 1)
    if min(nx, ny) > 12:  # the surface and its stencil stay inside
        p.update(surf_xyz=np.asarray(p["center"] + (0.0,)) + 3.0 * n, surf_normal=n,
                 surf_area=np.full(96, 2 * np.pi * 3.0 / 96))
    return p


def run(P, probs, storage, calls):
    h = P.LBWave(probs, storage=storage, trace_steps=256)
    for i, p in enumerate(probs):
        h.set_state(i, workloads.random_state(40 + i, p["nx"] * p["ny"], 5))
    for n in calls:
        h.step(n)
    out = ([h.get_state(i) for i in range(h.n)], [h.trace(i, sum(calls)) for i in range(h.n)],
           h.force(allow_empty=True))
    h.close()
    return out


SHAPES = [[(128, 64)], [(128, 63), (127, 64), (113, 20)], [(128, 64), (17, 64), (64, 128)],
          [(64, 127), (63, 65), (64, 128)], [(64, 64), (49, 33), (16, 70)], [(9, 5), (3, 3), (128, 1)]]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("shapes", SHAPES, ids=lambda s: "+".join("%dx%d" % t for t in s))
def test_equal_to_single_steps(P, shapes, storage):
    probs = [problem(s, stop) for s, stop in zip(shapes, (0, 21, 75))]
    a = run(P, probs, storage, [8, 1, 3, 66, 64, 9])
    b = run(P, probs, storage, [1] * 151)
    for x, y in zip(a[0] + a[1], b[0] + b[1]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1])
