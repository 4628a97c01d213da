"""GPU: every plan of several steps per launch (steps per launch x wavefronts per block) against one
step per launch, bit for bit, from random populations.

One handle holds rows of one to four wavefronts (with three, a block has wavefronts without cells)
and rows cut into strips, with the object, its sound-speed box and its surface across a wavefront
or strip edge, row blocks that end past ny, and boxes of as many planes as leave chunks of unequal
length.  State, per-step force and time average are compared; they are not zero.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

PLANS = {"f64": [(2, 4), (2, 8)], "f32": [(2, 4), (2, 8), (3, 4), (3, 8)],
         "f16": [(2, 4), (3, 4)], "bf16": [(2, 4), (3, 4)]}
# (nx, ny, nz), centre x of the object
BOXES = [((60, 16, 13), 30.0), ((127, 24, 14), 63.6), ((180, 20, 13), 128.2), ((256, 16, 17), 191.7),
         ((300, 20, 13), 252.3), ((520, 16, 12), 255.8), ((520, 12, 19), 503.6)]


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_02346_amd as P
    P.lib()
    return P


def problem(shape, cx, stop=0):
    nx, ny, nz = shape
    c0 = 0.45
    center = (cx, ny / 2.0 + 0.3, nz / 2.0 - 0.2)
    xyz, nrm, area = workloads.fibonacci_surface(center, 3.5, 96)
    return {"dim": 3, "nx": nx, "ny": ny, "nz": nz, "xbc": "driven", "c0": c0, "rho0": 1.0,
            "center": center, "radius": 2.0, "cp": 0.55, "d": 4.0, "rho_a": 1.0,
            "omega": 2 * np.pi * c0 / nx, "wall_phi": 0.99, "avg_start": 3, "max_steps": stop,
            "surf_xyz": xyz, "surf_normal": nrm, "surf_area": area}


def run(P, probs, storage, plan, calls, graph):
    h = P.LBWave(probs, storage=storage, trace_steps=64)
    if plan:
        h.set_steps_per_launch(2)
        h.set_launch_plan(*plan)
        assert h.launch_plan() == plan and h.launch_steps() == plan[0]
    h.set_graph(graph)
    for i, p in enumerate(probs):
        h.set_state(i, workloads.random_state(90 + i, p["nx"] * p["ny"] * p["nz"], 7))
    for n in calls:
        h.step(n)
    out = ([h.get_state(i) for i in range(h.n)], [h.trace(i, sum(calls)) for i in range(h.n)],
           *h.force())
    h.close()
    return out


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("stops", [False, True])
def test_every_plan_gives_the_bits_of_one_step(P, storage, stops):
    # in the second case instances stop inside what would be a launch
    probs = [problem(s, cx, (0, 17, 0, 23, 12, 0, 31)[i] if stops else 0)
             for i, (s, cx) in enumerate(BOXES)]
    calls, graph = ((13, 20), 12) if stops else ((19,), 0)
    ref = run(P, probs, storage, None, calls, graph)
    for f, tr in zip(ref[0], ref[1]):
        assert np.all(np.abs(f).max(axis=0) > 0) and np.all(tr[1:12, 0] != 0)
    for plan in PLANS[storage]:
        print(f"{storage}, {plan[0]} steps, {plan[1]} wavefronts, stops {stops}", flush=True)
        got = run(P, probs, storage, plan, calls, graph)
        for x, y in zip(got[0] + got[1], ref[0] + ref[1]):
            assert np.array_equal(x, y)
        assert np.array_equal(got[2], ref[2]) and np.array_equal(got[3], ref[3])


def test_plans_that_do_not_apply_are_refused(P):
    h = P.LBWave([problem(*BOXES[0])], storage="f16")
    before = h.launch_plan()
    for plan in ((1, 4), (4, 4), (2, 8), (2, 6), (0, 0)):
        with pytest.raises(P.LBError):
            h.set_launch_plan(*plan)
        assert h.launch_plan() == before
    assert h.launch_steps() == 1  # a plan alone does not turn several steps on
    h.close()
    h = P.LBWave([problem((60, 18, 13), 30.0)], storage="f32")  # rows that no row block divides
    assert h.launch_plan() == (1, 0)
    with pytest.raises(P.LBError):
        h.set_launch_plan(2, 4)
    h.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_autotune_takes_a_plan_and_resets(P, storage):
    probs = [problem(*b) for b in BOXES[:3]]
    ref = run(P, probs, storage, None, (20,), 0)
    h = P.LBWave(probs, storage=storage, trace_steps=64)
    assert h.autotune(4) > 0 and h.t == 0
    assert h.launch_plan() in PLANS[storage]
    assert h.launch_steps() == (h.launch_plan()[0] if h.steps_per_launch() == 2 else 1)
    for i, p in enumerate(probs):
        h.set_state(i, workloads.random_state(90 + i, p["nx"] * p["ny"] * p["nz"], 7))
    h.step(20)
    for i in range(h.n):
        assert np.array_equal(h.get_state(i), ref[0][i]) and np.array_equal(h.trace(i, 20), ref[1][i])
    assert np.array_equal(h.force()[0], ref[2])
    h.close()


@pytest.mark.parametrize("storage,shape,n,steps", [
    ("f32", (128, 128, 128), 1, 2), ("f32", (1456, 32, 32), 1, 2), ("f32", (64, 64, 64), 1, 2),
    ("f32", (128, 128, 128), 4, 3), ("f32", (192, 192, 192), 1, 3), ("f16", (192, 192, 192), 1, 2)])
def test_untuned_steps_per_launch(P, storage, shape, n, steps):
    # the faster of two and three steps where they differ by more than a tenth
    h = P.LBWave([dict(problem(shape, 0.5 * shape[0]))] * n, storage=storage)
    assert h.launch_plan()[0] == steps
    h.close()
