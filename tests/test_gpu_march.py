"""GPU: several lattice steps per launch (march_kernel) at the edges of its tiling.

Rows of 1 to 4 wavefronts and strips (252 owned cells) with partial last strips, row blocks that
end past ny, boxes of fewer planes than the halo, chunks of unequal length, and blocks of eight
wavefronts (handles larger than the memory-side cache): state, per-step force and time average
must equal one step per launch bit for bit, for step counts that leave 0, 1 and 2 steps over.
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


def problem(shape, surf=True):
    nx, ny, nz = shape
    c0 = 0.45
    p = {"dim": 3, "nx": nx, "ny": ny, "nz": nz, "xbc": "driven", "c0": c0, "rho0": 1.0,
         "center": (0.55 * nx, ny / 2.0 + 0.3, nz / 2.0 - 0.2), "radius": 2.0, "cp": 0.55, "d": 4.0,
         "rho_a": 1.0, "omega": 2 * np.pi * c0 / nx, "wall_phi": 0.99, "avg_start": 3}
    if surf:
        xyz, nrm, area = workloads.fibonacci_surface(p["center"], 4.0, 96)
        p.update(surf_xyz=xyz, surf_normal=nrm, surf_area=area)
    return p


def state(h, i):
    import torch
    v, p = h.state_view(i), h.problems[i]
    raw = h.ws[v.offset_bytes: v.offset_bytes + 7 * v.plane_bytes]
    kind = {2: torch.int16, 4: torch.float32, 8: torch.float64}[v.elem_bytes]
    return raw.view(kind).as_strided((7, p["nz"], p["ny"], p["nx"]),
                                     (v.plane_bytes // v.elem_bytes, p["ny"] * v.pitch, v.pitch, 1))


def run(P, probs, storage, spl, steps, graph, random=True):
    h = P.LBWave(probs, storage=storage, trace_steps=64)
    h.set_steps_per_launch(spl)
    h.set_graph(graph)
    if random:
        for i, p in enumerate(probs):
            h.set_state(i, workloads.random_state(40 + i, p["nx"] * p["ny"] * p["nz"], 7))
    for n in steps:
        h.step(n)
    out = ([state(h, i).clone() for i in range(h.n)], [h.trace(i, sum(steps)) for i in range(h.n)],
           h.force(allow_empty=True))
    h.close()
    return out


def same(a, b):
    import torch
    for x, y in zip(a[0], b[0]):
        assert torch.equal(x, y)
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(64, 32, 1), (65, 24, 2), (192, 12, 3), (129, 8, 11),
                                   (252, 20, 13), (257, 12, 9), (505, 16, 5)])
def test_edges_of_the_tiling(P, storage, shape):
    print(f"march vs one step, {storage}, {shape}", flush=True)
    p = problem(shape, surf=min(shape[1:]) > 11)
    for steps, graph in (((13,), 0), ((14, 15), 0), ((33,), 10)):
        same(run(P, [p], storage, 2, steps, graph), run(P, [p], storage, 1, steps, graph))


@pytest.mark.parametrize("storage,shape", [("f32", (256, 96, 200)), ("f64", (256, 96, 100)),
                                           ("f32", (700, 52, 140))])
def test_blocks_of_eight_wavefronts(P, storage, shape):
    print(f"march vs one step, blocks of 8 wavefronts, {storage}, {shape}", flush=True)
    p = problem(shape)
    same(run(P, [p], storage, 2, (20,), 0, random=False),
         run(P, [p], storage, 1, (20,), 0, random=False))


@pytest.mark.parametrize("storage,shapes,depth", [
    ("f16", [(257, 12, 150)] * 40, 3), ("bf16", [(65, 12, 40), (257, 12, 150)] + [(257, 12, 150)] * 38, 3),
    ("f16", [(96, 16, 96)], 2), ("bf16", [(60, 16, 31)] * 3, 2)])
def test_steps_of_a_launch_in_16_bit(P, storage, shapes, depth):
    print(f"march vs one step, {storage}, {len(shapes)} boxes, {depth} steps a launch", flush=True)
    probs = [problem(s, surf=False) for s in shapes]
    h = P.LBWave(probs, storage=storage)
    h.set_steps_per_launch(2)
    assert h.launch_steps() == depth
    h.close()
    same(run(P, probs, storage, 2, (13,), 0, random=False),
         run(P, probs, storage, 1, (13,), 0, random=False))
