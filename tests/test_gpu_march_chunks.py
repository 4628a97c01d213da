"""GPU: several steps per launch where a block marches through many planes: boxes of 97 planes, a prime,
so that the chunks of every plan but the trivial ones differ in length, as many boxes as give long
chunks, every one from random populations, with the object across the middle.  State, per-step force
and average equal one step per launch, bit for bit, for every plan.
"""
import numpy as np
import pytest

from test_gpu_launch_plans import P, PLANS, problem  # noqa: F401

pytestmark = pytest.mark.gpu


def run(P, probs, storage, plan):  # noqa: F811
    import torch
    kind = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16,
            "bf16": torch.bfloat16}[storage]
    h = P.LBWave(probs, storage=storage, trace_steps=16)
    if plan:
        h.set_steps_per_launch(2)
        h.set_launch_plan(*plan)

    def populations(i):
        v, p = h.state_view(i), probs[i]
        raw = h.ws[v.offset_bytes: v.offset_bytes + 7 * v.plane_bytes].view(kind)
        return raw.as_strided((7, p["nz"], p["ny"], p["nx"]),
                              (v.plane_bytes // v.elem_bytes, p["ny"] * v.pitch, v.pitch, 1))

    torch.cuda.manual_seed(5)
    for i, p in enumerate(probs):
        populations(i).copy_(0.2 * torch.rand((7, p["nz"], p["ny"], p["nx"]), device="cuda",
                                              dtype=torch.float32) - 0.1)
    h.step(11)  # leaves 2 steps over three at a time, 1 over two
    out = ([populations(i).clone() for i in range(h.n)], [h.trace(i, 11) for i in range(h.n)],
           h.force()[0])
    h.close()
    return out


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("shapes", [[(256, 64, 97)] * 16, [(500, 64, 97)] * 8, [(150, 32, 97)] * 24,
                                    [(60, 32, 97), (100, 32, 97), (190, 32, 97), (256, 32, 97)] * 8])
def test_chunks_of_unequal_length(P, shapes, storage):  # noqa: F811
    import torch
    probs = [problem(s, 0.5 * s[0]) for s in shapes]
    ref = run(P, probs, storage, None)
    assert all(bool((f != 0).any()) for f in ref[0]) and all(np.all(t[1:, 0] != 0) for t in ref[1])
    for plan in PLANS[storage]:
        print(f"{storage}, {len(shapes)} boxes of {shapes[0]}, plan {plan}", flush=True)
        got = run(P, probs, storage, plan)
        for x, y in zip(got[0], ref[0]):
            assert torch.equal(x, y)
        for x, y in zip(got[1], ref[1]):
            assert np.array_equal(x, y)
        assert np.array_equal(got[2], ref[2])
