"""GPU: the 2D resident kernel over every share of columns that a wavefront can have (0 to 8, even and
uneven over the wavefronts), rows that fill the lanes and rows that do not, and boxes that fill all three
of its tiles: state, per-step force and time average equal calls of one step each, bit for bit.
"""
import numpy as np
import pytest

from test_gpu_resident import P, problem, run  # noqa: F401

pytestmark = pytest.mark.gpu

WIDTHS = [(5, 31, 47, 63), (16, 33, 48, 64), (50, 65, 79, 96), (97, 100, 111, 113), (119, 126, 127, 128)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("widths", WIDTHS, ids=lambda w: "+".join(map(str, w)))
def test_every_share_of_columns(P, widths, storage):  # noqa: F811
    for rows in ([64, 17, 63, 33], [128, 128, 66, 127]):
        shapes = [(nx, ny) for nx, ny in zip(widths, rows) if ny <= 64 or nx <= 64]
        if not shapes:
            continue
        print(f"{storage}, {shapes}", flush=True)
        probs = [problem(s) for s in shapes]
        a, b = run(P, probs, storage, [20, 8, 65, 1]), run(P, probs, storage, [1] * 94)
        assert all(np.abs(f).max() > 0 for f in b[0])
        for x, y in zip(a[0] + a[1], b[0] + b[1]):
            assert np.array_equal(x, y)
        assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1])
