"""Limits of the 2D resident kernel, seen through the workspace size (128 slots of moment boxes and
partial sums with it, 8 without): the partial sums count towards the 8 GiB that its slots may take, and
one launch's surface blocks (of 64 steps) must fit a grid of less than 2^32 threads.
"""
import ctypes

import numpy as np
import pytest

from test_gpu_resident import problem


def bytes_per_box(n, points):
    """Workspace bytes per box of n equal FP32 boxes of 9 x 5 cells with one surface of coincident
    points, which meets 3 x 3 cells (256 bytes of moments per slot, 32 per 64 points of sums)."""
    import paper_2404_02346_amd as P
    p = dict(problem((9, 5)), surf_xyz=np.tile([4.0, 2.0, 0.0], (points, 1)),
             surf_normal=np.tile([1.0, 0.0, 0.0], (points, 1)), surf_area=np.ones(points))
    one, keep = P.make_descs([p], "f32")
    arr = (type(one[0]) * n).from_buffer_copy(bytes(one) * n)
    assert ctypes.sizeof(arr) == n * ctypes.sizeof(one[0])
    size = P.lib().lb_wave_workspace_bytes(arr, n)
    assert size > 0
    del keep
    return size / n


@pytest.mark.parametrize("n,resident", [(1000, True), (200000, True), (240000, False), (262144, False)])
def test_slots_of_moments_and_sums_are_bounded(n, resident):
    # 64 MiB a slot: 256 + 32 bytes a box allow 233016 of them, 256 alone 262144
    with_surface, without = bytes_per_box(n, 1), bytes_per_box(n, 0)
    assert (with_surface - without > 100 * 256) == resident


@pytest.mark.parametrize("points,resident", [(250000, True), (262400, False)])
def test_surface_blocks_of_a_launch_fit_a_grid(points, resident):
    # 64 boxes: 64 * 64 steps * points / 64 blocks of 256 threads; besides its sums, a surface point
    # takes a record of 136 bytes
    sums = 32 * ((points + 63) // 64)
    extra = bytes_per_box(64, points) - bytes_per_box(64, 0) - 136 * points
    assert (extra > 100 * sums) == resident
