"""The moment boxes that the 2D resident kernel keeps for the steps of two launches take at most 8 GiB:
handles of more boxes fall back to the small workspace of one step per launch."""
import pytest

from test_gpu_resident import problem


@pytest.mark.parametrize("n,slots", [(1, 128), (512, 128), (32768, 8)])
def test_moment_boxes_are_bounded(n, slots):
    import paper_2404_02346_amd as P
    p = problem((128, 64))
    size = {}
    for surf in (True, False):
        q = dict(p)
        if not surf:
            for k in ("surf_xyz", "surf_normal", "surf_area"):
                del q[k]
        arr, keep = P.make_descs([q] * n, "f64")
        size[surf] = P.lib().lb_wave_workspace_bytes(arr, n) / n
    # the surface of radius 3 with its stencils meets 9 x 9 cells at most, 7 x 7 at least; 32 bytes
    # a cell and slot, 2 x 32 bytes of partial sums, and 96 surface points of less than 256 bytes
    per_slot = (size[True] - size[False]) / slots
    assert 49 * 32 < per_slot < 81 * 32 + 64 + 256 + 96 * 256 / slots
