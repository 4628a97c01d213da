"""GPU: several steps per launch (march_kernel) with a sound-speed table of more than 4 GiB.

c varies over a whole FP64 lattice of 1024 x 512 x 1025 cells, so the c^2 table holds 2^29 + 2^19 cells
of 8 bytes and the cells of the last plane lie past a 32-bit byte offset.  c repeats every seven
planes, which 1024 is no multiple of: a wrapped offset takes another c.  Seeded random populations;
two steps in one launch must equal two one-step launches bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NX, NY, NZ = 1024, 512, 1025


def test_table_larger_than_32_bit_offsets():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 72 << 30:
        pytest.skip("needs 72 GiB of free GPU memory")
    import paper_2404_02346_amd as P
    plane = (np.arange(NY)[:, None] * 3 + np.arange(NX)[None, :] * 5) % 11
    field = np.empty((NZ, NY, NX))
    for z in range(NZ):
        field[z] = 0.30 + 0.02 * (z % 7) + 0.005 * plane
    p = {"dim": 3, "nx": NX, "ny": NY, "nz": NZ, "xbc": "driven", "c0": 0.5, "rho0": 1.0,
         "c_field": field, "rho_a": 1.0, "omega": 0.01, "wall_phi": 0.99}
    h = P.LBWave([p], storage="f64")
    del field, p["c_field"]
    rows = [NZ - 3, NZ - 2, NZ - 1, 0, 1, 2]  # the planes beyond the offset and their neighbours

    def populations():
        v = h.state_view(0)
        raw = h.ws[v.offset_bytes: v.offset_bytes + 7 * v.plane_bytes].view(torch.float64)
        return raw.as_strided((7, NZ, NY, NX), (v.plane_bytes // 8, NY * v.pitch, v.pitch, 1))

    def two_steps(per_launch):
        h.reset()
        torch.cuda.manual_seed(7)
        f = populations()
        for z in rows:
            f[:, z] = torch.empty((7, NY, NX), dtype=torch.float64, device="cuda").uniform_(-0.1, 0.1)
        h.set_steps_per_launch(per_launch)
        h.step(2)
        return populations()[:, rows].clone()

    print("FP64, c varies over 1024 x 512 x 1025 cells", flush=True)
    one = two_steps(1)
    assert bool((one[:, 2] != 0).any())
    assert torch.equal(two_steps(2), one)
    h.close()
    del h
    torch.cuda.empty_cache()
