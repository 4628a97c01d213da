"""GPU: the cavity calibration at the widths where its kernel changes, against the FP64 oracle.

One wavefront with 1, 2 or 4 cells to a lane up to 64, 128 and 256 cells; a wavefront per 224
cells with a halo of 16 above.  Bounds as for the other calibration test (FP64 on both sides, the
same steps): 1e-10 of the largest amplitude.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_02346_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("nx", [16, 63, 64, 65, 127, 128, 129, 255, 256, 257, 448, 449, 1121, 2048])
def test_widths(P, nx):
    import oracle as orc
    om = 2 * np.pi * 0.5 / nx
    n = 6 if nx > 1000 else 12
    print(f"cavity of {nx} cells", flush=True)
    ref = orc.cavity_calibration(nx, 0.5, om, n_periods=n, n_fit=2)
    got = P.cavity_calibrate(nx, 0.5, om, n_periods=n, n_fit=2)
    assert np.abs(got["P"] - ref["P"]).max() <= 1e-10 * np.abs(ref["P"]).max()
    assert got["A"] == pytest.approx(ref["A"], rel=1e-10)
