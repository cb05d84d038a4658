"""Grids whose pair of f buffers is larger than the last-level cache: the FP32
fused kernel requests four rows ahead there.  Bitwise as in separate kernels,
which the oracle checks on small grids."""
import math

import numpy as np
import pytest

from paper_1206_3229_amd import inputs as I

pytestmark = pytest.mark.gpu

# the first size at which f is 120 MiB, odd rows, and tiles of both widths
CASES = {
    "sheet_zero_p": I.Params(I.MODEL_SHEET, 8191, 3851, -10.0, 10.0, -4.0, 4.0, 0.01, bc_x=I.BC_ZERO, bc_p=I.BC_ZERO,
                             storage=I.STORAGE_F32),
    "hmf_wide": I.Params(I.MODEL_HMF, 8193, 3840, -math.pi, math.pi, -2.5, 2.5, 0.5, storage=I.STORAGE_F32),
}


@pytest.mark.parametrize("name", list(CASES))
def test_far_grid(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1206_3229_amd import vlasov as V
    V.load()
    p = CASES[name]
    assert 4 * p.nx * p.np_ >= 120 << 20
    got = []
    for width in (230, 0):
        s = V.Solver(p, V.ic_waterbag(2.0, 1.5, 0.5, 3))
        s.set_tuning(128, 32, width, 2)
        print(f"far {name} {p.nx}x{p.np_} width {width}", flush=True)
        s.step(3)
        s.profile(True)
        s.step(2)
        ran = s.profile_read()
        s.profile(False)
        assert (ran["drift2"][1] == 0) == (width == 230)  # fused, or not
        got.append(s.read_f())
        s.close()
    assert np.array_equal(got[0], got[1])
