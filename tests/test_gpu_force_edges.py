"""Edges of the force kernels of the single grids, against the oracle, bit for
bit: sheet grids of one sample per lane and less, of whole and ragged chunks,
around the rounds of a workgroup (4096 columns), the largest staged in LDS and
the first that is not (16384, 16385); HMF grids around one column per thread
and four."""
import math

import numpy as np
import pytest

from paper_1206_3229_amd import inputs as I

pytestmark = pytest.mark.gpu

SHEET = [16, 63, 64, 65, 127, 1023, 1024, 1025, 1100, 4095, 4096, 4097, 5000, 16383, 16384, 16385, 16450]
HMF = [16, 65, 1024, 1025, 4096, 4097, 4600]
# density and force in one kernel: up to 8, 16 and 32 blocks of 16 rows, 1024
# columns and 16384 sums, and past each limit
SMALL = [(16, 16), (63, 17), (64, 128), (65, 129), (127, 256), (256, 257), (512, 512), (31, 512), (33, 513), (513, 512),
         (1024, 256), (1023, 256), (1024, 257), (1025, 16)]


@pytest.mark.parametrize("model,nx,np_", [(I.MODEL_SHEET, n, 16) for n in SHEET] + [(I.MODEL_HMF, n, 16) for n in HMF] +
                         [(m, *s) for m in (I.MODEL_SHEET, I.MODEL_HMF, I.MODEL_RING) for s in SMALL])
def test_force(oracle, model, nx, np_):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1206_3229_amd import vlasov as V
    V.load()
    sheet = model == I.MODEL_SHEET
    half = 10.0 if sheet else math.pi
    p = I.Params(model, nx, np_, -half, half, -4.0, 4.0, 0.05, bc_x=I.BC_ZERO if sheet else I.BC_PERIODIC)
    f0 = np.random.default_rng(nx).random((np_, nx))
    f0[:, : nx // 7] = 0.0
    s = V.Solver(p, f0)
    s.drift(1)
    f = s.read_f()
    F, mm = s.force()
    s.close()
    F_want, mm_want = oracle.force(p, oracle.density(p, f))
    assert np.array_equal(F, F_want)
    assert sheet or mm == mm_want
