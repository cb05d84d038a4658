"""Half drifts without a kick on lines around the length from which their loads
take 16 bytes a lane (512 columns), and around whole tiles of 224 and 230:
windows that pass either end of the line at every place within such a load,
shifts beyond the line, odd lines, last rows alone, tiles of one block and of
two.  Bitwise against the oracle, with the density partial sums (through the
force)."""
import math

import numpy as np
import pytest

from paper_1206_3229_amd import inputs as I

pytestmark = pytest.mark.gpu

# (nx, np, dt): the 512-column rows shift by up to about 1, 40 and 2000 cells
SIZES = [(511, 33, 0.02), (512, 33, 0.02), (513, 16, 0.7), (514, 47, 0.7), (515, 81, 30.0), (672, 40, 0.02),
         (673, 17, 30.0), (690, 65, 0.7), (691, 31, 0.02), (1026, 129, 0.7), (2300, 50, 30.0), (512, 20000, 0.02)]


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("nx,np_,dt", SIZES)
def test_half_drifts(oracle, nx, np_, dt, zero, storage):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1206_3229_amd import vlasov as V
    V.load()
    if zero:
        p = I.Params(I.MODEL_SHEET, nx, np_, -10.0, 10.0, -4.0, 4.0, 3.0 * dt, bc_x=I.BC_ZERO, storage=storage)
    else:
        p = I.Params(I.MODEL_HMF, nx, np_, -math.pi, math.pi, -2.5, 2.5, dt, storage=storage)
    print(f"wide drift {nx}x{np_} dt {dt} zero {zero} storage {storage}", flush=True)
    f0 = np.random.default_rng(7).uniform(-0.25, 1.0, (np_, nx)) / (p.nx * p.np_ * p.dx * p.dp)
    if storage == I.STORAGE_F32:
        f0 = f0.astype(np.float32).astype(np.float64)
    one = oracle.sweep_x(p, f0, 0.5 * p.dt)
    s = V.Solver(p, f0)
    s.drift(1)
    assert np.array_equal(s.read_f(), one)
    s.write_f(f0)
    s.drift(2)
    assert np.array_equal(s.read_f(), oracle.sweep_x(p, one, 0.5 * p.dt))
    s.write_f(f0)
    s.step(1)  # partial sums, kick and last half drift
    assert np.array_equal(s.read_f(), oracle.run(p, f0, 1))
    s.close()
