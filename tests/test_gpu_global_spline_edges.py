"""Edges of the global spline's kernels (33 cells of a row or 32 rows of a column
per thread, 31 samples beyond them): lines around these sizes, the shortest
and the longest, one and two half drifts in a pass, shifts beyond a line.
Against the oracle to the global spline's bars: 1e-13 of the largest |f| for
one or two sweeps in FP64, 1e-5 in FP32."""
import math

import numpy as np
import pytest

from paper_1206_3229_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1206_3229_amd import vlasov
    vlasov.load()
    return vlasov


# (nx, np, dt): dt = 9 moves the outer rows by several lengths of a short line
SIZES = [(16, 16, 0.05), (33, 31, 0.05), (34, 32, 0.3), (35, 33, 9.0), (66, 64, 0.05), (67, 129, 0.3), (131, 65, 9.0),
         (1057, 40, 0.05), (2048, 16, 0.05), (4096, 17, 0.05), (18, 4096, 0.05)]


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("nx,np_,dt", SIZES)
def test_sweeps(V, oracle, nx, np_, dt, zero, storage):
    bc = I.BC_ZERO if zero else I.BC_PERIODIC
    p = I.Params(I.MODEL_EXTERNAL, nx, np_, -10.0, 10.0, -4.0, 4.0, dt, bc_x=bc, bc_p=bc, storage=storage,
                 spline=I.SPLINE_GS)
    print(f"global spline {nx}x{np_} dt {dt} bc {bc} storage {storage}", flush=True)
    rng = np.random.default_rng(1)
    f0 = rng.uniform(-0.25, 1.0, (np_, nx))
    if storage == I.STORAGE_F32:
        f0 = f0.astype(np.float32).astype(np.float64)
    F = rng.uniform(-60.0, 60.0, nx) * p.dp / p.dt
    bar = 1e-13 if storage == I.STORAGE_F64 else 1e-5

    def close(got, want, what):
        assert np.max(np.abs(got - want)) <= bar * np.max(np.abs(want)) + 1e-300, what

    s = V.Solver(p, f0)
    s.set_external_force(F)
    s.drift(1)
    close(s.read_f(), oracle.sweep_x(p, f0, 0.5 * dt), "one half drift")
    s.write_f(f0)
    s.drift(2)
    close(s.read_f(), oracle.sweep_x(p, oracle.sweep_x(p, f0, 0.5 * dt), 0.5 * dt), "two half drifts")
    s.write_f(f0)
    s.force()
    s.kick()
    close(s.read_f(), oracle.sweep_p(p, f0, F, dt), "kick")
    s.close()
