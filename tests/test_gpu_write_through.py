"""Grids from the size on at which the drifts write through the L2s (512 KiB of
f in FP64, 2 MiB in FP32; and just under it): rows of odd length, whose pairs
are aligned to one value only, tiles of both widths, last rows and columns
alone, both boundaries, one half drift and two.  All bitwise."""
import math

import numpy as np
import pytest

from paper_1206_3229_amd import inputs as I

pytestmark = pytest.mark.gpu


def _hmf(nx, np_, dt, storage, **kw):
    return I.Params(I.MODEL_HMF, nx, np_, -math.pi, math.pi, -2.5, 2.5, dt, storage=storage, **kw)


def _sheet(nx, np_, dt, storage, **kw):
    return I.Params(I.MODEL_SHEET, nx, np_, -10.0, 10.0, -4.0, 4.0, dt, bc_x=I.BC_ZERO, storage=storage, **kw)


D, S = I.STORAGE_F64, I.STORAGE_F32
CASES = {
    "f64_under": _hmf(255, 256, 0.02, D),
    "f64_first": _hmf(256, 256, 0.02, D),
    "f64_odd": _sheet(461, 163, 0.02, D, bc_p=I.BC_ZERO),
    "f64_wide": _sheet(601, 113, 0.3, D),
    "f64_wide_periodic": _hmf(369, 227, 0.7, D, bc_p=I.BC_ZERO),
    "f32_under": _sheet(724, 724, 0.02, S),
    "f32_first": _sheet(512, 1024, 0.02, S),
    "f32_odd": _hmf(731, 733, 0.02, S, bc_p=I.BC_ZERO),
    "f32_wide": _sheet(2301, 241, 0.15, S),
}


@pytest.mark.parametrize("name", list(CASES))
def test_large_results_match_the_oracle(oracle, name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1206_3229_amd import vlasov as V
    V.load()
    p = CASES[name]
    f0 = np.random.default_rng(11).uniform(-0.25, 1.0, (p.np_, p.nx)) / (p.nx * p.np_ * p.dx * p.dp)
    print(f"through {name} {p.nx}x{p.np_}", flush=True)
    s = V.Solver(p, f0)
    want = f0
    for n in (1, 2):
        s.step(n)
        want = oracle.run(p, want, n)
        assert np.array_equal(s.read_f(), want), (name, n)
    s.drift(1)
    want = oracle.sweep_x(p, want, 0.5 * p.dt)
    assert np.array_equal(s.read_f(), want), (name, "one half drift")
    s.drift(2)
    want = oracle.sweep_x(p, oracle.sweep_x(p, want, 0.5 * p.dt), 0.5 * p.dt)
    assert np.array_equal(s.read_f(), want), (name, "two half drifts")
    s.close()


@pytest.mark.parametrize("storage", [D, S])
@pytest.mark.parametrize("zero", [False, True])
def test_large_global_spline(oracle, storage, zero):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import test_gpu_global_spline_edges as E
    from paper_1206_3229_amd import vlasov as V
    V.load()
    nx, np_ = (515, 131) if storage == D else (1027, 517)
    E.test_sweeps(V, oracle, nx, np_, 0.05, zero, storage)
