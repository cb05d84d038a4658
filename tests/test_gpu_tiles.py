"""Edges of the fused kick and drift tiles (230 columns by 16 to 64 rows, 182
columns where the drift offsets spread over more than 8 columns of a tile) and
of the drift kernel: grids around one and two tiles, the smallest grids, odd
rows, a last kick fused with one half drift in every call.  All bitwise."""
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


def _hmf(nx, np_, dt, **kw):
    return I.Params(I.MODEL_HMF, nx, np_, -math.pi, math.pi, -2.5, 2.5, dt, **kw)


def _sheet(nx, np_, dt, **kw):
    return I.Params(I.MODEL_SHEET, nx, np_, -10.0, 10.0, -4.0, 4.0, dt, bc_x=I.BC_ZERO, **kw)


def _spread(p, rows, both):
    """Largest spread of the drift offsets inside `rows` rows: of both half drifts, or of one."""
    xi = -((p.pmin + np.arange(p.np_) * p.dp) * (0.5 * p.dt) / p.dx)
    m = np.floor(xi) * (2 if both else 1)
    return max(np.ptp(m[b:b + rows]) for b in range(0, p.np_, rows))


CASES = {
    "smallest": _hmf(16, 16, 0.05),
    "smallest_zero": _sheet(16, 17, 0.3, bc_p=I.BC_ZERO),
    "tile_less_one": _sheet(229, 31, 0.02, bc_p=I.BC_ZERO),
    "one_tile": _hmf(230, 16, 0.01),
    "tile_and_one": _hmf(231, 17, 0.02),
    "two_tiles_and_one": _sheet(461, 65, 0.02),
    "odd_rows": _hmf(313, 47, 0.02, bc_p=I.BC_ZERO),
    "wide": _sheet(601, 48, 0.3),
    "wide_periodic": _hmf(365, 50, 0.3, bc_p=I.BC_ZERO),
    "wide_pair_only": _hmf(183, 40, 0.2),
    "wide_last_only": _hmf(1000, 77, 0.7),
}


def test_cases_reach_the_wide_tiles():
    for name, p in CASES.items():
        assert (8 < _spread(p, 16, name != "wide_last_only") <= 56) == name.startswith("wide"), name
    assert _spread(CASES["wide"], 16, False) > 8
    assert _spread(CASES["wide_pair_only"], 16, False) <= 8


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("name", list(CASES))
def test_tiles_match_the_oracle(V, oracle, name, storage):
    p = I.Params(**{**CASES[name].as_dict(), "storage": storage})
    f0 = np.random.default_rng(7).uniform(-0.25, 1.0, (p.np_, p.nx)) / (p.nx * p.np_ * p.dx * p.dp)
    for blocks in (1, 2):
        print(f"tiles {name} {p.nx}x{p.np_} storage {storage} blocks {blocks}", flush=True)
        s = V.Solver(p, f0)
        s.set_tuning(128, 16, 230, blocks)
        want = f0
        for n in (1, 3):
            s.step(n)
            want = oracle.run(p, want, n)
            assert np.array_equal(s.read_f(), want), (name, blocks, n)
        s.drift(1)
        want = oracle.sweep_x(p, want, 0.5 * p.dt)
        assert np.array_equal(s.read_f(), want), (name, "one half drift")
        s.drift(2)
        want = oracle.sweep_x(p, oracle.sweep_x(p, want, 0.5 * p.dt), 0.5 * p.dt)
        assert np.array_equal(s.read_f(), want), (name, "two half drifts")
        s.close()
