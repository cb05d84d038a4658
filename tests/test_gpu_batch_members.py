"""Batches of one member, and of members that all take steps but one, with
grids whose drift offsets spread too much inside a tile for the fused kernel
among them; each grid bitwise as stepped alone."""
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


def _spread(p):
    """Largest difference (columns) of the offsets of both half drifts within 16 rows."""
    m = np.floor(-(p.pmin + np.arange(p.np_) * p.dp) * (0.5 * p.dt) / p.dx)
    if p.bc_x == I.BC_ZERO:
        m = np.clip(m, -(p.nx + 16), p.nx + 16)
    return max(int(np.ptp(2 * m[j:j + 16])) for j in range(0, p.np_, 16))


def _hmf(nx, np_, dt, storage):
    return I.Params(I.MODEL_HMF, nx, np_, -math.pi, math.pi, -2.5, 2.5, dt, storage=storage)


def _sheet(nx, np_, dt, storage):
    return I.Params(I.MODEL_SHEET, nx, np_, -10.0, 10.0, -4.0, 4.0, dt, bc_x=I.BC_ZERO, storage=storage)


def _ring(nx, np_, dt, storage):
    return I.Params(I.MODEL_RING, nx, np_, -math.pi, math.pi, -3.0, 3.0, dt, storage=storage)


# by their spread: up to 8 columns, 9 to 56 (wide tiles), more (no fused kernel)
GRIDS = {"hmf": (_hmf, 100, 70, 0.05, 0, 8), "hmf_wide": (_hmf, 400, 40, 0.3, 9, 56), "hmf_apart": (_hmf, 400, 40, 1.0, 57, 1 << 30),
         "sheet": (_sheet, 231, 33, 0.05, 0, 8), "sheet_apart": (_sheet, 300, 32, 20.0, 57, 1 << 30),
         "ring_apart": (_ring, 333, 47, 2.0, 57, 1 << 30)}


def _grid(name, storage):
    make, nx, np_, dt, lo, hi = GRIDS[name]
    p = make(nx, np_, dt, storage)
    assert lo <= _spread(p) <= hi, (name, _spread(p))
    return p


def _run(V, grids, steps, **kw):
    rng = np.random.default_rng(4)
    f0 = [rng.uniform(0.0, 1.0, (p.np_, p.nx)) / (p.nx * p.np_ * p.dx * p.dp) for p in grids]
    alone = []
    for p, f, n in zip(grids, f0, steps):
        s = V.Solver(p, f)
        s.step(n)
        alone.append(s.read_f())
        s.close()
    solvers = [V.Solver(p, f) for p, f in zip(grids, f0)]
    V.batch_step(solvers, steps, **kw)
    for k, (s, want) in enumerate(zip(solvers, alone)):
        assert np.array_equal(s.read_f(), want), (k, kw)
        s.close()
    for f, want, n in zip(f0, alone, steps):
        assert n == 0 or not np.array_equal(f, want)  # it did move


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("name", list(GRIDS))
def test_one_member(V, name, fuse, storage):
    for n in (1, 2, 7):
        _run(V, [_grid(name, storage)], [n], chunk_cycles=4, fuse=fuse)


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("fuse", [True, False])
def test_every_member_steps_but_one(V, fuse, storage):
    names = [list(GRIDS)[k % len(GRIDS)] for k in range(66)]
    steps = [0 if k == 31 else 1 + k % 6 for k in range(66)]
    _run(V, [_grid(name, storage) for name in names], steps, chunk_cycles=4, fuse=fuse)
