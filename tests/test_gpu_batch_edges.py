"""Batches: the phases that a cycle launches (fused last kicks, members that
cannot fuse, a graph only after some chunks, more than 64 members), each grid
bitwise as stepped alone."""
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


def _grid(k, storage):
    """Grid k of a batch: all models, ragged sizes; every 7th cannot fuse, every 5th is too short in x for a
    fused last kick on a periodic axis."""
    nx, np_ = (16 if k % 5 == 0 else 33 + 29 * (k % 11)), 17 + 13 * (k % 9)
    dt = 3.0 if k % 7 == 0 else 0.05
    if k % 3 == 0:
        return I.Params(I.MODEL_SHEET, nx, np_, -10.0, 10.0, -4.0, 4.0, dt, bc_x=I.BC_ZERO, storage=storage)
    return I.Params(I.MODEL_HMF if k % 3 == 1 else I.MODEL_RING, nx, np_, -math.pi, math.pi, -2.5, 2.5, dt,
                    storage=storage)


def _run(V, grids, steps, **kw):
    rng = np.random.default_rng(2)
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
        assert np.array_equal(s.read_f(), want, equal_nan=True), (k, kw)
        s.close()


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("members", [1, 64, 65, 130])
def test_members(V, members, fuse, storage):
    _run(V, [_grid(k, storage) for k in range(members)], [k % 6 for k in range(members)], chunk_cycles=4, fuse=fuse)


@pytest.mark.parametrize("fuse", [True, False])
def test_graph_after_many_chunks(V, fuse):
    grids = [_grid(k, I.STORAGE_F64) for k in (1, 2, 3, 4, 6)]
    _run(V, grids, [41, 60, 50, 33, 60], chunk_cycles=2, fuse=fuse)
