"""Kernel times of one form of a call beside another form's, measured in the same
process: a form that falls behind does so by a cause of its own (loads that wait
for each other, too few workgroups), not by the chip's."""
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


def _time(s, kernels, call):
    """Least mean time (us) of a launch of `kernels` over 20 windows of ten calls."""
    call()
    best = math.inf
    for _ in range(20):
        s.profile(True)
        for _ in range(10):
            call()
        t = s.profile_read()
        s.profile(False)
        best = min(best, sum(t[k][0] for k in kernels) * 1e3 / sum(t[k][1] for k in kernels))
    return best


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
@pytest.mark.parametrize("n", [256, 1024])
def test_global_spline_kick_with_zero_p(V, n, storage):
    """The same kick on a zero-extended p axis as on a periodic one: the same samples and sums but for the
    boundary rule.  1.8 to 2.3 times as long where each load near the ends waits for the one before it; the limit
    is the geometric mean of that and 1."""
    times = []
    for bc in (I.BC_PERIODIC, I.BC_ZERO):
        p = I.Params(I.MODEL_EXTERNAL, n, n, -10.0, 10.0, -4.0, 4.0, 0.02, bc_p=bc, storage=storage,
                     spline=I.SPLINE_GS)
        s = V.Solver(p, V.ic_waterbag(1.2, 0.9))
        s.set_external_force(np.sin(2.0 * math.pi * np.arange(n) / n) * 5.0 * p.dp / p.dt)
        s.force()
        times.append(_time(s, ["kick"], s.kick))
        s.close()
    print(f"global spline kick {n}^2 storage {storage}: periodic {times[0]:.2f} us, zero {times[1]:.2f} us", flush=True)
    assert times[1] <= 1.35 * times[0]


@pytest.mark.parametrize("storage", [I.STORAGE_F64, I.STORAGE_F32])
def test_global_spline_drift_of_a_small_grid(V, storage):
    """A half drift (with its density partial sums) of 64 rows of 64 takes no longer than one of 512 rows of 512,
    which has 64 times the values: 1.15 to 1.2 times as long where two threads move a row of 64 and one workgroup
    has all rows."""
    times = []
    for n in (64, 512):
        p = I.Params(I.MODEL_HMF, n, n, -math.pi, math.pi, -2.5, 2.5, 0.02, storage=storage, spline=I.SPLINE_GS)
        s = V.Solver(p, V.ic_waterbag(1.2, 0.9))
        times.append(_time(s, ["drift"], lambda: s.drift(1)))
        s.close()
    print(f"global spline half drift storage {storage}: 64^2 {times[0]:.2f} us, 512^2 {times[1]:.2f} us", flush=True)
    assert times[0] <= times[1]


def _copy_time(V, nbytes):
    """Least mean time (us) of ten copies of nbytes from one device buffer to another and back."""
    import torch
    a = torch.rand(nbytes // 8, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    best = math.inf
    for _ in range(20):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for k in range(10):
            V.device_copy(*((b, a) if k % 2 else (a, b)), nbytes)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 100.0)
    return best


def test_fused_kernel_beyond_the_last_level_cache(V):
    """The FP32 fused kernel on 256 MiB of f against a copy of that size, which reads and writes the same bytes:
    1.8 times as long where it wrote through the L2s and requested two rows ahead, 1.4 times as it was before it
    did either; the limit lies between."""
    n = 8192
    p = I.Params(I.MODEL_SHEET, n, n, -10.0, 10.0, -4.0, 4.0, 0.005, bc_x=I.BC_ZERO, storage=I.STORAGE_F32)
    s = V.Solver(p, V.ic_waterbag(1.2, 0.9, 1e-4, 1))
    fused = _time(s, ["kick_drift2"], lambda: s.step(3))
    s.close()
    copy = _copy_time(V, 4 * n * n)
    print(f"fused kernel on 256 MiB {fused:.1f} us, copy {copy:.1f} us", flush=True)
    assert fused <= 1.6 * copy


def test_read_f_against_a_plain_copy(V):
    """32 MiB of f in FP64 into a buffer that has been written before, against torch's copy from the device into it:
    5 times as long by way of fresh memory of the same size; the limit is the geometric mean of that and 1."""
    import time

    import torch
    n = 2048
    s = V.Solver(I.Params(I.MODEL_HMF, n, n, -math.pi, math.pi, -2.5, 2.5, 0.02), V.ic_waterbag(1.2, 0.9))
    out = np.ones((n, n))
    src = torch.rand(n, n, dtype=torch.float64, device="cuda")
    best = []
    for call in (lambda: V.check(V.load().vlasov_read_f(s._ctx, V._dptr(out))), lambda: torch.from_numpy(out).copy_(src)):
        call()
        times = []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call()
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best.append(min(times) * 1e6)
    s.close()
    print(f"read_f of 32 MiB {best[0]:.0f} us, torch copy {best[1]:.0f} us", flush=True)
    assert best[0] <= 2.3 * best[1]
