"""The time step and the volume integrals on rows of every length that the
signal-speed kernel packs differently (up to 16, 17 to 32, more zones, and a
remainder), against the oracle; and the step's dt formed on the device."""
import numpy as np
import pytest
import torch

from tests import gpu_cases as GC
from paper_1607_02214_amd import inputs as I

pytestmark = pytest.mark.gpu


def _case(n):
    nx, ny, nz = n
    rng = np.random.default_rng(nx)
    faces = [np.concatenate([[0.0], np.cumsum(rng.uniform(0.7, 1.3, k))]) for k in n]
    return GC.Case("smooth", [f / f[-1] for f in faces], I.random_smooth_state((nz, ny, nx), seed=nx))


# both sides add and multiply in FP64; their orders differ: 1e-12 is some 1e3
# roundings of a sum of at most 1e4 terms of one magnitude
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [(8, 11, 9), (16, 9, 8), (17, 8, 13), (32, 9, 9), (33, 10, 8), (64, 8, 9), (65, 9, 11),
                               (130, 8, 8)])
def test_signal_speed_and_totals(n, dtype):
    case = _case(n)
    u = torch.from_numpy(case.U).to("cuda", dtype).contiguous()
    U = u.double().cpu().numpy()
    ctx, ora = case.context(), case.oracle()
    want = ora.cfl_dt(U, 0.4)
    for _ in range(2):                          # nothing of the first call is left for the second
        assert abs(ctx.cfl_dt(u, 0.4) - want) <= 1e-12 * want
    got, ref = np.asarray(ctx.totals(u)), ora.totals(U)
    assert np.all(np.abs(got - ref) <= 1e-12 * np.abs(ref).max())
    assert abs(ctx.cfl_dt(u, 0.4) - want) <= 1e-12 * want


# the first step of a call takes the dt that the host gets for the same state,
# bit for bit: formed in the first sweep, and by its own kernel (over 2^20 zones)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,segments", [((20, 17, 33), 0), ((40, 24, 31), 2), ((112, 97, 97), 0)])
def test_time_after_a_step(n, segments, dtype):
    case = _case(n)
    ctx = case.context()
    for axis in range(3):
        ctx.set_segments(axis, segments)
    u = torch.from_numpy(case.U).to("cuda", dtype).contiguous()
    v = u.clone()
    dt = ctx.cfl_dt(u, 0.4)
    ctx.advance(u, 1, 0.4)
    assert ctx.time(u) == dt
    dt2 = ctx.cfl_dt(u, 0.4)
    ctx.advance(u, 1, 0.4)
    assert ctx.time(u) == dt + dt2
    host = case.context()                       # and a step with the host's dt is the same step
    for axis in range(3):
        host.set_segments(axis, segments)
    host.step(v, dt)
    assert host.time(v) == dt
    host.step(v, dt2)
    assert host.time(v) == dt + dt2 and torch.equal(u, v)
