"""A pressure of exactly zero (p_floor 0) where the transverse field goes
through zero: the zone's tracing speed is zero and everything else is finite,
so the sweep has to stay finite and equal the oracle's."""
import numpy as np
import pytest

import gpu_cases as GC
from paper_1607_02214_amd import inputs as I

torch = pytest.importorskip("torch")


def cold_sheet(n):
    """Gas without pressure at rest, B_t1 = -1, 0, +1 across zone 10 of every
    pencil along x (n = 0), y or z; the energy is the field's alone."""
    shape = [8, 8, 8]
    shape[n] = 21
    case = GC.Case("cold-sheet", [I.uniform_faces(k) for k in shape], None, bc_lo=(1, 1, 1), bc_hi=(1, 1, 1),
                   p_floor=0.0)
    b = np.sign(np.arange(21) - 10.0)
    b = np.broadcast_to(b.reshape([-1 if 2 - a == n else 1 for a in range(3)]), shape[::-1])
    U = np.zeros((8,) + b.shape)
    U[0] = 1.0
    U[4 + n] = 0.25
    U[4 + (n + 1) % 3] = b
    U[7] = 0.5 * (0.25 ** 2 + b * b)
    case.U = U
    return case


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_the_oracle_is_finite(axis):
    case = cold_sheet(axis)
    out = case.oracle().sweep(case.U, 0.01, axis)
    assert np.all(np.isfinite(out)) and np.max(np.abs(out - case.U)) > 1e-3


# one sweep in 64 bits, and the bound of the parity tests (rounding of a few
# hundred operations per zone)
@pytest.mark.gpu
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_sweep_of_a_cold_sheet(axis):
    case = cold_sheet(axis)
    ref = case.oracle().sweep(case.U, 0.01, axis)
    u = torch.from_numpy(case.U).to("cuda").contiguous()
    case.context().sweep(u, 0.01, axis)
    err = GC.familywise_errors(u.cpu().numpy(), ref)
    assert np.all(np.isfinite(err)) and np.max(err) <= 1e-12, err
