"""The shell solve takes half of the longitude modes and rebuilds the other
half: odd counts of longitudes (no Nyquist mode), the smallest shells, a narrow
and the largest, against the oracle.  Bounds as for the even shells: the
current takes the same FP64 arithmetic (1e-12 of its largest value), the
potential comes from two direct solves of one system (1e-11)."""
import numpy as np
import pytest
import torch

import gpu_cases as GC
from test_gpu_ionosphere import _case, _dev, _host, _oracle_couple

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_theta,n_phi", [(2, 4), (2, 5), (3, 5), (5, 6), (17, 33), (32, 63), (24, 7), (3, 129), (64, 64)])
def test_shell_of(n_theta, n_phi):
    from paper_1607_02214_amd import ppmlr
    case = _case()
    prm = ppmlr.iono_default_params()
    prm.n_theta, prm.n_phi = n_theta, n_phi
    jr = torch.zeros((2, n_theta, n_phi), dtype=torch.float64, device="cuda")
    phi = torch.zeros_like(jr)
    case.context().ionosphere_couple(_dev(case.U), prm, jr=jr, phi=phi)
    jr_o, phi_o, _, _ = _oracle_couple(case, case.oracle(), case.U, prm)
    e_jr = float(np.max(np.abs(_host(jr) - jr_o)) / np.max(np.abs(jr_o)))
    e_phi = float(np.max(np.abs(_host(phi) - phi_o)) / np.max(np.abs(phi_o)))
    GC.log(f"[iono] {n_theta} x {n_phi}: jr {e_jr:.2e} phi {e_phi:.2e}")
    assert e_jr <= 1e-12 and e_phi <= 1e-11
