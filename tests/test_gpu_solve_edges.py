"""QMR where p^T (H + sigma) p all but vanishes: theta's square overflows, gamma is
zero and the step changes nothing, so the residual stays what it was."""
import numpy as np
import pytest
import torch

from tests.gpu_common import rsg

pytestmark = pytest.mark.gpu


def test_qmr_step_without_progress_keeps_its_residual():
    R = rsg()
    g = R.Grid(1.0, n=11)
    c = int(np.nonzero((g.coords() == 5).all(axis=1))[0][0])
    V = torch.zeros(g.np, dtype=torch.float64, device="cuda")
    V[c] = 0.5 * (3.0 * (-205.0 / 72.0))  # kin / h^2 = -1/2: the diagonal of H at the centre is exactly zero
    H = R.Hamiltonian(g, V=V, kin=-0.5)
    b = torch.zeros(1, g.np, dtype=torch.complex128, device="cuda")
    b[0, c] = 1.0
    assert R.hpsi(H, b)[0, c] == 0
    x, info = R.shifted_solve(H, b, 1e-158j, method="qmr", tol=1e-10, maxiter=1)
    true = torch.linalg.vector_norm(b - R.hpsi(H, x) - 1e-158j * x)
    assert info["rel_res"][0] == pytest.approx(float(true), rel=1e-12) and info["status"][0] != 0
