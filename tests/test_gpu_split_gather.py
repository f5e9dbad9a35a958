"""Projector gathers whose support is split into chunks: 2 and 3, and past the 8
chunk sums that are loaded together (9, 11, 18), with 1 to 9 orbitals.  Every
reader of the chunk sums against the oracle: the scatter in FP64, mixed
precision and under the mask, the energy, and the solvers' p^T H p from the
stencil and from a pass of its own."""
import numpy as np
import pytest
import torch

import oracle
from oracle import shifted as sv
from tests.gpu_common import System, orbital_rel_err, rsg

pytestmark = pytest.mark.gpu

# support radius -> chunks of a single atom at h = 0.3: one per 512 support points
CASES = [(1.95, 1, 2), (2.2, 9, 3), (3.15, 3, 9), (3.35, 2, 11), (3.95, 1, 18)]


def build(rcut, nst, chunks, align):
    s = System(0.3, R=4.5, potential="wells", natoms=1, nst=nst, seed=17, dipole_axis=1, rcut=rcut, well_ball=0.2,
               pad=2, align=align)
    n = len(s.proj.idx[0])
    assert (n + 15) // 16 * 4 // 128 == chunks, n  # groups of 4 entries over 8 x 16 slots
    return s


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("rcut,nst,chunks", CASES)
def test_scatter_and_energy(rcut, nst, chunks, align):
    R = rsg()
    s = build(rcut, nst, chunks, align)
    psi = s.to_gpu(s.psi)
    h = oracle.hpsi(s.oh, s.psi, field=0.03, nst=nst)
    assert orbital_rel_err(s.from_gpu(R.hpsi(s.gh, psi, field=0.03)), h, nst) <= 1e-12
    e = 0.3 ** 3 * np.sum(np.conj(s.psi[:, :nst]) * h[:, :nst], axis=0)
    np.testing.assert_allclose(R.energy(s.gh, psi, field=0.03).cpu().numpy(), e, rtol=0, atol=1e-12 * np.abs(e).max())
    ref = oracle.taylor_step(s.oh, s.psi, 0.005, field=0.03, nst=nst)
    x = R.propagate_step(s.gh, psi.clone(), 0.005, field=0.03)
    assert orbital_rel_err(s.from_gpu(x), ref, nst) <= 1e-12
    # four FP32 applications of H, |H psi| dt below 2 |psi|, terms rounded to 6e-8
    x = R.propagate_step(s.gh, psi.clone(), 0.005, field=0.03, dtype="mixed")
    assert orbital_rel_err(s.from_gpu(x), ref, nst) <= 2e-6
    mask = np.cos(0.2 * np.linalg.norm(s.pos, axis=1)) ** 2
    s.gh.set_mask(torch.from_numpy(s.slots(mask)).cuda())
    x = R.propagate_step(s.gh, psi.clone(), 0.005, field=0.03)
    assert orbital_rel_err(s.from_gpu(x), ref * mask[:, None], nst) <= 1e-12


@pytest.mark.parametrize("method", ["qmr", "cg"])
@pytest.mark.parametrize("rcut,nst,chunks", CASES)
def test_solves(rcut, nst, chunks, method):
    R = rsg()
    s = build(rcut, nst, chunks, 1)
    shifts = np.full(nst, 0.4 + 0.1j if method == "qmr" else 9.0)
    ref, _, _, _ = sv.solve_batch(s.oh, s.psi, shifts, method, tol=0.0, maxiter=6, nst=nst)
    for tx, ty, zc in ((32, 16, 0), (8, 8, 1)):
        R.set_tile(s.gh, nst, 1, tx, ty, zc, 1, 0, 2)
        x, _ = R.shifted_solve(s.gh, s.to_gpu(s.psi), shifts, method=method, tol=0.0, maxiter=6)
        assert orbital_rel_err(s.from_gpu(x), ref, nst) <= 1e-10, (tx, ty, zc)
