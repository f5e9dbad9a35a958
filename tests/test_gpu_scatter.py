"""The projector scatter updates every covered point once, with all the atoms
that cover it: one atom, a few, and more on one spot than are staged at a time
(16), with remainders in points and orbitals, split and unsplit gathers, and
the absorber mask, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import System, orbital_rel_err, rsg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("natoms,ball,nst", [(1, 0.5, 1), (3, 2.0, 9), (17, 0.4, 3), (33, 1.0, 8)])
def test_scatter_matches_oracle(natoms, ball, nst, align):
    R = rsg()
    s = System(0.3, R=3.3, potential="wells", natoms=natoms, nst=nst, seed=90 + natoms, dipole_axis=0, rcut=1.7,
               well_ball=ball, pad=2, align=align)
    psi = s.to_gpu(s.psi)
    out = R.hpsi(s.gh, psi, field=0.03)
    assert orbital_rel_err(s.from_gpu(out), oracle.hpsi(s.oh, s.psi, field=0.03, nst=nst), nst) <= 1e-12
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
