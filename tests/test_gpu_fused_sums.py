"""Sums that the stencil takes on the way of an H application: energies without
H psi, and p^T H p / p^H H p of the shifted solves, with and without
projectors, on both storages, for a tile of every march form (one and two
columns per thread, both depths, lean) and both places of CG's partials."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import System, rsg

pytestmark = pytest.mark.gpu

TILES = [(8, 8, 0, 1), (32, 16, 0, 1), (32, 16, 5, 2), (32, 32, 0, 1), (32, 16, 1, 0)]


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("natoms", [0, 3])
def test_energy_matches_oracle(natoms, align):
    R = rsg()
    s = System(0.3, R=3.6, potential="wells", natoms=natoms, nst=5, seed=41, dipole_axis=1, rcut=1.5, align=align, pad=1)
    h = oracle.hpsi(s.oh, s.psi, field=0.04, nst=5)
    ref = 0.3 ** 3 * np.sum(np.conj(s.psi[:, :5]) * h[:, :5], axis=0)
    psi = s.to_gpu(s.psi)
    got = [R.energy(s.gh, psi, field=0.04)]
    for tx, ty, zc, pd in TILES:
        R.set_tile(s.gh, 5, 1, tx, ty, zc, pd, 0, 2)
        got.append(R.energy(s.gh, psi, field=0.04))
    for e in got:
        np.testing.assert_allclose(e.cpu().numpy(), ref, rtol=0, atol=1e-12 * np.abs(ref).max())


def test_scaled_energy_is_the_product_with_h_psi():
    R = rsg()
    g = R.Grid(0.3, R=3.0)
    gen = torch.Generator(device="cuda").manual_seed(3)
    psi = torch.view_as_complex(torch.randn(3, g.np, 2, dtype=torch.float64, device="cuda", generator=gen))
    V = torch.randn(g.np, dtype=torch.float64, device="cuda", generator=gen)
    H = R.Hamiltonian(g, V=V)
    H.set_complex_scaling(0.3, 0.2 * V)
    ref = R.dot(g, psi, R.hpsi(H, psi))
    assert float((R.energy(H, psi) - ref).abs().max()) <= 1e-12 * float(ref.abs().max())


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("method", ["cg", "qmr"])
def test_solves_do_not_depend_on_the_tile(method, align):
    """Twelve iterations from zero: a pass of its own (CG on 1-plane chunks) and
    the stencil's sums give the same iterate to rounding, and its residual is
    the recurrence's."""
    R = rsg()
    s = System(0.3, R=3.6, potential="wells", natoms=2, nst=4, seed=43, rcut=1.5, align=align)
    b = s.to_gpu(s.psi)
    sigma = 9.0 if method == "cg" else 0.4 + 0.1j
    xs = []
    for tx, ty, zc, pd in [(8, 8, 1, 1)] + TILES:
        R.set_tile(s.gh, 4, 1, tx, ty, zc, pd, 0, 2)
        x, info = R.shifted_solve(s.gh, b, sigma, method=method, tol=1e-14, maxiter=12, check_every=5)
        assert list(info["iters"]) == [12] * 4
        res = b - R.hpsi(s.gh, x) - sigma * x
        rel = (torch.linalg.vector_norm(res, dim=1) / torch.linalg.vector_norm(b, dim=1)).cpu().numpy()
        np.testing.assert_allclose(info["rel_res"], rel, rtol=1e-9)
        xs.append(x)
    for x in xs[1:]:
        assert float((x - xs[0]).abs().max()) <= 1e-10 * float(xs[0].abs().max())
