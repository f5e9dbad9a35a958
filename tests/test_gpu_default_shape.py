"""The tile a launch gets that nobody tuned changes with the points times
orbitals of the call: on both sides of each line of the rule it is a compiled
tile and gives the bits of a fixed 16 x 8 tile, in FP64, mixed precision and
complex-scaled."""
import pytest
import torch

from tests.gpu_common import rsg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("nst", [1, 3, 4, 6, 7, 12, 13, 50, 51, 128, 129])
def test_default_tiles_give_the_bits_of_a_fixed_one(nst, align):
    R = rsg()
    g = R.Grid(0.25, R=6.6, align=align)  # 77 k points: lines at 1e5, 2.5e5, 1e6, 4e6 and 1e7 values
    gen = torch.Generator(device="cuda").manual_seed(5)
    live = torch.zeros(g.np, dtype=torch.float64, device="cuda")
    live[torch.from_numpy(g.live()).cuda()] = 1.0
    V = torch.randn(g.np, dtype=torch.float64, device="cuda", generator=gen) * live
    psi = torch.view_as_complex(torch.randn(nst, g.np, 2, dtype=torch.float64, device="cuda", generator=gen)) * live

    def results(tile):
        out = []
        for dtype in ("c128", "mixed"):
            H = R.Hamiltonian(g, V=V, dipole_axis=1)
            if tile:
                R.set_tile(H, nst, 1, 16, 8, 0, 1, dtype=dtype)
            else:
                t = R.get_tile(H, nst, dtype)
                assert any((t["TX"], t["TY"], t["PD"]) == (c["TX"], c["TY"], c["PD"]) for c in R.tile_candidates(dtype))
            out.append(R.propagate_step(H, psi.clone(), 0.01, field=0.03, dtype=dtype))
        H = R.Hamiltonian(g, V=V)
        H.set_complex_scaling(0.3, 0.1 * V)
        if tile:
            R.set_tile(H, nst, 1, 16, 8, 0, 1)
        out.append(R.hpsi(H, psi))
        return out

    for a, b in zip(results(False), results(True)):
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
