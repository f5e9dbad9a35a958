"""Tiles of few threads leave the projector gather to a launch of its own where their
marches are short: the same bits as with the gather in the stencil's launch, and
a stage that does not wait for one or two waves."""
import pytest
import torch

from tests.gpu_common import System, rsg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "mixed"])
@pytest.mark.parametrize("rcut,nst", [(1.7, 9), (2.2, 1)])  # whole and split supports
def test_same_bits(dtype, rcut, nst):
    R = rsg()
    s = System(0.3, R=3.9, potential="wells", natoms=3, nst=nst, seed=23, dipole_axis=0, rcut=rcut, well_ball=1.0, align=8)
    out = []
    for tx, ty, zc in ((32, 8, 2), (16, 8, 2), (16, 8, 0)) + (((8, 8, 2), (8, 8, 0)) if dtype == "c128" else ()):
        R.set_tile(s.gh, nst, 1, tx, ty, zc, 1, 0, 1, 2 if zc else 0, dtype=dtype)
        out.append(R.propagate_step(s.gh, s.to_gpu(s.psi), 0.01, field=0.02, dtype=dtype))
    for x in out[1:]:
        assert torch.equal(torch.view_as_real(x), torch.view_as_real(out[0]))


def test_one_wave_tiles_do_not_wait_for_the_gather():
    """8 x 8 tiles in chunks of 2 planes: 32 us a stage with the gather on their one
    wave, 14.6 with its own launch, 13 in 32 x 8 tiles."""
    R = rsg()
    s = System(0.3, n=23, potential="wells", natoms=2, nst=2, seed=5, rcut=2.0)
    psi, stream = s.to_gpu(s.psi), torch.cuda.Stream()
    ws = torch.empty(s.gh.workspace_bytes("step", 2, psi.shape[1], R.C128), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    best = {}
    for tile in ((8, 8), (32, 8)):
        R.set_tile(s.gh, 2, 1, *tile, 2, 1, 0, 1, 2)
        with torch.cuda.stream(stream):
            for _ in range(8):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                R.propagate(s.gh, psi, 1e-4, 10, graph=True, ws=ws)
                b.record()
                b.synchronize()
                best[tile] = min(best.get(tile, 1e9), a.elapsed_time(b))
    assert best[8, 8] <= 1.6 * best[32, 8]
