"""The rule behind default tiles: every line of its tables is crossed (the
orbitals of each side follow from the grid's points), each side has the tile
and the order that its row names, the chunk of a small launch is the shortest
whose work items fit, and the widest tiles give the bits of a fixed one."""
import numpy as np
import pytest
import torch

from tests.gpu_common import rsg

pytestmark = pytest.mark.gpu

# {below: (TX, TY, PD, BO)}; the row after the last line is under None
BIG64 = {1e7: (16, 16, 1, 2), 4e7: (32, 16, 1, 2), None: (32, 16, 1, 2)}
BIG32 = {4e7: (32, 8, 2, 2), None: (32, 16, 1, 2)}
RULES = {
    ("c128", "box", False): {1e6: (32, 8, 1, 1), 2e6: (32, 8, 1, 1), 4e6: (32, 8, 1, 1), **BIG64},
    ("c128", "sphere", False): {2.5e5: (32, 8, 1, 1), 1e6: (16, 8, 1, 1), 2e6: (16, 8, 1, 1), 4e6: (16, 8, 1, 1), **BIG64},
    ("mixed", "sphere", False): {1e5: (32, 8, 1, 1), 2.5e5: (16, 8, 1, 1), 1e6: (16, 8, 1, 1), 2e6: (16, 8, 1, 1),
                                 1e7: (16, 8, 1, 1), **BIG32},
    ("mixed", "sphere", True): {2.5e5: (32, 8, 1, 1), 1e6: (32, 8, 1, 1), 2e6: (32, 8, 1, 1), 4e6: (32, 8, 2, 1),
                                1e7: (32, 8, 2, 1), **BIG32},
}
RULES[("c128", "sphere", True)] = RULES[("c128", "box", True)] = RULES[("c128", "box", False)]
RULES[("mixed", "box", False)] = RULES[("mixed", "sphere", False)]
RULES[("mixed", "box", True)] = RULES[("mixed", "sphere", True)]


def system(box, projectors, align=1):
    R = rsg()
    g = R.Grid(0.25, R=5.0, align=align) if box == "sphere" else R.Grid(0.25, n=34, align=align)
    V = torch.zeros(g.np, dtype=torch.float64, device="cuda")
    proj = []
    if projectors:
        idx = torch.from_numpy(g.live()[:20].astype(np.int32)).cuda()
        proj = [(idx, torch.ones(20, 4, dtype=torch.float64, device="cuda"), [1.0, 1.0, 1.0, 1.0])]
    return g, R.Hamiltonian(g, V=V, projectors=proj)


@pytest.mark.parametrize("dtype,box,projectors", sorted(RULES))
def test_every_line_is_crossed(dtype, box, projectors):
    R = rsg()
    g, H = system(box, projectors)
    rows = list(RULES[dtype, box, projectors].items())
    for (below, row), (_, after) in zip(rows, rows[1:]):
        n = int(np.ceil(below / g.npoints)) - 1  # the last count below the line
        assert n >= 1 and n * g.npoints < below <= (n + 1) * g.npoints
        for nst, want in ((n, row), (n + 1, after)):
            t = R.get_tile(H, nst, dtype)
            assert (t["TX"], t["TY"], t["PD"], t["BO"]) == want, (below, nst, t)


@pytest.mark.parametrize("align", [1, 16])
@pytest.mark.parametrize("box,nst,limit,zmin", [("box", 1, 768, 1), ("box", 5, 768, 1), ("box", 24, 768, 1), ("box", 30, 1536, 6),
                                                ("sphere", 3, 768, 1), ("sphere", 11, 1536, 3), ("sphere", 40, 3072, 4)])
def test_chunks_are_the_shortest_that_fit(box, nst, limit, zmin, align):
    R = rsg()
    g, H = system(box, False, align)
    t = R.get_tile(H, nst)
    c = g.coords()[g.live()]
    x0, x1 = c[:, 0] // align * align, (c[:, 0] // align + 1) * align - 1  # a point's row owns whole lines
    ends = {}
    for x in (x0, x1):
        for tx, ty, z in zip(x // t["TX"], c[:, 1] // t["TY"], c[:, 2]):
            lo, hi = ends.get((tx, ty), (z, z))
            ends[tx, ty] = (min(lo, z), max(hi, z))
    # tiles strictly between a line's ends hold points of their own when they are as wide as a line
    assert t["TX"] >= align
    items = lambda zc: nst * sum(hi // zc - lo // zc + 1 for lo, hi in ends.values())  # noqa: E731
    nz = g.dims[2]
    chunks = -(-nz // t["ZC"])
    assert t["ZC"] == -(-nz // chunks) and t["ZC"] >= zmin and items(t["ZC"]) <= limit
    shorter = [z for z in (-(-nz // k) for k in range(chunks + 1, nz + 1)) if z < t["ZC"]]
    assert not shorter or shorter[0] < zmin or items(shorter[0]) > limit


@pytest.mark.parametrize("nst", [260, 1000])
def test_widest_defaults_give_the_bits_of_a_fixed_tile(nst):
    """The last two rows of every table, in the form that large systems run."""
    R = rsg()
    g, _ = system("box", False, 8)
    gen = torch.Generator(device="cuda").manual_seed(7)
    live = torch.zeros(g.np, dtype=torch.float64, device="cuda")
    live[torch.from_numpy(g.live()).cuda()] = 1.0
    V = torch.randn(g.np, dtype=torch.float64, device="cuda", generator=gen) * live
    psi = torch.view_as_complex(torch.randn(nst, g.np, 2, dtype=torch.float64, device="cuda", generator=gen)) * live
    for dtype in ("c128", "mixed"):
        out = []
        for tile in (False, True):
            H = R.Hamiltonian(g, V=V, dipole_axis=1)
            if tile:
                R.set_tile(H, nst, 1, 16, 8, 0, 1, dtype=dtype)
            else:
                t = R.get_tile(H, nst, dtype)
                assert (t["TX"], t["TY"]) == ((32, 8) if dtype == "mixed" and nst * g.npoints < 4e7 else (32, 16))
            out.append(R.propagate_step(H, psi.clone(), 0.01, field=0.03, dtype=dtype))
        assert torch.equal(torch.view_as_real(out[0]), torch.view_as_real(out[1]))
