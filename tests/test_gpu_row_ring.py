"""The pipelined march takes its row entries from an LDS ring that is refilled
once per unroll period (10 planes at depth 1, 12 at depth 2): marches that end
before, at and after the first refills, on both storages and in both
directions, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import System, orbital_rel_err, rsg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("nz", [1, 4, 9, 10, 11, 12, 13, 23, 37])
def test_marches_of_every_length(nz, align):
    R = rsg()
    s = System(0.3, box=(37, 21, nz), potential="wells", natoms=1, nst=2, seed=80 + nz, dipole_axis=2, rcut=0.9,
               pad=3, align=align)
    ref = oracle.hpsi(s.oh, s.psi, field=0.05, nst=s.nst)
    psi = s.to_gpu(s.psi)
    for t in R.tile_candidates("c128"):
        for zm in (0, 1):  # upward; from the centre plane both ways
            R.set_tile(s.gh, s.nst, t["B"], t["TX"], t["TY"], 0, t["PD"], 0, 1, zm)
            out = R.hpsi(s.gh, psi, field=0.05, out=psi.clone())
            e = orbital_rel_err(s.from_gpu(out), ref, s.nst)
            assert e <= 1e-12, (t, zm, e)
            assert s.pad_untouched(out) and not np.any(s.dead_values(out)), (t, zm)


@pytest.mark.parametrize("align", [1, 8])
@pytest.mark.parametrize("box", [(32, 16, 8), (33, 17, 13), (70, 9, 5), (5, 5, 5)])
def test_full_boxes_compute_their_items_and_rows(box, align):
    """On a full box a workgroup computes its tile, chunk and row entries; the
    same tiles in Morton order come from a list.  Both give the oracle's result
    and each other's bits, for every order of chunks and orbitals."""
    R = rsg()
    s = System(0.3, box=box, potential="wells", natoms=1, nst=3, seed=90 + box[0], dipole_axis=1, rcut=0.9,
               pad=3, align=align)
    ref = oracle.hpsi(s.oh, s.psi, field=0.05, nst=s.nst)
    psi = s.to_gpu(s.psi)
    for t in R.tile_candidates("c128"):
        for zc in (0, 1, 4):
            R.set_tile(s.gh, s.nst, t["B"], t["TX"], t["TY"], zc, t["PD"], 1, 1, 0)
            listed = R.hpsi(s.gh, psi, field=0.05, out=psi.clone())
            for bo, zm in ((0, 0), (1, 2), (2, 2)):
                R.set_tile(s.gh, s.nst, t["B"], t["TX"], t["TY"], zc, t["PD"], 0, bo, zm)
                out = R.hpsi(s.gh, psi, field=0.05, out=psi.clone())
                e = orbital_rel_err(s.from_gpu(out), ref, s.nst)
                assert e <= 1e-12, (t, zc, bo, zm, e)
                assert s.pad_untouched(out) and not np.any(s.dead_values(out)), (t, zc, bo, zm)
                assert np.array_equal(s.from_gpu(out), s.from_gpu(listed)), (t, zc, bo, zm)
