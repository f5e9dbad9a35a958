"""A tuned tile is no slower than the one it replaces: the tuner times the launch
that runs, with the projector gather that rides in it, and the default tile among
its candidates."""
import re

import pytest
import torch

from tests.gpu_common import System, rsg

pytestmark = pytest.mark.gpu


def step_us(R, H, psi, dtype, steps=10):
    """Best of eight replays of a captured sequence, microseconds a step."""
    s = torch.cuda.Stream()
    ws = torch.empty(H.workspace_bytes("step", psi.shape[0], psi.shape[1], R._dt(dtype)), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    best = 1e9
    with torch.cuda.stream(s):
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            R.propagate(H, psi, 1e-4, steps, dtype=dtype, graph=True, ws=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / steps)
    return best


@pytest.mark.parametrize("dtype", ["c128", "mixed"])
def test_tuned_step_is_no_slower_with_projectors(dtype):
    """Without the gather 16 x 8 tiles lead in mixed precision; with it, on their
    two waves, a step takes 97 us and 70 in 32 x 8 ones."""
    R = rsg()
    s = System(0.25, n=41, potential="wells", natoms=2, nst=10, seed=5, rcut=2.0)
    psi = s.to_gpu(s.psi)
    before = step_us(R, s.gh, psi, dtype)
    R.autotune(s.gh, psi, dtype=dtype, reps=2)
    assert step_us(R, s.gh, psi, dtype) <= 1.1 * before


def test_cache_key_names_kernels_and_projectors(tmp_path):
    R = rsg()
    path = str(tmp_path / "tiles.txt")
    a = System(0.3, R=2.4, potential="wells", natoms=1, nst=2, seed=21, rcut=1.2)
    psi = a.to_gpu(a.psi)
    assert not R.autotune_cached(a.gh, psi, path, reps=1)[2]
    line = open(path).read()
    assert " atoms=1 support=" in line and " kernels=" in line
    # the same box without projectors is another launch
    b = System(0.3, R=2.4, potential="wells", natoms=0, nst=2, seed=21)
    assert not R.autotune_cached(b.gh, b.to_gpu(b.psi), path, reps=1)[2]
    # an entry of other kernels is not taken
    open(path, "w").write(re.sub(r"kernels=\d+", "kernels=0", line))
    assert not R.autotune_cached(a.gh, psi, path, reps=1)[2]
