"""The batch tuner keeps what it cannot beat: it compares whole stages as a step
runs them, with the present tiles among the choices; and a class's information
describes the launch that runs its items."""
import numpy as np
import pytest
import torch

from tests.gpu_common import rsg

pytestmark = pytest.mark.gpu


def batch(radii, nsts, align=1):
    R = rsg()
    gen = torch.Generator(device="cuda").manual_seed(3)
    systems = []
    for rad, nst in zip(radii, nsts):
        g = R.Grid(0.25, R=float(rad), align=align)
        V = torch.zeros(g.np, dtype=torch.float64, device="cuda")
        psi = torch.view_as_complex(torch.randn(nst, g.np, 2, dtype=torch.float64, device="cuda", generator=gen))
        systems.append((R.Hamiltonian(g, V=V), psi, nst))
    return R, R.Batch(systems)


def stage_ms(R, b):
    best = 1e9
    for _ in range(6):
        with R.kernel_timing() as k:
            b.propagate(1e-6, 3)
            torch.cuda.synchronize()
        best = min(best, k.total_ms / 12)
    return best


@pytest.mark.parametrize("align", [1, 8])
def test_tuned_stage_is_no_slower(align):
    """12 spheres of three classes: one launch takes 0.21 ms, the classes' own
    fastest tiles one after another 0.27."""
    rng = np.random.default_rng(9)
    R, b = batch(rng.uniform(4.0, 12.0, 12), rng.integers(2, 9, 12), align)
    assert int(b.classes().max()) == 2
    before = stage_ms(R, b)
    b.autotune(reps=3)
    assert stage_ms(R, b) <= 1.1 * before


def test_class_info_describes_the_launch():
    R, b = batch([4.0, 4.5, 7.0], [2, 3, 2])
    info = [b.class_info(c) for c in range(2)]
    assert [i["nsys"] for i in info] == [2, 1]
    total = sum(i["nitems"] for i in info)
    assert total < 256  # fewer than the compute units, so every item has a workgroup
    # both classes start on one tile: one launch runs them
    assert [i["grid"] for i in info] == [total, total]
    b.set_tile(1, 16, 8, 0, 1, 0, cls=0)
    info = [b.class_info(c) for c in range(2)]
    assert [i["grid"] for i in info] == [i["nitems"] for i in info]
    b.set_grid(5)
    assert [b.class_info(c)["grid"] for c in range(2)] == [5, 5]


def test_a_refused_tile_leaves_the_batch_as_it_was():
    R, b = batch([4.0, 7.0], [2, 2])
    tiles, info = [b.get_tile(c) for c in range(2)], [b.class_info(c) for c in range(2)]
    with pytest.raises(Exception):
        b.set_tile(1, 24, 16, 0, 1, 0, cls=1)
    with pytest.raises(Exception):
        b.set_classes([0, 2])
    assert tiles == [b.get_tile(c) for c in range(2)] and info == [b.class_info(c) for c in range(2)]
