"""The fused prediction's branch-free z loop on ragged tiles and short z
ranges.  Lanes past a smaller tile repeat its last cell; the xy tiles are
dealt over the XCDs in two orders.  Its cell
arithmetic is the general loop's in the same order, so a whole step (three
predictions, the correcting ones included) is equal bit for bit."""
import numpy as np
import pytest

from test_gpu_navier_stokes import device_state, periodic_plan, random_state, scratch_for

pytestmark = pytest.mark.gpu

SHAPES = [
    (6, 4, 2),         # fewer cells than a tile along x and y, one range of two planes
    (64, 8, 4),        # one whole tile, two ranges of two planes
    (60, 10, 5),       # ranges of two and three planes
    (72, 10, 18),      # 8 and 2 cells past a tile
    (450, 20, 30),     # eight tiles along x: the order by column
    (200, 90, 27),     # 4 x 12 tiles, the last row of two cells
    (128, 48, 270),    # three ranges at least
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_every_shape_equals_the_general_loop(shape, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx, ny, nz = shape
    vel, _, p = random_state(5 + nx, (nz, ny, nx))
    out = []
    for general in (False, True):
        if general:
            monkeypatch.setenv("POISSON_RK3_GENERAL", "1")
        else:
            monkeypatch.delenv("POISSON_RK3_GENERAL", raising=False)
        plan, _ = periodic_plan(nx, ny, nz, (1.0, 0.7, 1.2))
        dvel, work, dad, dp, phi = device_state(vel, np.zeros_like(vel), p)
        print("rk3 tiles", shape, "general" if general else "default", flush=True)
        plan.rk3_step(0.001, 0.003, dvel, work, dad, dp, phi, scratch_for((nz, ny, nx)))
        torch.cuda.synchronize()
        out.append((dvel.clone(), dp.clone()))
        plan.close()
    assert torch.isfinite(out[0][0]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
