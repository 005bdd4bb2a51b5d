"""The projection's right-hand side and update alone, where their tiles and z
ranges end: fewer cells than a tile, a cell or more past a tile of 64 x 4, ranges of
four to six planes, one range for few planes, every wall kind on every side.

An updated velocity is one difference, two products and one subtraction of
values of size 1: each rounds once, so against the oracle it is off by at most
8 units of 2^-53 of |u| + gdt 2 |Phi| / h."""
import numpy as np
import pytest

from gpu_util import UNIT, rel_l2, to_dev, to_host
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    ((6, 4, 3), ("P", "P", "NN")),
    ((64, 4, 4), ("NN", "DD", "P")),
    ((65, 6, 10), ("ND", "P", "P")),
    ((72, 6, 130), ("P", "NN", "DD")),
    ((160, 10, 33), ("DD", "DN", "ND")),
    ((128, 128, 67), ("NN", "NN", "NN")),
]


@pytest.mark.parametrize("shape,bcs", CASES)
def test_projection_kernels_at_tile_ends(shape, bcs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import projection as pj
    from paper_1802_10323_amd import Plan
    prob = inputs.make_uniform(*shape, bcs, seed=sum(shape), with_rhs=False)
    vel = inputs.prediction_velocity(prob, 3)
    rng = np.random.default_rng(9)
    pres, phi = (rng.uniform(-1, 1, prob.shape) for _ in range(2))
    gdt = 0.25
    args = (prob.hx, prob.hy, prob.hz, prob.bcs)
    plan = Plan.from_problem(prob)
    print("projection ranges", shape, bcs, flush=True)
    dvel = [to_dev(a) for a in vel]
    dp, dphi = to_dev(pres), to_dev(phi)
    rhs = torch.empty(prob.points, dtype=torch.float64, device="cuda")
    plan.projection_rhs(*dvel, gdt, rhs)
    assert rel_l2(to_host(rhs).reshape(prob.shape), pj.projection_rhs(*vel, gdt, *args)) <= 1e-14
    plan.projection_update(dphi, gdt, *dvel, dp)
    ref = pj.project(*vel, pres, phi, gdt, *args)
    for got, before, want, h, bc, axis in zip(dvel, vel, ref, args[:3], bcs, (2, 1, 0)):
        got = to_host(got).reshape(want.shape)
        bound = 8 * UNIT * (max(np.abs(a).max() for a in vel)
                        + gdt * 2.0 / np.min(h))
        assert np.abs(got - want).max() <= bound
        for side, index in ((0, 0), (-1, -1)):
            if bc != "P" and bc[side] == "N":     # a Neumann wall keeps its velocity
                assert np.array_equal(got.take(index, axis), np.asarray(before).take(index, axis))
    assert np.array_equal(to_host(dp).reshape(prob.shape), pres + phi)
    plan.close()
