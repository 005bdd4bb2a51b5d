"""The solve inside pressure_correction.  On an FP64 plan it runs the kernels
of the variant table and, for lines of a length without any, the elimination
padded to the next specialised length (regular, non-periodic lines of 43 points
and more): every array within 1e-12 relative L2 of the oracle, for strided and
contiguous lines, each padded length, uniform and stretched, and with every
launch capped at 16 blocks, so that blocks loop over tiles, the same bits.  On a
refined plan it is solve()."""
import numpy as np
import pytest

from gpu_util import rel_l2, to_dev, to_host
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu

# one line length below each specialised one, and one just past the one before it
CASES = [((24, 20, 45), ("P", "NN", "DD"), None), ((24, 20, 66), ("P", "ND", "DN"), 1.8),
         ((40, 12, 100), ("NN", "P", "ND"), 1.8), ((24, 18, 191), ("P", "NN", "DD"), 1.8),
         ((20, 16, 193), ("NN", "NN", "DN"), None), ((36, 10, 320), ("P", "P", "DD"), None),
         ((12, 10, 480), ("DD", "P", "ND"), 1.8), ((20, 250, 8), ("P", "DD", "P"), None),     # s = y
         ((47, 30, 12), ("DD", "NN", "P"), None), ((191, 18, 10), ("DN", "P", "P"), None),    # s = x
         ((480, 6, 10), ("DD", "NN", "P"), None)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


def _fields(prob, seed):
    u, v, w = inputs.prediction_velocity(prob, seed)
    return u, v, w, np.random.default_rng(seed + 1).uniform(-1, 1, prob.shape)


def _correct(prob, arrays, gdt, refined=False, whole=True):
    import torch
    from paper_1802_10323_amd import FP32_REFINED, Plan
    plan = Plan.from_problem(prob)
    if refined:
        plan.set_precision(FP32_REFINED, 1e-10, 6)
    du, dv, dw, dp = (to_dev(a) for a in arrays)
    phi = torch.empty(prob.points, dtype=torch.float64, device="cuda")
    if whole:
        plan.pressure_correction(du, dv, dw, dp, gdt, phi)
    else:
        plan.projection_rhs(du, dv, dw, gdt, phi)
        plan.solve(phi)
        plan.projection_update(phi, gdt, du, dv, dw, dp)
    out = [to_host(t) for t in (du, dv, dw, dp, phi)]
    plan.close()
    return out


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + "-" + "".join(c[1]))
def test_padded_lines(case, monkeypatch):
    from oracle import projection as pj
    shape, bcs, stretch = case
    prob = inputs.make_uniform(*shape, bcs, seed=sum(shape), stretch_z=stretch, with_rhs=False)
    arrays = _fields(prob, sum(shape))
    ref = pj.pressure_correction(*arrays, 0.37, prob.hx, prob.hy, prob.hz, prob.bcs)
    got = _correct(prob, arrays, 0.37)
    for name, g, r in zip(("u", "v", "w", "p", "phi"), got, ref):
        assert rel_l2(g.reshape(r.shape), r) <= 1e-12, (name, rel_l2(g.reshape(r.shape), r))
    monkeypatch.setenv("POISSON_GRID_CAP", "16")
    assert all(np.array_equal(a, b) for a, b in zip(_correct(prob, arrays, 0.37), got))


@pytest.mark.parametrize("shape,bcs", [((64, 60, 50), ("P", "NN", "NN")), ((54, 36, 33), ("NN", "P", "DD"))])
def test_refined_correction_is_the_three_calls(shape, bcs):
    prob = inputs.make_uniform(*shape, bcs, seed=sum(shape), with_rhs=False)
    arrays = _fields(prob, sum(shape))
    for a, b in zip(_correct(prob, arrays, 0.37, refined=True),
                    _correct(prob, arrays, 0.37, refined=True, whole=False)):
        assert np.array_equal(a, b)
