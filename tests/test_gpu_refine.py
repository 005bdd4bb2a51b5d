"""The sweeps of the refined solve at the edges of their access widths and
tiles: odd and even x extents (single points and pairs per access), fewer
points than a block, rows that are no multiple of a block's, one plane, marches
of one to many planes.  Singular problems (the mean of f at the start, the mean
of Phi from the last update, or from a sum of its own after a single FP32
solve), regular ones, each against the oracle (<= 1e-10 refined; one FP32 solve
within 4 transforms x 13 rounding steps x 2^-24), and the zero weighted mean of a
singular solution: at most the rounding of an FP64 sum over N values, N 2^-53 of
the mean modulus."""
import numpy as np
import pytest

from gpu_util import gpu_solve, oracle_solve, rel_l2
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu

# (shape, boundary pairs, stretch of z)
CASES = [((45, 16, 10), ("NN", "P", "P"), None),      # odd x (eliminated), singular
         ((33, 20, 6), ("DN", "P", "P"), None),       # odd x, regular
         ((36, 20, 33), ("P", "NN", "NN"), 1.8),      # pairs, stretched weights
         ((144, 18, 40), ("P", "P", "NN"), 1.8),      # more than one block along x
         ((4, 6, 5), ("NN", "NN", "NN"), None),       # less than a block
         ((24, 50, 1), ("P", "P", "NN"), None),       # one plane
         ((300, 90, 64), ("P", "P", "NN"), 1.8)]      # several runs per thread


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
def test_refined_sweeps(case):
    from paper_1802_10323_amd import Plan
    shape, bcs, stretch = case
    prob = inputs.make_uniform(*shape, bcs, seed=sum(shape), stretch_z=stretch)
    singular = inputs.has_null_space(*bcs)
    if singular:
        prob.rhs = prob.rhs + 0.75                    # a mean for the projection to take out
    plan = Plan.from_problem(prob)
    ref = oracle_solve(prob, plan.roles)
    plan.close()
    got, (_, _, converged) = gpu_solve(prob, mixed=True)
    once, _ = gpu_solve(prob, mixed=True, max_iters=1)
    assert converged and rel_l2(got, ref) <= 1e-10
    assert rel_l2(once, ref) <= 4 * 13 * 2.0 ** -24
    if singular:
        for phi in (got, once):
            w = np.broadcast_to(prob.hz[:, None, None], phi.shape)
            assert abs((w * phi).sum()) <= phi.size * 2.0 ** -53 * np.abs(w * phi).sum()
