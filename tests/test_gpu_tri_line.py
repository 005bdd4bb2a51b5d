"""Elimination of lines of any length in chunks of their own (17 <= n <= 512
without a size-specialised kernel): the edges of every chunking (all chunks
whole, one short, all but one short), every boundary pair, singular and
regular, cyclic, uniform and stretched, strided and contiguous lines.  The
stage alone with the checks of the other eliminations (backward error of
every regular line <= 1e-14, the conditioned forward bound), and whole solves
against the oracle and the size-generic kernel (each <= 1e-12 of the oracle),
with the grid capped so that blocks loop over tiles, and in FP32 +
refinement, whose eliminations run in FP64 arithmetic."""
import numpy as np
import pytest

from gpu_util import check_elimination, gpu_solve, oracle_solve, rel_l2
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu

KINDS = ("P", "NN", "DD", "ND", "DN")
# 8 lanes: 17 (all but one short), 24 (whole), 25, 32; 16: 33, 47, 50, 144 (whole), 175, 176;
# 32: 177, 193, 224, 351, 352; 64: 353, 383, 385, 448, 449, 511
LENGTHS = (17, 24, 25, 32, 33, 47, 50, 144, 175, 176, 177, 193, 224, 351, 352, 353, 383, 385, 448, 449, 511)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("kind", KINDS)
def test_elimination_stage(kind, n):
    check_elimination(n, kind)


SOLVES = [((36, 24, 144), ("P", "P", "NN"), 1.8), ((30, 50, 33), ("NN", "NN", "NN"), None),
          ((18, 10, 353), ("P", "P", "P"), 1.8), ((177, 20, 24), ("P", "P", "P"), None),
          ((47, 30, 12), ("DD", "NN", "P"), None), ((45, 16, 10), ("NN", "P", "P"), None),
          ((20, 175, 6), ("P", "NN", "P"), None), ((36, 2, 25), ("P", "P", "DN"), None)]


@pytest.mark.parametrize("case", SOLVES, ids=lambda c: "x".join(map(str, c[0])) + "".join(c[1]))
def test_solve(case, monkeypatch):
    from paper_1802_10323_amd import Plan
    shape, bcs, stretch = case
    prob = inputs.make_uniform(*shape, bcs, seed=sum(shape), stretch_z=stretch)
    plan = Plan.from_problem(prob)
    ref = oracle_solve(prob, plan.roles)
    plan.close()
    got, _ = gpu_solve(prob)
    monkeypatch.setenv("POISSON_GENERIC_TRI", "1")
    generic, _ = gpu_solve(prob)
    monkeypatch.delenv("POISSON_GENERIC_TRI")
    assert rel_l2(got, ref) <= 1e-12 and rel_l2(generic, ref) <= 1e-12
    monkeypatch.setenv("POISSON_GRID_CAP", "1")
    assert np.array_equal(gpu_solve(prob)[0], got)
    mixed, (_, _, converged) = gpu_solve(prob, mixed=True)
    assert converged and rel_l2(mixed, ref) <= 1e-10


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_infinities_and_nans_spread_as_in_the_generic_kernel(bad, monkeypatch):
    """A line with an infinity or a NaN among its rows comes out without a
    finite value, also where the reduction ends early (strong shift), and no
    other line does."""
    from gpu_util import to_dev, to_host
    from paper_1802_10323_amd import Plan
    f = np.random.default_rng(3).uniform(-1.0, 1.0, (144, 20, 36))
    f[70, 3, 5] = bad
    masks = []
    for generic in ("0", "1"):
        monkeypatch.setenv("POISSON_GENERIC_TRI", generic)
        plan = Plan(36, 20, 144, 0.1, 0.1, np.full(144, 1.0), ("P", "P", "NN"))
        d = to_dev(f)
        plan.tridiag_stage(d)
        masks.append(np.isfinite(to_host(d)))
        plan.close()
    assert not masks[0][:, 3, 5].any() and masks[0].sum() == f.size - 144
    assert np.array_equal(*masks)
