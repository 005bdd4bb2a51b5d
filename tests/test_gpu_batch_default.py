"""A batch against single solves on a table that nothing set: the batch runs
the kernel variants, the single solves the lengths' own kernels, whose pivots are
the more exact.  Each is within 1e-12 of the oracle (the solve's bound), and so
the two within 2e-12 of each other."""
import pytest

from conftest import TABLE_KEYS
from gpu_util import gpu_solve, oracle_solve, rel_l2, to_dev, to_host
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


@pytest.mark.parametrize("seed", [1, 11])
def test_default_batch_and_default_single_solves(seed):
    from paper_1802_10323_amd import Batch, Plan, tuned_entry
    assert all(tuned_entry(*k) == -1 for k in TABLE_KEYS)
    probs = inputs.batch(seed, count=6)
    plans = [Plan.from_problem(p) for p in probs]
    fields = [to_dev(p.rhs) for p in probs]
    batch = Batch(plans)
    batch.bind(fields)
    batch.launch()
    for p, f in zip(probs, fields):
        got, (single, _), ref = to_host(f), gpu_solve(p), oracle_solve(p)
        print(p, "batch", rel_l2(got, ref), "single", rel_l2(single, ref), "between", rel_l2(got, single), flush=True)
        assert rel_l2(got, ref) <= 1e-12 and rel_l2(single, ref) <= 1e-12
        assert rel_l2(got, single) <= 2e-12
    batch.close()
    for pl in plans:
        pl.close()
