"""Every chunking of the elimination of lines of any length (tri_line_shape in
csrc/tri_line.h): for each count of chunks P and of rows per chunk, the lengths
whose chunks are all whole, all but one, and one only, as far as they lie in the
range of P; and both sides of each range's ends.  The lengths with variants are
among them (64, 96, 128, 192, 256, 384, 512): their strided lines take this
kernel too while nothing is tuned or set.  The stage alone (backward error of
every regular line <= 1e-14 and the conditioned forward bound), two blocks, so
that each loops over tiles."""
import pytest

from conftest import ELIM_LENGTHS
from gpu_util import check_elimination

pytestmark = pytest.mark.gpu

RANGES = ((17, 48, 4), (49, 96, 8), (97, 176, 16), (177, 192, 16), (193, 256, 16), (257, 352, 32),
          (353, 512, 32))    # first and last length, chunks


def lengths():
    found = set()
    for first, last, p in RANGES:
        found |= {first, last}
        for rows in range(-(-first // p), -(-last // p) + 1):
            found |= {n for n in (rows * p, rows * p - 1, rows * p - p + 1) if first <= n <= last}
    return sorted(found)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


def test_lengths_cover_the_ones_with_variants():
    assert set(ELIM_LENGTHS) <= set(lengths())


@pytest.mark.parametrize("n", lengths())
def test_every_chunking(n, monkeypatch):
    from paper_1802_10323_amd import tuned_entry
    if n in ELIM_LENGTHS:
        assert tuned_entry(1, n, 0) == -1
    monkeypatch.setenv("POISSON_GRID_CAP", "2")
    check_elimination(n, "NN")                              # singular lines and regular ones
    check_elimination(n, ("P", "DD", "ND", "DN")[n % 4])
