import contextlib
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


FAST_M = [16, 32, 48, 64, 72, 80, 96, 128, 144, 160, 192, 256]
ELIM_LENGTHS = [64, 96, 128, 192, 256, 384, 512]


TABLE_KEYS = ([(0, 2 * M, layout, fp64) for M in FAST_M for layout in (0, 1) for fp64 in (True, False)]
              + [(1, n, layout, fp64) for n in ELIM_LENGTHS for layout in (0, 1) for fp64 in (True, False)])


@contextlib.contextmanager
def variants():
    """Solves run the kernel variants: an entry of the table that nothing set
    holds the variant that it names (solves of its length would otherwise run
    the length's own kernels, which a batch does not have).  Afterwards every
    entry is what it was, an unset one unset."""
    from paper_1802_10323_amd import set_tuned_entry, set_tuned_variant, tuned_entry, tuned_variant
    saved = [(k, tuned_entry(*k)) for k in TABLE_KEYS]
    for (family, n, layout, fp64), _ in saved:
        set_tuned_variant(family, n, layout, tuned_variant(family, n, layout, fp64), fp64)
    try:
        yield
    finally:
        for (family, n, layout, fp64), entry in saved:
            set_tuned_entry(family, n, layout, entry, fp64)


@pytest.fixture
def default_variants():
    """The test runs on the kernel variants, and every entry of the table is
    put back to what it was before the test."""
    with variants():
        yield


def pytest_collection_modifyitems(items):
    # compares a tuned batch with single solves to 1e-14, which holds where
    # both run the variants
    for item in items:
        if item.name == "test_batch_autotune_whole_batch":
            item.fixturenames.append("default_variants")
