"""The kernel-variant table without a GPU: an entry that nothing set is told
from one that holds its default variant, and any entry can be written back as it
was; the fixture of the variant tests leaves the table as it found it."""
import os

import pytest

from conftest import TABLE_KEYS, variants
from paper_1802_10323_amd import poisson as P

pytestmark = pytest.mark.skipif(not os.path.exists(P.LIB_PATH), reason="library not built")


def test_entries_are_written_back_as_they_were():
    for key in ((0, 64, 0, True), (0, 512, 1, False), (1, 256, 0, True)):
        family, n, layout, fp64 = key
        assert P.tuned_entry(*key) == P.UNSET
        default = P.tuned_variant(*key)
        P.set_tuned_variant(family, n, layout, default, fp64)
        assert P.tuned_entry(*key) == default           # set by hand, though to the default
        P.set_tuned_entry(family, n, layout, P.UNSET, fp64)
        assert P.tuned_entry(*key) == P.UNSET and P.tuned_variant(*key) == default
    P.set_tuned_entry(1, 192, 0, 1 + P.LINE_FASTER)
    assert P.tuned_entry(1, 192, 0) == 1 + P.LINE_FASTER and P.tuned_variant(1, 192, 0) == 1
    P.set_tuned_entry(1, 192, 0, P.UNSET)


@pytest.mark.parametrize("family,n,entry,code", [
    (0, 64, 8, P.EINVAL), (0, 64, -2, P.EINVAL), (1, 64, 4, P.EINVAL), (1, 64, 4 + P.LINE_FASTER, P.EINVAL),
    (2, 64, 0, P.EINVAL), (0, 270, P.UNSET, P.EUNSUPPORTED), (1, 144, 0, P.EUNSUPPORTED),
    (0, 512, P.LINE_FASTER, P.EUNSUPPORTED)])
def test_refused_entries(family, n, entry, code):
    with pytest.raises(P.PoissonError) as e:
        P.set_tuned_entry(family, n, 0, entry)
    assert e.value.code == code


def test_fixture_leaves_the_table_as_it_was():
    P.set_tuned_entry(0, 128, 1, 3 + P.LINE_FASTER)
    P.set_tuned_entry(1, 64, 0, 1)
    before = [P.tuned_entry(*k) for k in TABLE_KEYS]
    assert P.UNSET in before
    with variants():
        inside = [P.tuned_entry(*k) for k in TABLE_KEYS]
        assert all(0 <= e < P.LINE_FASTER for e in inside)
        assert inside == [P.tuned_variant(*k) for k in TABLE_KEYS]
        P.set_tuned_variant(0, 64, 0, 2)
    assert [P.tuned_entry(*k) for k in TABLE_KEYS] == before
    for k in ((0, 128, 1), (1, 64, 0)):
        P.set_tuned_entry(*k, P.UNSET)
