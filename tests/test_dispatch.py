"""Which kernels a call takes, on the host: the library's own rules, called with the shapes on
both sides of each line (no GPU needed)."""
import pytest

from parity import one_workgroup_selection

UNITS = [(1, 1), (1, 8), (8, 8), (15, 8), (16, 8), (25, 8), (32, 8), (256, 1), (64, 8), (256, 8),
         (48, 3)]


@pytest.mark.parametrize("batch,hkv", UNITS)
def test_selection_of_wide_tables_is_split(batch, hkv):
    """One workgroup per unit lasts as long as the longest unit that the table admits, whatever
    the batch's other lengths: past 512 pages the split kernels are used at every unit count."""
    for width in (513, 768, 1024, 2047, 2048, 2049, 4096, 15360):
        assert not one_workgroup_selection(batch, hkv, width), width


@pytest.mark.parametrize("batch,hkv", UNITS)
def test_selection_of_narrow_tables_is_one_workgroup(batch, hkv):
    for width in (1, 63, 64, 448):
        assert one_workgroup_selection(batch, hkv, width), width
    for width in (449, 512):
        assert one_workgroup_selection(batch, hkv, width) == (batch * hkv >= 128), width


def test_thousands_of_short_units_are_split():
    assert not one_workgroup_selection(512, 8, 63)
    assert one_workgroup_selection(512, 8, 64)
    assert one_workgroup_selection(256, 8, 63)
