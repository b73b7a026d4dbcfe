"""The views of the binning tests take the binning that they are there for."""
import pytest

import binning_cases as bc
from layout_probe import layouts


@pytest.mark.parametrize("cases,path", [(bc.TWO_LEVELS, "two levels"), (bc.ROWS, "rows")])
def test_cases_take_their_binning(cases, path):
    got = layouts([bc.layout_request(c) for c in cases.values()])
    assert {k: L["path"] for k, L in zip(cases, got)} == {k: path for k in cases}


def test_overflow_cases_cover_the_three_binnings():
    got = layouts([bc.layout_request(c) for c in bc.OVERFLOW.values()])
    assert [L["path"] for L in got] == list(bc.OVERFLOW)


def test_batch_views_are_binned_in_two_levels():
    got = layouts([(bc.BATCH_N, bc.BATCH_CAPACITY, w, h, d, ox, oy, bc.BATCH_TILE)
                   for w, h, d, ox, oy in bc.BATCH_VIEWS])
    assert [L["path"] for L in got] == ["two levels"] * len(bc.BATCH_VIEWS)
