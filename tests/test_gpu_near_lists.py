"""Flagged pairs found on the device: the same list, in order, as by their definition."""
import numpy as np
import pytest

from near_lists import CASES, expected, mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,factor", CASES)
def test_device_list(bie, name, factor):
    V, T = mesh(name)
    op = bie.Operator(V, T, 0.1, storage="c64", near_factor=factor)
    got = op.near_pairs()
    op.close()
    assert np.array_equal(got, expected(V, T, factor))
