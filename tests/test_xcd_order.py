"""The orders in which workgroups take their items (a contiguous range per XCD,
or XCDs in turns of RUN items) name every item once, for any number of them."""
import numpy as np
import pytest


def remap(b, n):
    xcd, idx, per, rem = b % 8, b // 8, n // 8, n % 8
    return np.where(xcd < rem, xcd * (per + 1) + idx, rem * (per + 1) + (xcd - rem) * per + idx)


def turns(b, n, run):
    turn = 8 * run
    whole = n // turn * turn
    t = b // turn * turn + b % 8 * run + b // 8 % run
    return np.where(b < whole, t, whole + remap(b - whole, n - whole))


@pytest.mark.parametrize('run', [16, 23, 128])
def test_orders_are_bijections(run):
    for n in [1, 7, 8, 9, 8 * run - 1, 8 * run, 8 * run + 1, 8 * run + 9, 24 * run + 5, 2049, 4097]:
        b = np.arange(n)
        assert np.array_equal(np.sort(remap(b, n)), b)
        assert np.array_equal(np.sort(turns(b, n, run)), b)
