"""The orders in which workgroups take their items, as the kernels' own functions
(csrc/xcd_order.h, compiled for the host) give them: every item once, for grids
around every size at which the order changes; ranges and turns give each XCD
(workgroups b with equal b % 8) neighbouring items."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope='module')
def items(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp('host') / 'xcd_order.so')
    subprocess.run(['g++', '-O1', '-std=c++17', '-shared', '-fPIC', '-D__HIP_PLATFORM_AMD__=1', '-I/opt/rocm/include',
                    '-I' + os.path.join(ROOT, 'paper_2308_10896_amd', 'csrc'),
                    os.path.join(ROOT, 'tests', 'xcd_order_host.cpp'), '-o', lib], check=True)
    fn = ctypes.CDLL(lib).xcd_items

    def run(form, gx, gy):
        out = np.full(gx * gy, -1, np.int32)
        fn(form, gx, gy, out.ctypes.data_as(ctypes.c_void_p))
        return out
    return run


@pytest.mark.parametrize('form', range(5))
def test_every_item_once(items, form):
    for gx in (1, 7, 8, 127, 128, 129, 183, 184, 185, 1023, 1024, 1025, 2049, 4096, 8193):
        for gy in (1, 2, 3, 7, 8, 9, 16, 31, 32, 33):
            n = gx * gy
            assert np.array_equal(np.sort(items(form, gx, gy)), np.arange(n)), (gx, gy)


def test_neighbours_share_an_xcd(items):
    b = np.arange(24576)
    ranges, turns, grid = items(0, len(b), 1), items(1, len(b), 1), items(2, len(b), 1)
    for xcd in range(8):
        mine = ranges[b % 8 == xcd]
        assert np.array_equal(mine, np.arange(mine[0], mine[0] + len(b) // 8))
        for order, run in ((turns, 23), (grid, 128)):
            m = order[b % 8 == xcd][: len(b) // 8 // run * run - run].reshape(-1, run)
            assert (np.diff(m, axis=1) == 1).all() and (np.diff(m[:, 0]) == 8 * run).all()
