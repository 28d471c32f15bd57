"""The stand-alone filter on both sides of the number of tiles at which its
tile height changes (wide filters), at map sides that end inside a tile of
either height.  Forward against a float64 filter by clamped indexing, the
transpose as its exact adjoint; bound: k products and sums a direction, each
within u = 2^-24, so 2 (k + 1) u times the filter of the absolute values."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _line(S, k):
    """Matrix of the one-dimensional Gaussian filter with the kernel's float32 taps."""
    r, s = (k - 1) // 2, (k - 1) / 3.0
    t = np.exp(-np.arange(-r, r + 1) ** 2 / (2 * s * s))
    t = (t / t.sum()).astype(np.float32).astype(np.float64)
    m = np.zeros((S, S))
    for i in range(k):
        np.add.at(m, (np.arange(S), np.clip(np.arange(S) + i - r, 0, S - 1)), t[i])
    return m


@pytest.mark.parametrize('adjoint', [False, True])
@pytest.mark.parametrize('n,S,k', [(1, 17, 15), (2, 130, 11), (62, 127, 13), (64, 127, 13), (3, 515, 31)])
def test_filter_against_float64(n, S, k, adjoint):
    from paper_2308_10896_amd import dsm
    maps = np.random.default_rng([n, S, k]).standard_normal((n, 2, S, S)).astype(np.float32)
    got = dsm.filter_moments(torch.as_tensor(maps).cuda(), 'gaussian', k, 0.0, adjoint).cpu().numpy()
    m = _line(S, k)
    m = m.T if adjoint else m
    want = m @ maps.astype(np.float64) @ m.T
    # the transpose adds the clamped taps as up to k more terms a direction
    bound = 2 * (2 * k + 1 if adjoint else k + 1) * 2.0 ** -24 * (np.abs(m) @ np.abs(maps) @ np.abs(m.T))
    assert (np.abs(got - want) <= bound).all()
