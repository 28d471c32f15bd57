"""The tile raster's per-lane and wave-wide sample tests and its tile groups.

CPU: the record it forms per (triangle, tile) -- edges 1 and 2 relative to the
tile's first pixel, edge 0 as A - E_1 - E_2, one subtracted on edges that are
neither top nor left -- decides every sample as the 64-bit integer definition
does.  GPU: keys equal the oracle's bit for bit on a triangle soup whose boxes
straddle every size at which a triangle changes from the per-lane to the
wave-wide test, on tiles crowded past one workgroup's worth of entries, and on
views that end inside a tile or a group of tiles, at every tile side."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import gpu_run, oracle_run

SUB = 256


def _edge(xa, ya, xb, yb, px, py):
    return (xb - xa) * (py - ya) - (yb - ya) * (px - xa)


def test_record_matches_integer_definition():
    rng = np.random.default_rng(11)
    lim = 32768 * SUB - 1
    for case in range(6000):
        ox, oy = (int(v) * 8 for v in rng.integers(0, 1024, 2))
        if case % 3 == 0:       # the whole admitted range
            X, Y = ([int(v) for v in rng.integers(-lim, lim + 1, 3)] for _ in range(2))
        elif case % 3 == 1:     # small, near the tile, on sample centres (zero edge values)
            X = [ox * SUB + 128 + SUB * int(v) for v in rng.integers(-9, 18, 3)]
            Y = [oy * SUB + 128 + SUB * int(v) for v in rng.integers(-9, 18, 3)]
        else:
            X = [ox * SUB + int(v) for v in rng.integers(-3000, 6000, 3)]
            Y = [oy * SUB + int(v) for v in rng.integers(-3000, 6000, 3)]
        A = (X[1] - X[0]) * (Y[2] - Y[0]) - (Y[1] - Y[0]) * (X[2] - X[0])
        if A == 0:
            continue
        if A < 0:
            X[1], X[2], Y[1], Y[2], A = X[2], X[1], Y[2], Y[1], -A
        ends = [(1, 2), (2, 0), (0, 1)]
        tl = [Y[b] < Y[a] or (Y[b] == Y[a] and X[b] > X[a]) for a, b in ends]
        t = [0.0 if q else 1.0 for q in tl]
        f = np.float64
        a1, b1, a2, b2 = f(Y[2] - Y[0]), f(X[0] - X[2]), f(Y[0] - Y[1]), f(X[1] - X[0])
        px0, py0 = f(ox * SUB), f(oy * SUB)
        c1 = a1 * (px0 - f(X[2])) + (b1 * (py0 - f(Y[2])) - t[1])
        c2 = a2 * (px0 - f(X[0])) + (b2 * (py0 - f(Y[0])) - t[2])
        Am = f(A) - ((t[0] + t[1]) + t[2])
        for x, y in rng.integers(0, 8, (6, 2)):
            sx, sy = f(int(x) * SUB + 128), f(int(y) * SUB + 128)
            e1 = a1 * sx + (b1 * sy + c1)
            e2 = a2 * sx + (b2 * sy + c2)
            e0 = (Am - e1) - e2
            px, py = (ox + int(x)) * SUB + 128, (oy + int(y)) * SUB + 128
            E = [_edge(X[a], Y[a], X[b], Y[b], px, py) for a, b in ends]
            assert [int(e0 + t[0]), int(e1 + t[1]), int(e2 + t[2])] == E
            inside = all(v > 0 or (v == 0 and q) for v, q in zip(E, tl))
            assert inside == (not (np.signbit(e0) or np.signbit(e1) or np.signbit(e2)))


def _soup(w, h, res, n=700):
    """Triangles of 1 to about 60 samples a side at random depths over the
    view, facing the camera, above a ground quad."""
    rng = np.random.default_rng([5, w, h])
    size = np.exp(rng.uniform(np.log(0.01), np.log(0.5), n))
    c = np.stack([rng.uniform(-1.2, 1.2, n), rng.uniform(0.1, 1.5, n), rng.uniform(-1.2, 1.2, n)], 1)
    v = (c[:, None, :] + size[:, None, None] * rng.uniform(-0.5, 0.5, (n, 3, 3))).reshape(-1, 3)
    f = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    v, f = sg.merge([(v, f), sg.quad(2.0)])
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    b.lights[0].resolution, b.lights[0].k = res, 1
    b.cameras[0].width, b.cameras[0].height = w, h
    return b


def _crowded():
    """9k triangles on about two dozen 8 x 8 tiles: hundreds of entries a tile."""
    b = sg.config2(n_scenes=1, resolution=64, with_pose=False)
    b.cameras[0].width, b.cameras[0].height = 61, 43
    return b


def _stacked():
    """600 triangles at random heights, each over most of a small view, and four
    small ones after each: some hundred boxes of more samples than a lane
    tests alone in every chunk of a tile's entries, more than the shared list
    holds at once."""
    rng = np.random.default_rng(23)
    parts = []
    for y in rng.uniform(0.0, 1.0, 600):
        parts.append(np.array([[-5, y, -3], [0, y + rng.uniform(-.2, .2), 2.8], [5, y, -3]]))
        for x, z in rng.uniform(-1.5, 1.5, (4, 2)):
            parts.append(np.array([[x, y, z], [x, y, z + .5], [x + .5, y, z]]))
    v = np.concatenate(parts)
    f = np.arange(len(v), dtype=np.int32).reshape(-1, 3)
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    b.lights[0].resolution, b.lights[0].k = 9, 1
    b.cameras[0].width, b.cameras[0].height = 21, 13
    return b


CASES = {'soup': lambda: _soup(250, 190, 200), 'soup_narrow': lambda: _soup(67, 9, 33), 'one_pixel': lambda: _soup(1, 1, 1),
         'crowded': _crowded, 'stacked': _stacked}


@pytest.mark.gpu
@pytest.mark.parametrize('tile', [8, 16, 32])
@pytest.mark.parametrize('name', list(CASES))
def test_keys_match_oracle(name, tile):
    b = CASES[name]()
    g, o = gpu_run(b, tile_size=tile), oracle_run(b)
    for v, (kg, ko) in enumerate(zip(g['keys'], o['keys'])):
        assert kg.shape == ko.shape and np.array_equal(kg, ko), f'view {v}: {int((kg != ko).sum())} keys differ'
    assert g['stats']['overflow'] == 0
