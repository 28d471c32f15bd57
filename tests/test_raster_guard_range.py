"""The raster's sample tests over the whole range of screen coordinates that the
setup admits (|X|, |Y| < 2^23 in 1/256 pixel), where an edge spans up to 65,536
pixels and its function changes by up to 2^32 from one sample to the next.

CPU: the functions of csrc/raster_tri.h, compiled for the host, against the
64-bit integer definition of coverage and the float32 depth.  GPU: keys equal
the oracle's bit for bit where lanes test such triangles alone (few samples of a
view's last tile beside small triangles; more than 48 whole tiles in a wave)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import scenegen as sg
from parity_helpers import gpu_run, oracle_run

SUB, LIM = 256, 32768 * 256 - 1
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SETUP = np.dtype([('A', 'i8'), ('X', 'i4', 3), ('Y', 'i4', 3), ('z', 'f4', 3), ('box', 'u2', 4), ('facing', 'i1'),
                  ('rest', 'u1', 3), ('pad', 'i4', 2)])


@pytest.fixture(scope='module')
def host(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp('host') / 'raster_tri.so')
    subprocess.run(['g++', '-O1', '-std=c++17', '-shared', '-fPIC', '-ffp-contract=off', '-D__HIP_PLATFORM_AMD__=1',
                    '-I/opt/rocm/include', '-I' + os.path.join(ROOT, 'paper_2308_10896_amd', 'csrc'),
                    os.path.join(ROOT, 'tests', 'raster_tri_host.cpp'), '-o', lib], check=True)
    return ctypes.CDLL(lib)


def _cases(kind, n=4000):
    """n oriented triangles as setup records, tile origins and boxes."""
    rng = np.random.default_rng([17, len(kind)])
    o = rng.integers(0, 1024, (n, 2)) * 8
    base = o[:, None, :] * SUB
    if kind == 'random':                    # corners anywhere
        p = rng.integers(-LIM, LIM + 1, (n, 3, 2))
    elif kind == 'through':                 # long edges through the tile: one corner near it, two far away
        p = rng.integers(-LIM, LIM + 1, (n, 3, 2))
        p[:, 0] = base[:, 0] + rng.integers(-1000, 3000, (n, 2))
    elif kind == 'around':                  # the tile deep inside, or at a diagonal through it
        far = rng.integers(2 ** 22, LIM, (n, 3, 2))
        p = np.stack([-far[:, 0], far[:, 1], far[:, 2] * np.array([1, -1])], 1)
        p[::2, 2] = -p[::2, 1] + 2 * base[::2, 0] + rng.integers(-2000, 4000, (len(p[::2]), 2))
        p = np.clip(p, -LIM, LIM)
    else:                                   # extremes of the range
        p = rng.choice([-LIM, -LIM // 2, 0, LIM // 2, LIM], (n, 3, 2))
    p = p.astype(np.int64)
    A = ((p[:, 1, 0] - p[:, 0, 0]) * (p[:, 2, 1] - p[:, 0, 1]) - (p[:, 1, 1] - p[:, 0, 1]) * (p[:, 2, 0] - p[:, 0, 0]))
    p[A < 0] = p[A < 0][:, [0, 2, 1]]
    keep = A != 0
    p, A, o = p[keep], np.abs(A[keep]), o[keep]
    t = np.zeros(len(p), SETUP)
    t['A'], t['X'], t['Y'] = A, p[:, :, 0], p[:, :, 1]
    t['z'] = rng.uniform(-0.2, 1.2, (len(p), 3)).astype(np.float32)
    x, y = np.sort(rng.integers(0, 8, (len(p), 2))), np.sort(rng.integers(0, 8, (len(p), 2)))
    x[::2], y[::2] = [0, 7], [0, 7]
    return t, o.astype(np.int32), np.concatenate([x, y], 1).astype(np.int32)


@pytest.mark.parametrize('kind', ['random', 'through', 'around', 'extremes'])
def test_host_functions_match_integer_definition(host, kind):
    t, o, box = _cases(kind)
    n = len(t)
    assert SETUP.itemsize == 64 and n > 1000
    X, Y = t['X'].astype(np.int64), t['Y'].astype(np.int64)
    assert (np.abs(Y[:, [2, 0]] - Y[:, [0, 1]]) >= 2 ** 23).any(1).sum() > 300
    stepped, direct = np.zeros((n, 64), np.uint64), np.zeros((n, 64), np.uint64)
    touch = np.zeros(n, np.uint8)
    host.raster_tri_keys(n, *(a.ctypes.data_as(ctypes.c_void_p) for a in (t, o, box, stepped, direct, touch)))

    # every sample of the tile: coverage in int64, the depth in float32 from 1 / A
    q = np.arange(64)
    px, py = (o[:, :1] + q % 8) * SUB + SUB // 2, (o[:, 1:] + q // 8) * SUB + SUB // 2
    inside, E = np.ones((n, 64), bool), []
    for a, b in ((1, 2), (2, 0), (0, 1)):
        dx, dy = X[:, b] - X[:, a], Y[:, b] - Y[:, a]
        e = dx[:, None] * (py - Y[:, a, None]) - dy[:, None] * (px - X[:, a, None])
        inside &= (e > 0) | ((e == 0) & ((dy < 0) | ((dy == 0) & (dx > 0)))[:, None])
        E.append(e)
    rA = (np.float32(1) / t['A'].astype(np.float32))[:, None]
    z = t['z'][:, :, None]
    z01 = (z[:, 0] + (E[1].astype(np.float32) * rA) * (z[:, 1] - z[:, 0])) \
        + (E[2].astype(np.float32) * rA) * (z[:, 2] - z[:, 0])
    inbox = (q % 8 >= box[:, :1]) & (q % 8 <= box[:, 1:2]) & (q // 8 >= box[:, 2:3]) & (q // 8 <= box[:, 3:])
    cover = inside & inbox & (z01 >= 0) & (z01 <= 1)
    want = np.where(cover, ((z01.view(np.uint32) & 0x7fffffff).astype(np.uint64) << np.uint64(32)) | np.uint64(7),
                    ~np.uint64(0))
    assert np.array_equal(direct, want)
    assert np.array_equal(stepped, want), f'{int((stepped != want).sum())} samples differ'
    assert touch[(inside & inbox).any(1)].all()
    assert kind == 'random' or cover.sum() > 1000


def _ground(res, n=300, layers=0):
    """A ground quad of some 16,800 pixels on each side of a directional light's
    map of `res` pixels, its diagonal through the map, under n triangles of a few
    pixels spread over the map and its last columns; `layers` more such quads."""
    rng = np.random.default_rng([31, res, layers])
    px = 0.06 / res                                    # a pixel of the map
    half = 16800 * px
    parts = []
    for k in range(1 + layers):
        v, f = sg.quad(half)
        dx, dz = rng.uniform(-res / 4, res / 4, 2) * px
        v = v + np.array([dx, -0.03 * k + rng.uniform(-0.01, 0.01), dz])
        v[:, 1] += 0.02 * v[:, 0] / half               # not level: the depth order follows the weights
        parts.append((v, f))
    c = rng.uniform(-0.03, 0.03, (n, 2))
    c[: n // 2] = rng.uniform(0.03 - 10 * px, 0.03, (n // 2, 2))
    c[: n // 4] *= rng.choice([-1, 1], (n // 4, 2))
    tri = np.stack([c[:, 0], rng.uniform(-0.3, 0.3, n), c[:, 1]], 1)[:, None, :] + \
        4 * px * rng.uniform(-1, 1, (n, 3, 3)) * np.array([1, 0.1, 1])
    parts.append((tri.reshape(-1, 3), np.arange(3 * n, dtype=np.int32).reshape(n, 3)))
    v, f = sg.merge(parts)
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v.astype(np.float32), faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    b.lights = [sg.Light('directional', sg.f32([0, -1, 0]), resolution=res, k=1, ortho_half=0.03,
                         up=sg.f32([0, 0, 1]))]
    b.cameras[0].eye, b.cameras[0].width, b.cameras[0].height = sg.f32([0.3, 0.4, 0.2]), 34, 18
    return b


@pytest.mark.gpu
@pytest.mark.parametrize('tile', [8, 16, 32])
@pytest.mark.parametrize('res,n,layers', [(66, 300, 0), (65, 300, 3), (34, 40, 60), (16, 4, 200)])
def test_keys_of_huge_triangles_match_oracle(res, n, layers, tile):
    b = _ground(res, n, layers)
    g, o = gpu_run(b, tile_size=tile, bin_scale=256), oracle_run(b)
    assert g['stats']['overflow'] == 0
    for v, (kg, ko) in enumerate(zip(g['keys'], o['keys'])):
        assert kg.shape == ko.shape and np.array_equal(kg, ko), f'view {v}: {int((kg != ko).sum())} keys differ'
    assert (np.abs(np.diff(g['verts'][:4, 0])) > 33000 * 0.06 / res).any()
