"""Per-(triangle, tile) sums of samples that share a triangle: tessellated
planes whose triangles hold from one to some forty samples of a tile (sums by
atomics, with neighbours added first, and by the whole wave), partly turned
away from the light, against the oracle and against the sums of larger tiles."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import GRAD_TOL, check_gradients, gpu_grads, normwise, oracle_run, random_grad

pytestmark = pytest.mark.gpu


def _batch(n, channels):
    """An n x n grid of quads with a fold, above a ground quad."""
    u = np.linspace(-1.0, 1.0, n + 1)
    x, z = np.meshgrid(u, u, indexing='ij')
    y = 0.5 + 0.9 * np.abs(x + 0.1)
    v = np.stack([x, y, z], -1).reshape(-1, 3)
    i, j = (a.reshape(-1) for a in np.meshgrid(np.arange(n), np.arange(n), indexing='ij'))
    a, b, c, d = i * (n + 1) + j, i * (n + 1) + j + 1, (i + 1) * (n + 1) + j, (i + 1) * (n + 1) + j + 1
    f = np.concatenate([np.stack([a, b, c], 1), np.stack([b, d, c], 1)]).astype(np.int32)
    v, f = sg.merge([(v, f), sg.quad(2.0)])
    s = sg.config0()
    alb = sg.f32(np.random.default_rng(n).uniform(0.3, 0.9, (len(f), channels)))
    s.scenes = [sg.Scene(verts=v, faces=f, albedo=alb)]
    s.channels = channels
    s.lights[0].resolution, s.lights[0].k = 150, 3
    s.cameras[0].width, s.cameras[0].height = 141, 126
    return s


@pytest.mark.parametrize('n,channels', [(46, 1), (18, 3), (11, 1), (6, 3)])
def test_gradients(n, channels):
    b = _batch(n, channels)
    G = random_grad(b, n)
    check_gradients(b, G, oracle_run(b))
    G = [g.astype(np.float32) for g in G]
    ref, got = gpu_grads(b, [G], tile_size=16)[0], gpu_grads(b, [G])[0]
    for k in ('gverts', 'glight', 'galbedo'):
        normwise(k, got[k], ref[k], GRAD_TOL)
