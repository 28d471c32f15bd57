"""The lookup's adjoint takes the lights of a render one after another and the
renders of a camera share its pixels' geometry: renders with 0, 1, 2 and 4
lights of one RGB camera, and the same gradients at every tile side."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import GRAD_TOL, check_gradients, gpu_grads, normwise, oracle_run, random_grad

pytestmark = pytest.mark.gpu


def _batch(channels):
    b = sg.config3(n_lat=12, sm_res=96, view_res=90, n_cams=1, n_lights=4)
    b.cameras[0].width = 101
    for light in b.lights:
        light.k, light.sigma = 3, 1.0
    b.renders = [sg.Render(0, [2]), sg.Render(0, []), sg.Render(0, [0, 3]), sg.Render(0, [3, 2, 1, 0])]
    b.channels = channels
    sc = b.scenes[0]
    sc.albedo = sg.f32(np.random.default_rng(4).uniform(0.2, 0.9, (len(sc.faces), channels)))
    return b


@pytest.mark.parametrize('channels', [1, 3])
def test_gradients_match_oracle(channels):
    b = _batch(channels)
    check_gradients(b, random_grad(b, 5), oracle_run(b))


@pytest.mark.parametrize('channels', [1, 3])
@pytest.mark.parametrize('tile,bins', [(16, 0), (32, 0), (8, 1), (16, 1)])
def test_gradients_independent_of_tiles_and_bins(tile, bins, channels):
    """The same sums over other tiles, or with overflowed triangles."""
    b = _batch(channels)
    G = [g.astype(np.float32) for g in random_grad(b, 6)]
    ref, got = gpu_grads(b, [G])[0], gpu_grads(b, [G], tile_size=tile, bin_scale=bins)[0]
    for k in ('gverts', 'glight', 'galbedo'):
        normwise(k, got[k], ref[k], GRAD_TOL)
