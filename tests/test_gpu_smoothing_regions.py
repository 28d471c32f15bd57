"""The smoothing kernels' 64 x 4 regions: views and maps that end inside a
region or hold less than one, several renders of one camera (the pairs are
evaluated once for all of them), cameras with different numbers of renders,
one and three channels.  Forward stages and gradients against the oracle at
the parity contract's tolerances."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import check_gradients, gpu_run, oracle_run, random_grad
from test_gpu_render import check_forward

pytestmark = pytest.mark.gpu


def _batch(w, h, res, channels=1):
    b = sg.config3(n_lat=14, sm_res=res, view_res=64, n_cams=2, n_lights=2)
    for cam in b.cameras:
        cam.width, cam.height = w, h
    for light in b.lights:
        light.k, light.sigma = 3, 1.0
    # three renders of the first camera, one of the second
    b.renders = [sg.Render(0, [0]), sg.Render(1, [1]), sg.Render(0, [1]), sg.Render(0, [0, 1])]
    if channels == 3:
        b.channels = 3
        sc = b.scenes[0]
        sc.albedo = sg.f32(np.random.default_rng(9).uniform(0.2, 0.9, (len(sc.faces), 3)))
    return b


@pytest.mark.parametrize('w,h,res,channels', [(1, 1, 3, 1), (63, 3, 65, 3), (65, 5, 64, 1), (64, 4, 127, 1)])
def test_forward_at_region_edges(w, h, res, channels):
    b = _batch(w, h, res, channels)
    check_forward(b, gpu_run(b), oracle_run(b))


@pytest.mark.parametrize('w,h,res,channels', [(129, 66, 131, 1), (96, 97, 128, 3)])
def test_gradients_at_region_edges(w, h, res, channels):
    b = _batch(w, h, res, channels)
    o = oracle_run(b)
    check_forward(b, gpu_run(b), o)
    check_gradients(b, random_grad(b, 21), o)
