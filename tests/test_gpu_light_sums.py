"""The light gradient's two ways to its sum: finished by the vertex gather's
last workgroup of each scene (up to 256 vertex workgroups), or by a launch of
its own; and the cut of its renders into 16 shares, for lights of no, one, five
and 20 renders."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import GRAD_TOL, check_gradients, gpu_grads, normwise, oracle_run, random_grad

pytestmark = pytest.mark.gpu


def _one():
    one = sg.config0()
    one.lights[0].resolution = 40
    one.cameras[0].width = one.cameras[0].height = 48
    return one


@pytest.mark.parametrize('n', [2, 256, 257])
def test_scenes_on_both_sides_of_the_rule(n):
    one = _one()
    many = sg.Batch('many', [], [], [], [], channels=1)
    for i in range(n):
        many.scenes.append(one.scenes[0])
        many.lights.append(sg.Light(**{**one.lights[0].__dict__, 'scene': i}))
        many.cameras.append(sg.Camera(**{**one.cameras[0].__dict__, 'scene': i}))
        many.renders.append(sg.Render(i, [i]))
    G = random_grad(one, 3)[0].astype(np.float32)
    ref = gpu_grads(one, [[G]])[0]
    check_gradients(one, [G], oracle_run(one))
    got = gpu_grads(many, [[G * np.float32(1 + i % 3) for i in range(n)]])[0]
    scale = (1 + np.arange(n) % 3).astype(np.float32)
    for k in ('glight', 'gverts'):
        r = np.asarray(ref[k], np.float32).reshape(1, -1)
        normwise(k, np.asarray(got[k]).reshape(n, -1), r * scale[:, None], GRAD_TOL)


def test_lights_of_many_and_of_no_renders():
    def batch(n_lights):
        b = sg.config3(n_lat=10, sm_res=72, view_res=56, n_cams=20, n_lights=4)
        b.lights = b.lights[:n_lights]
        for light in b.lights:
            light.k, light.sigma = 3, 1.0
        b.renders = ([sg.Render(c, [1]) for c in range(20)] + [sg.Render(c, [2]) for c in range(5)] +
                     [sg.Render(7, [0])])
        return b
    b = batch(3)
    G = random_grad(b, 8)
    check_gradients(b, G, oracle_run(b))
    G = [g.astype(np.float32) for g in G]
    used, more = gpu_grads(b, [G])[0], gpu_grads(batch(4), [G])[0]
    glight = np.asarray(more['glight']).reshape(4, 3)
    assert not glight[3].any()
    normwise('glight', glight[:3], np.asarray(used['glight']).reshape(3, 3), GRAD_TOL)
