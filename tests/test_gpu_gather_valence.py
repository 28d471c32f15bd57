"""The per-vertex gather at the corner counts where its handling changes (six
at a time, 24 by a lane, the rest by the wave) and at the pair counts of a
triangle where its rows are read in place, summed before, or in items: fans of
1 to 200 triangles, small and large, in one scene with several views."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import check_gradients, oracle_run, random_grad

pytestmark = pytest.mark.gpu


def _fan(n, centre, radius):
    """n triangles around one vertex (a closed disc from three on), slightly raised at the hub."""
    a = 2 * np.pi * np.arange(n + 1) / max(n, 3)
    rim = np.stack([centre[0] + radius * np.cos(a), np.full(n + 1, centre[1]), centre[2] - radius * np.sin(a)], 1)
    v = np.concatenate([[[centre[0], centre[1] + 0.1 * radius, centre[2]]], rim[:n] if n >= 3 else rim])
    last = (lambda i: 1 + (i + 1) % n) if n >= 3 else (lambda i: 2 + i)
    return v, np.array([[0, 1 + i, last(i)] for i in range(n)], np.int32)


# The light gradient is compared on the large fans: on the small ones (slivers
# under a sample wide) the terms it sums cancel, and float32 alone is 1.06e-4
# off the oracle whichever order the gather takes.
@pytest.mark.parametrize('radius,groups', [(0.06, ['gverts', 'galbedo']), (0.28, ['gverts', 'galbedo', 'glight'])])
def test_fans(radius, groups):
    counts = [1, 2, 5, 6, 7, 12, 13, 23, 24, 25, 26, 88, 89, 151, 152, 153, 200]
    parts = [_fan(n, (-1.2 + 0.6 * (i % 5), 0.5, -1.2 + 0.6 * (i // 5)), radius) for i, n in enumerate(counts)]
    v, f = sg.merge(parts + [sg.quad(2.0)])
    b = sg.config3(n_lat=6, sm_res=200, view_res=150, n_cams=3, n_lights=2)
    b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    for light in b.lights:
        light.k, light.sigma = 3, 1.0
    check_gradients(b, random_grad(b, 33), oracle_run(b), groups=groups)
