"""Binning of triangles with many tiles: cut into items that workgroups share,
at the sizes where the handling changes (32 tiles; one and several items), with
more pairs than the bins hold (the items may then be incomplete and the passes
walk the triangles), and with more workgroups than one scan of their totals
(many small views).  Keys bit-exact against the oracle."""
import numpy as np
import pytest

import scenegen as sg
from parity_helpers import check_gradients, gpu_run, loss_grad, oracle_run

pytestmark = pytest.mark.gpu


def _planes(res, w, h):
    """Stacked quads from a few tiles to the whole view, over a small cube."""
    parts = [sg.quad(half, 0.02 * k) for k, half in enumerate((2.0, 1.3, 0.7, 0.33, 0.2, 0.1))]
    v, f = sg.merge(parts + [sg.cube((0.3, 0.6, 0.1), 0.2)])
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    b.lights[0].resolution = res
    b.cameras[0].width, b.cameras[0].height = w, h
    return b


def _keys_equal(g, o):
    for v, (kg, ko) in enumerate(zip(g['keys'], o['keys'])):
        assert np.array_equal(kg, ko), f'view {v}: {int((kg != ko).sum())} keys differ'


@pytest.mark.parametrize('tile,bins', [(8, 0), (8, 1), (16, 0), (8, 2)])
def test_large_triangles(tile, bins):
    b = _planes(400, 333, 250)
    o = oracle_run(b)
    g = gpu_run(b, tile_size=tile, bin_scale=bins)
    _keys_equal(g, o)
    if bins == 0:
        assert g['stats']['overflow'] == 0
    if bins == 1:
        assert g['stats']['overflow'] > 0


def test_large_triangle_gradients():
    b = _planes(400, 333, 250)
    o = oracle_run(b)
    check_gradients(b, loss_grad(b, o['images']), o)


def test_more_workgroups_than_totals_summed_directly():
    """600 one-cube scenes: 1200 views, a triangle workgroup each."""
    one = sg.config0()
    one.lights[0].resolution = 24
    one.cameras[0].width = one.cameras[0].height = 24
    many = sg.Batch('many', [], [], [], [], channels=1)
    for i in range(600):
        many.scenes.append(one.scenes[0])
        many.lights.append(sg.Light(**{**one.lights[0].__dict__, 'scene': i}))
        many.cameras.append(sg.Camera(**{**one.cameras[0].__dict__, 'scene': i}))
        many.renders.append(sg.Render(i, [i]))
    a, m = gpu_run(one), gpu_run(many)
    for i in range(600):
        assert np.array_equal(m['keys'][i], a['keys'][0]) and np.array_equal(m['keys'][600 + i], a['keys'][1])
        assert np.array_equal(m['images'][i], a['images'][0])
    assert m['stats']['pairs'] == 600 * a['stats']['pairs']


@pytest.mark.parametrize('w,h,res', [(512, 512, 504), (520, 512, 513), (1024, 8, 1)])
def test_tiles_of_a_workgroup_around_the_table(w, h, res):
    """Triangles in no order, so that the tiles of every 256 of them span the
    view: 64 x 64 tiles (as many as the count pass has counters for), one
    column more, and a strip; then the same in two scenes, so that a view's
    tiles start away from zero."""
    rng = np.random.default_rng([9, w])
    n = 900
    c = np.stack([rng.uniform(-2.5, 2.5, n), rng.uniform(0.0, 0.6, n), rng.uniform(-2.5, 2.5, n)], 1)
    size = np.where(rng.random(n) < 0.1, 0.4, 0.06)
    v = (c[:, None, :] + size[:, None, None] * rng.uniform(-0.5, 0.5, (n, 3, 3))).reshape(-1, 3)
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v, faces=np.arange(3 * n, dtype=np.int32).reshape(n, 3),
                         albedo=np.full((n, 1), 0.8, np.float32))]
    b.lights[0].resolution, b.lights[0].k = res, 1
    b.cameras[0].width, b.cameras[0].height = w, h
    o = oracle_run(b)
    _keys_equal(gpu_run(b), o)
    two = sg.Batch('two', b.scenes * 2, [], [], [], channels=1)
    for i in range(2):
        two.lights.append(sg.Light(**{**b.lights[0].__dict__, 'scene': i}))
        two.cameras.append(sg.Camera(**{**b.cameras[0].__dict__, 'scene': i}))
        two.renders.append(sg.Render(i, [i]))
    g = gpu_run(two)
    for i in range(2):
        for k, kg in enumerate((g['keys'][i], g['keys'][2 + i])):
            assert np.array_equal(kg, o['keys'][k]), f'scene {i} view {k}'


@pytest.mark.parametrize('n', [1100, 33000])
def test_totals_by_groups_and_scanned(n):
    """n lights and n cameras of one small view each, a triangle workgroup
    each: their totals summed by groups, and scanned past 65,536 of them.  The
    quads' tiles in every view follow from the totals before it."""
    import torch
    from paper_2308_10896_amd import dsm
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))
                for v, f in [sg.merge([sg.quad(2.0), sg.cube((0.1, 0.5, 0.0), 0.5)])]]
    b.lights[0].resolution, b.lights[0].k = 5, 1
    b.cameras[0].width = b.cameras[0].height = 6
    ref = gpu_run(b)
    lights, cams = [b.lights[0]] * n, [b.cameras[0]] * n
    many = sg.Batch('many', b.scenes, lights, cams, [sg.Render(i, [i]) for i in range(n)], channels=1)
    plan = dsm.Plan(many)
    verts, lp, alb, _ = dsm.batch_inputs(many)
    saved, scratch = plan.workspace()
    images = plan.forward(verts, lp, alb, saved, scratch)
    flat = images.reshape(n, -1).cpu().numpy()
    assert np.array_equal(flat, np.broadcast_to(ref['images'][0].reshape(1, -1), flat.shape))
    for v in (0, 1, 63, 64, n - 1, n, n + 65, 2 * n - 1):
        k = plan.view_keys(saved, v).cpu().numpy().view(np.uint64)
        assert np.array_equal(k, ref['keys'][0 if v < n else 1]), f'view {v}'
    assert plan.stats(saved)['pairs'] == n * ref['stats']['pairs']
