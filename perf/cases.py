"""Measured workloads of the renderer: what a user's program does with it, from
one tiny scene to a batch of 64, through the public entry points.

A render case draws the images of one plan and, in mode ``train``, pulls an
upstream image gradient back to every parameter (world vertices or poses,
lights, albedo) through autograd; mode ``graph`` replays the same pass as one
captured HIP graph; mode ``view`` only draws.  A filter case runs the
stand-alone moment filter or its transpose.

Meshes come from the seeded scene generator; a case's seed moves their
vertices, lights, poses and albedo a little and draws the upstream gradient,
so that every seed is a different input of the same sizes.
"""
import functools
import math

import numpy as np
import torch

import scenegen as sg
from paper_2308_10896_amd import dsm


def listed():
    return [
        # one 14-triangle scene, 256^2: the smallest call, all latency and launches
        dict(name='tiny cube 256', kind='tiny', mode='train', res=256, w=256, h=256, k=5),
        # one step of the minimal-plane pose experiment (occluder pose, view smaller than the map)
        dict(name='minimal plane pose', kind='plane', mode='train', res=256, w=128, h=128, k=9, tess=1),
        # one object under a spot light with a Gaussian filter, 512^2
        dict(name='icosphere spot 512', kind='spot', mode='train', res=512, w=512, h=512, k=7, subdiv=4),
        # an omnidirectional light (six faces filtered across their seams), exponential
        # maps with light-bleeding reduction, a view of odd size
        dict(name='cube light ragged', kind='cube', mode='train', res=256, w=250, h=190, k=5, warp=10.0, bleed=0.2),
        # a small batch of posed objects at sizes that are no multiple of anything
        dict(name='4 blobs ragged', kind='blobs', mode='train', n=4, res=200, w=250, h=190, k=5),
        # a mid-size batch of the pose-estimation loop
        dict(name='12 blobs 300', kind='blobs', mode='train', n=12, res=300, w=300, h=300, k=5),
        # the benchmark: 64 posed scenes at 512^2, one captured graph a step
        dict(name='64 blobs 512 graph', kind='blobs', mode='graph', n=64, res=512, w=512, h=512, k=5),
        # many cameras and lights around one dense object, a render for every pair
        dict(name='multi-view 8x16', kind='multi', mode='train', n_lat=158, res=1024, w=512, h=512, k=9, lights=8,
             cams=16),
        # one large RGB frame of a 330k-triangle scene, three 2048^2 lights summed
        dict(name='complex 1080p', kind='complex', mode='train', res=2048, w=1920, h=1080, k=11, objects=20,
             detail=1.0),
        # drawing without gradients: a target image or a preview at half that size
        dict(name='complex 540p view', kind='complex', mode='view', res=1024, w=960, h=540, k=11, objects=20,
             detail=0.5),
        # the moment filter by itself on a batch of maps
        dict(name='filter 64x512 box 5', kind='filter', mode='forward', n=64, res=512, k=5, gauss=False),
        # its transpose on large maps of a side that is no multiple of the tiles
        dict(name='filter^T 3x1000 gauss 11', kind='filter', mode='adjoint', n=3, res=1000, k=11, gauss=True),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(['tiny', 'plane', 'spot', 'cube', 'blobs', 'blobs', 'multi', 'complex', 'filter'])
    mode = rng.choice(['train', 'train', 'train', 'graph', 'view'])
    odd = [1, 3, 5, 7, 9, 11, 13, 15]
    if kind == 'filter':
        res, gauss = _log(rng, 64, 2048), rng.random() < 0.5
        n = _log(rng, 1, max(1, min(64, (1 << 24) // (res * res))))
        return dict(kind=kind, mode=rng.choice(['forward', 'adjoint']), n=n, res=res, k=rng.choice(odd), gauss=gauss)
    if kind == 'tiny':
        return dict(kind=kind, mode=mode, res=_log(rng, 64, 512), w=_log(rng, 64, 512), h=_log(rng, 64, 512),
                    k=rng.choice(odd))
    if kind == 'plane':
        return dict(kind=kind, mode=mode, res=_log(rng, 64, 512), w=_log(rng, 64, 256), h=_log(rng, 64, 256),
                    k=rng.choice(odd), tess=rng.choice([1, 2, 4, 8, 16]))
    if kind == 'spot':
        return dict(kind=kind, mode=mode, res=_log(rng, 128, 1024), w=_log(rng, 128, 1024), h=_log(rng, 128, 1024),
                    k=rng.choice(odd), subdiv=rng.choice([2, 3, 4, 5]))
    if kind == 'cube':
        return dict(kind=kind, mode=mode, res=_log(rng, 64, 512), w=_log(rng, 64, 512), h=_log(rng, 64, 512),
                    k=rng.choice([3, 5, 7, 9]), warp=rng.choice([0.0, 0.0, 10.0, 20.0]),
                    bleed=rng.choice([0.0, 0.2]))
    if kind == 'blobs':
        res = _log(rng, 128, 512)
        return dict(kind=kind, mode=mode, n=_log(rng, 1, 48), res=res, w=_log(rng, 128, 512), h=_log(rng, 128, 512),
                    k=rng.choice([3, 5, 7]))
    if kind == 'multi':
        return dict(kind=kind, mode=mode, n_lat=_log(rng, 20, 120), res=_log(rng, 256, 1024), w=_log(rng, 128, 512),
                    h=_log(rng, 128, 512), k=rng.choice([5, 9]), lights=rng.randint(1, 6), cams=rng.randint(1, 12))
    return dict(kind=kind, mode=mode, res=_log(rng, 256, 2048), w=_log(rng, 320, 1920), h=_log(rng, 240, 1080),
                k=rng.choice([5, 11]), objects=rng.randint(4, 16), detail=rng.choice([0.25, 0.5, 0.75]))


@functools.lru_cache(maxsize=1)
def _stream():
    """The stream that a program captures and replays its graphs on."""
    return torch.cuda.Stream()


@functools.lru_cache(maxsize=8)
def _scene_batch(shape):
    """The batch description of a case (its sizes as a sorted tuple)."""
    c = dict(shape)
    kind = c['kind']
    if kind == 'tiny':
        b = sg.config0()
    elif kind == 'plane':
        b = sg.minimal_plane(k=c['k'], resolution=c['res'], occluder_tess=c['tess'], offset=(0.06, 0.0, -0.04),
                             rotation=(0.0, 0.1, 0.0))
    elif kind == 'spot':
        b = sg.config1()
        rng = np.random.default_rng(1)
        sv, sf = sg.icosphere(c['subdiv'])
        sv = sv + rng.normal(0.0, 0.02, sv.shape) + np.array([0, 1.5, 0])
        v, f = sg.merge([(sv, sf), sg.quad(4.0)])
        b.scenes = [sg.Scene(verts=v, faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    elif kind == 'cube':
        b = sg.cube_light_scene(resolution=c['res'], k=c['k'])
        for light in b.lights:
            light.warp_exponent, light.bleed_reduction = c['warp'], c['bleed']
    elif kind == 'blobs':
        b = sg.config2(n_scenes=c['n'], resolution=c['res'])
    elif kind == 'multi':
        b = sg.config3(n_lat=c['n_lat'], n_cams=c['cams'], n_lights=c['lights'])
    else:
        b = sg.config4(n_objects=c['objects'], detail=c['detail'])
    for light in b.lights:
        light.resolution, light.k = c['res'], c['k']
        if light.filter == 'gaussian':
            light.sigma = 0.0                       # the width that follows from k
    for cam in b.cameras:
        cam.width, cam.height = c['w'], c['h']
    return b


def _shape(case):
    return tuple(sorted((k, v) for k, v in case.items() if k not in ('name', 'mode')))


def _posed(case):
    return case['kind'] in ('plane', 'blobs')


def prepare(case, seed):
    dev = torch.device('cuda')
    gen = torch.Generator(device=dev).manual_seed(seed)
    if case['kind'] == 'filter':
        n, s = case['n'], case['res']
        # depth moments: a smooth depth with steps, about a reference depth
        z = torch.rand(n, 1, s, s, device=dev, generator=gen) * 0.02 - 0.1
        z = z + 0.2 * (torch.rand(n, 1, s, s, device=dev, generator=gen) < 0.3)
        maps = torch.cat([z, z * z], 1)
        if case['mode'] == 'adjoint':
            maps = torch.randn(n, 2, s, s, device=dev, generator=gen) * 1e-3
        return dict(case=case, maps=maps.contiguous())

    batch = _scene_batch(_shape(case))
    local, lp, alb, poses = dsm.batch_inputs(batch, dev)

    def moved(t, sigma):
        return t + sigma * torch.randn(t.shape, device=dev, generator=gen)

    local, poses = moved(local, 2e-4), moved(poses, 0.01)
    # the faces of a cube light share one position
    lp = (lp + moved(torch.zeros(3, device=dev), 0.02)) if case['kind'] == 'cube' else moved(lp, 0.02)
    alb = 0.3 + 0.6 * torch.rand(alb.shape, device=dev, generator=gen)
    plan = dsm.Plan(batch)
    grad = 1e-3 * torch.randn(int(plan.info.image_floats), device=dev, generator=gen)
    st = dict(case=case, plan=plan, local=local, lp=lp, alb=alb, poses=poses, grad=grad)
    if case['mode'] == 'graph':
        saved, scratch = plan.workspace(dev)
        out = dict(images=torch.empty(int(plan.info.image_floats), device=dev), gverts=torch.empty_like(local),
                   glp=torch.empty_like(lp), galb=torch.empty_like(alb), gposes=torch.empty_like(poses))
        verts, stream = torch.empty_like(local), _stream()
        torch.cuda.synchronize()
        plan.graph_capture(stream, local, poses, verts, lp, alb, saved, scratch, out['images'], grad, out['gverts'],
                           out['glp'], out['galb'], out['gposes'])
        torch.cuda.synchronize()
        st.update(out=out, stream=stream, keep=(verts, saved, scratch))
    elif case['mode'] == 'train':
        leaves = [lp, alb, poses if _posed(case) else local]
        for t in leaves:
            t.requires_grad_(True)
    return st


def run(state):
    case = state['case']
    if case['kind'] == 'filter':
        return dsm.filter_moments(state['maps'], 'gaussian' if case['gauss'] else 'box', case['k'], 0.0,
                                  case['mode'] == 'adjoint')
    plan, local, lp, alb, poses = (state[k] for k in ('plan', 'local', 'lp', 'alb', 'poses'))
    if case['mode'] == 'graph':
        plan.graph_launch(state['stream'])
        return state['out']
    if case['mode'] == 'view':
        with torch.no_grad():
            verts = dsm.pose(plan, local, poses) if _posed(case) else local
            return dsm.render(plan, verts, lp, alb)
    if _posed(case):
        verts, leaves = dsm.pose(plan, local, poses), [lp, alb, poses]
    else:
        verts, leaves = local, [lp, alb, local]
    images = dsm.render(plan, verts, lp, alb)
    glp, galb, gleaf = torch.autograd.grad(images, leaves, state['grad'])
    return dict(images=images.detach(), glp=glp, galb=galb, gleaf=gleaf)


def work(case):
    if case['kind'] == 'filter':
        texels = 2.0 * case['n'] * case['res'] ** 2
        return dict(bytes=8.0 * texels, flops=4.0 * case['k'] * texels)
    b = _scene_batch(_shape(case))
    V = sum(len(s.verts) for s in b.scenes)
    F = sum(len(s.faces) for s in b.scenes)
    C = b.channels
    texels = float(sum(x.resolution ** 2 for x in b.lights))
    pix = float(sum(b.cameras[r.camera].width * b.cameras[r.camera].height for r in b.renders))
    lit = float(sum(b.cameras[r.camera].width * b.cameras[r.camera].height * len(r.lights) for r in b.renders))
    taps = 8.0 * case['k']                       # two channels, two directions, a multiply and an add
    # inputs in, images out; the moment maps between the passes (two floats a texel, written and read)
    nbytes = 12.0 * (V + F) + 4.0 * C * F + 4.0 * C * pix + 16.0 * texels
    flops = texels * (100.0 + taps) + pix * 120.0 + lit * 60.0 + 3.0 * 40.0 * F
    if case['mode'] != 'view':
        nbytes += 4.0 * C * pix + 12.0 * V + 4.0 * C * F + 16.0 * texels
        flops += texels * (150.0 + taps) + pix * 150.0 + lit * 150.0
    return dict(bytes=nbytes, flops=flops)


def exact(case, seed):
    """The moment filter in 64 bits.  The images have no such value: which
    triangle owns a sample is decided on a fixed-point grid."""
    if case['kind'] != 'filter':
        return None
    maps = prepare(case, seed)['maps'].double()
    n, _, s, _ = maps.shape
    k, r = case['k'], (case['k'] - 1) // 2
    if case['gauss'] and k > 1:
        sigma = (k - 1) / 3.0
        taps = torch.tensor([math.exp(-i * i / (2.0 * sigma * sigma)) for i in range(-r, r + 1)],
                            dtype=torch.float64, device=maps.device)
    else:
        taps = torch.ones(k, dtype=torch.float64, device=maps.device)
    taps = taps / taps.sum()
    at = torch.arange(s, device=maps.device)
    line = torch.zeros(s, s, dtype=torch.float64, device=maps.device)      # clamped one-dimensional filter
    for i in range(k):
        line.index_put_((at, (at + i - r).clamp(0, s - 1)), taps[i].expand(s), accumulate=True)
    if case['mode'] == 'adjoint':
        line = line.t().contiguous()
    flat = maps.reshape(2 * n, s, s)
    return torch.stack([line @ m @ line.t() for m in flat]).reshape(n, 2, s, s)
