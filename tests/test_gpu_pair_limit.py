"""More than 2^32 (triangle, tile) pairs, as an optimization that diverged can ask
for: triangles past the bins go through the overflow path as with fewer pairs.

17,500 slivers across a 4096^2 map, beyond the far plane, come after a small scene
in the face list, and its camera view comes after all of them: every result is
the scene's without the slivers."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def _batch(n_slivers):
    v, f = sg.merge([sg.quad(2.0), sg.cube((0.2, 1.0, 0.1), 0.4)])
    far = sg.f32([[-4.4, -60, -4.4], [4.4, -60, 4.4], [4.4, -60, 4.39]])
    k, n = len(v), len(f)
    v, f = np.concatenate([v, far]), np.concatenate([f, np.tile([[k, k + 1, k + 2]], (n_slivers, 1)).astype(f.dtype)])
    b = sg.config0()
    b.scenes = [sg.Scene(verts=v.astype(np.float32), faces=f, albedo=np.full((len(f), 1), 0.8, np.float32))]
    b.lights = [sg.Light('directional', sg.f32([0, -1, 0]), resolution=4096, k=1, up=sg.f32([0, 0, 1]))]
    b.cameras[0].width, b.cameras[0].height = 52, 44
    return b, k, n


def test_pairs_past_32_bits():
    from paper_2308_10896_amd import dsm
    out = []
    for n_slivers in (0, 17500):
        b, k, n = _batch(n_slivers)
        plan = dsm.Plan(b)
        verts, lp, alb, _ = dsm.batch_inputs(b)
        saved, scratch = plan.workspace()
        scratch.fill_(0x7f)                                  # rows that nothing clears would show (3.4e38)
        images = plan.forward(verts, lp, alb, saved, scratch)
        up = torch.randn(images.numel(), device='cuda', generator=torch.Generator('cuda').manual_seed(1))
        scratch.fill_(0x7f)
        gv, gl, ga = plan.backward(verts, lp, alb, saved, scratch, up)
        out.append((plan.view_keys(saved, 0), plan.view_keys(saved, 1), images, gv[:k], gl, ga[:n], plan.stats(saved)))
        if n_slivers:
            assert not gv[k:].any() and not ga[n:].any()
        torch.cuda.synchronize()
        print(n_slivers, out[-1][-1], flush=True)
    want, got = out
    assert got[6]['pairs'] > 2 ** 32 and got[6]['overflow'] > 17000 and got[6]['culled'] == want[6]['culled']
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(a, b)
    for a, b in zip(got[3:6], want[3:6]):
        assert torch.linalg.vector_norm(a - b) <= 1e-5 * torch.linalg.vector_norm(b)
