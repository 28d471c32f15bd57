"""Posed vertices of scenes that no light or camera views: as many as the largest
scene has, not the largest viewed one."""
import numpy as np
import pytest
import torch

import scenegen as sg
from oracle import pipeline as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('viewed', [0, 1])
def test_scenes_without_views_are_posed(viewed):
    from paper_2308_10896_amd import dsm
    b = sg.config0()
    (sv, sf), rng = sg.icosphere(4), np.random.default_rng(2)
    other = sg.Scene(verts=np.asarray(sv, np.float32), faces=sf, albedo=np.full((len(sf), 1), 0.5, np.float32),
                     pose_count=len(sv) - 300, pose_center=sg.f32([0.1, 0.2, 0.3]),
                     pose=rng.normal(0, 0.3, 6).astype(np.float32))
    b.scenes.insert(1 - viewed, other)
    for x in b.lights + b.cameras:
        x.scene = viewed
    assert len(other.verts) > 4 * 256
    plan = dsm.Plan(b)
    local, _, _, poses = dsm.batch_inputs(b)
    torch.full((1 << 20,), float('nan'), device='cuda')            # what new tensors find in their memory
    world = dsm.pose(plan, local, poses)
    base, leaves, _, _ = P.scene_leaves(b)
    want = torch.cat(P.world_vertices(b, base, leaves)).detach().numpy()
    assert np.abs(world.cpu().numpy() - want).max() < 1e-6
