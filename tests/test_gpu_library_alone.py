"""A Plan and its raw calls need the library only: without the autograd nodes'
module they work, and render and pose say what is missing."""
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def test_raw_calls_without_the_nodes(monkeypatch):
    from paper_2308_10896_amd import _lib, dsm
    b = sg.config2(n_scenes=2, resolution=96, with_pose=True)
    local, lp, alb, poses = dsm.batch_inputs(b)
    want = dsm.render(dsm.Plan(b), local, lp, alb)
    monkeypatch.setattr(_lib, '_ext', None)
    monkeypatch.setattr(_lib, 'EXT_PATH', _lib.EXT_PATH + '.missing')
    plan = dsm.Plan(b)
    saved, scratch = plan.workspace()
    images = plan.forward(local, lp, alb, saved, scratch)
    assert torch.equal(images, want)
    gv, gl, ga = plan.backward(local, lp, alb, saved, scratch, torch.ones_like(images))
    assert all(torch.isfinite(t).all() for t in (gv, gl, ga, plan.pose_backward(local, poses, gv)))
    assert plan.stats(saved)['overflow'] == 0
    for call in (lambda: dsm.render(plan, local, lp, alb), lambda: dsm.pose(plan, local, poses)):
        with pytest.raises(RuntimeError, match='is missing'):
            call()
    monkeypatch.undo()
    assert torch.equal(dsm.render(plan, local, lp, alb), want)
