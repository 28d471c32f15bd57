"""A Plan that refers to its own results is freed, and the library's plan lives as
long as a graph that needs it."""
import gc
import weakref

import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('keep', ['images', 'world'])
def test_plan_that_keeps_its_results_is_freed(keep):
    from paper_2308_10896_amd import dsm
    b = sg.config2(n_scenes=1, resolution=64, with_pose=True)
    plan = dsm.Plan(b)
    local, lp, alb, poses = dsm.batch_inputs(b)
    world = dsm.pose(plan, local, poses.requires_grad_(True))
    plan.last = world if keep == 'world' else dsm.render(plan, world, lp, alb)
    ref = weakref.ref(plan)
    del plan, world
    gc.collect()
    assert ref() is None


def test_graph_keeps_the_library_plan():
    from paper_2308_10896_amd import dsm
    b = sg.config2(n_scenes=1, resolution=64, with_pose=True)
    plan = dsm.Plan(b)
    local, lp, alb, poses = dsm.batch_inputs(b)
    images = dsm.render(plan, dsm.pose(plan, local, poses.requires_grad_(True)), lp, alb)
    want, = torch.autograd.grad(images.sum(), poses, retain_graph=True)
    library, handle = weakref.ref(plan._library), weakref.ref(plan)
    del plan
    gc.collect()
    assert handle() is None and library() is not None
    got, = torch.autograd.grad(images.sum(), poses)
    assert torch.linalg.vector_norm(got - want) <= 1e-5 * torch.linalg.vector_norm(want)
    del images
    gc.collect()
    assert library() is None
