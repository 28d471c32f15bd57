"""render and pose where a C++ autograd node would be passed by: a function
recorded by torch.jit.trace renders its own inputs (not the ones it was recorded
with, nor uninitialized memory) and is differentiable, and tensor subclasses
keep their class."""
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def _case(pose):
    from paper_2308_10896_amd import dsm
    b = sg.config2(n_scenes=2, resolution=96, with_pose=pose)
    plan = dsm.Plan(b)
    return (plan, *dsm.batch_inputs(b))


def _close(a, b):
    # the reverse pass adds with atomics: the same terms in another order
    assert torch.linalg.vector_norm(a - b) <= 1e-5 * torch.linalg.vector_norm(b)


def test_traced_render():
    from paper_2308_10896_amd import dsm
    plan, local, lp, alb, _ = _case(False)

    def f(verts, light, albedo):
        return dsm.render(plan, verts, light, albedo) * 2.0

    traced = torch.jit.trace(f, (local, lp, alb), check_trace=False)
    other = [(local * 1.01).requires_grad_(True), (lp + 0.05).requires_grad_(True), (alb * 0.5).requires_grad_(True)]
    want, got = f(*other), traced(*other)
    assert torch.equal(got, want) and not torch.equal(got, f(local, lp, alb))
    up = torch.randn_like(want)
    for a, b in zip(torch.autograd.grad(got, other, up), torch.autograd.grad(want, other, up)):
        _close(a, b)


def test_traced_pose():
    from paper_2308_10896_amd import dsm
    plan, local, _, _, poses = _case(True)
    traced = torch.jit.trace(lambda p: dsm.pose(plan, local, p), (poses,), check_trace=False)
    other = (poses + 0.1).requires_grad_(True)
    want, got = dsm.pose(plan, local, other), traced(other)
    assert torch.equal(got, want)
    up = torch.randn_like(want)
    _close(torch.autograd.grad(got, other, up)[0], torch.autograd.grad(want, other, up)[0])


def test_subclass_keeps_its_class():
    from paper_2308_10896_amd import dsm

    class Points(torch.Tensor):
        pass

    plan, local, lp, alb, poses = _case(True)
    world = dsm.pose(plan, local.as_subclass(Points), poses)
    assert type(world) is Points and torch.equal(world.as_subclass(torch.Tensor), dsm.pose(plan, local, poses))
    images = dsm.render(plan, world, lp, alb)
    assert torch.equal(images, dsm.render(plan, world.as_subclass(torch.Tensor), lp, alb))
    assert type(dsm.pose(plan, torch.nn.Parameter(local), poses)) is torch.Tensor
