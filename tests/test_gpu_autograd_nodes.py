"""The autograd nodes of render and pose: the raw calls' results, gradients only
where asked, upstream gradients of any strides, errors of the same classes as
the raw calls, a graph that outlives its plan's name, two threads."""
import gc
import threading

import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def _case(n=2, pose=True):
    from paper_2308_10896_amd import dsm
    b = sg.config2(n_scenes=n, resolution=96, with_pose=pose)
    plan = dsm.Plan(b)
    return (plan, *dsm.batch_inputs(b))


def _raw(plan, local, lp, alb, poses, g):
    world = plan.pose_forward(local, poses)
    saved, scratch = plan.workspace()
    images = plan.forward(world, lp, alb, saved, scratch)
    gv, gl, ga = plan.backward(world, lp, alb, saved, scratch, g)
    return images, gl, ga, plan.pose_backward(local, poses, gv)


def _close(a, b):
    # the reverse pass adds with atomics: the same terms in another order
    assert torch.linalg.vector_norm(a - b) <= 1e-5 * torch.linalg.vector_norm(b)


def test_same_as_raw_calls_and_strided_upstream():
    from paper_2308_10896_amd import dsm
    plan, local, lp, alb, poses = _case()
    lp, alb, poses = (t.requires_grad_(True) for t in (lp, alb, poses))
    images = dsm.render(plan, dsm.pose(plan, local, poses), lp, alb)
    wide = torch.randn(2 * images.numel(), device='cuda')[::2]          # every other element
    assert not wide.is_contiguous()
    with torch.no_grad():
        want = _raw(plan, local, lp, alb, poses, wide.contiguous())
    assert torch.equal(images, want[0])
    for got, w in zip(torch.autograd.grad(images, [lp, alb, poses], wide), want[1:]):
        _close(got, w)


def test_only_wanted_gradients():
    from paper_2308_10896_amd import dsm
    plan, local, lp, alb, poses = _case(pose=False)
    assert not dsm.render(plan, local, lp, alb).requires_grad
    lp.requires_grad_(True)
    images = dsm.render(plan, local, lp, alb)
    images.sum().backward()
    assert lp.grad is not None and alb.grad is None and local.grad is None


def test_errors():
    from paper_2308_10896_amd import _lib, dsm
    plan, local, lp, alb, poses = _case()
    with pytest.raises(ValueError, match='lp|light_params'):
        dsm.render(plan, local, lp.double(), alb)
    with pytest.raises(ValueError, match='albedo'):
        dsm.render(plan, local, lp, alb.repeat(1, 2)[:, ::2])
    with pytest.raises(ValueError, match='poses'):
        dsm.pose(plan, local, poses.cpu())
    with pytest.raises(_lib.DSMError) as e:
        _lib.ext().render(plan._nodes, local, lp, alb, torch.empty(256, dtype=torch.uint8, device='cuda'))
    assert e.value.status == 3                      # workspace too small
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda p: dsm.pose(plan, local, p))(poses[None])


def test_graph_outlives_plan_name():
    from paper_2308_10896_amd import dsm
    plan, local, lp, alb, poses = _case()
    poses.requires_grad_(True)
    images = dsm.render(plan, dsm.pose(plan, local, poses), lp, alb)
    del plan
    gc.collect()
    images.sum().backward()
    assert torch.isfinite(poses.grad).all()


def test_threads_with_their_own_plans_and_streams():
    from paper_2308_10896_amd import dsm
    cases = [_case(n=k + 1) for k in range(2)]
    want = []
    for plan, local, lp, alb, poses in cases:
        g = torch.ones(int(plan.info.image_floats), device='cuda')
        want.append(_raw(plan, local, lp, alb, poses, g))
    torch.cuda.synchronize()
    got, errors = [None, None], []

    def work(k):
        try:
            plan, local, lp, alb, poses = cases[k]
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(5):
                    q = poses.clone().requires_grad_(True)
                    im = dsm.render(plan, dsm.pose(plan, local, q), lp, alb)
                    im.sum().backward()
                torch.cuda.current_stream().synchronize()
                got[k] = (im.detach(), q.grad)
        except Exception as e:      # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errors, errors
    for k in range(2):
        assert torch.equal(got[k][0], want[k][0])
        _close(got[k][1], want[k][3])
