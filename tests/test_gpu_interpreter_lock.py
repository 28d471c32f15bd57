"""render and pose leave the interpreter to other threads while they launch."""
import sys
import threading
import time

import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('name', ['render', 'pose'])
def test_other_threads_run_during_a_call(name):
    from paper_2308_10896_amd import dsm
    plan = dsm.Plan(sg.config2(n_scenes=2, resolution=96, with_pose=True))
    local, lp, alb, poses = dsm.batch_inputs(sg.config2(n_scenes=2, resolution=96, with_pose=True))
    run = (lambda: dsm.render(plan, local, lp, alb)) if name == 'render' else (lambda: dsm.pose(plan, local, poses))
    run()
    torch.cuda.synchronize()
    turns, stop = [0], threading.Event()

    def other():
        while not stop.is_set():
            turns[0] += 1
            time.sleep(0)               # gives the lock back at once

    t = threading.Thread(target=other)
    interval = sys.getswitchinterval()
    # no thread is made to give the lock up: another one runs only while it is given up by choice
    sys.setswitchinterval(1000.0)
    try:
        t.start()
        while turns[0] == 0:
            time.sleep(0.001)
        before = turns[0]
        for _ in range(200):
            run()
        ran = turns[0] - before
    finally:
        stop.set()
        t.join()
        sys.setswitchinterval(interval)
    torch.cuda.synchronize()
    assert ran > 0
