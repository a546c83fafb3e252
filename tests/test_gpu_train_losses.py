"""The losses that hift_train returns are those of the steps taken one by one, whatever their number, and a step that is refused leaves those of the
steps before it."""
import ctypes

import numpy as np
import pytest

from hift_inputs import make_batch
from tests.hift_pair import make_pair, to_dev
from tests.test_gpu_step_fp32 import SMALL2

OPT = dict(kind="adamw", lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)


def _model(on_host):
    return make_pair(SMALL2, seed=5, opt=OPT, strategy="bottom2up", jitter=0.02, state_on_host=on_host)[1]


@pytest.mark.gpu
@pytest.mark.parametrize("on_host", [0, 1])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 131])
def test_losses_of_a_call_are_those_of_its_steps(on_host, n):
    dev = [to_dev(*make_batch(SMALL2, 5, t)) for t in range(1, 6)]
    a, b = _model(on_host), _model(on_host)
    got = a.train(dev, n)
    one = [b.step(*dev[i % 5], b.schedule_group_at(i + 1)) for i in range(n)]
    assert np.array_equal(got, np.array(one, dtype=np.float32))
    assert np.array_equal(a.read_params(), b.read_params())


@pytest.mark.gpu
def test_a_refused_step_leaves_the_losses_before_it():
    import paper_2401_15207_amd as H
    dev = [to_dev(*make_batch(SMALL2, 5, t)) for t in range(1, 4)]
    a, b = _model(0), _model(0)
    want = a.train(dev, 3)
    arr = (H.binding.Batch * 4)(*[H.binding.Batch(t.data_ptr(), l.data_ptr(), t.shape[0], t.shape[1]) for t, l in dev + dev[:1]])
    arr[3].batch = SMALL2["batch"] + 1
    losses = np.full(4, -1.0, dtype=np.float32)
    assert H.binding.lib.hift_train(b.h, arr, 4, 4, losses.ctypes.data_as(ctypes.c_void_p)) != 0
    assert np.array_equal(losses[:3], want) and losses[3] == -1.0
    assert b.cycle_index()[0] == 3
