"""The pose solves over a match of infinite confidence: its whitened norms are
infinite, so the robust cost is +inf at every Huber width, and no step is applied
(the system is not finite)."""
import numpy as np
import pytest

import synth
from test_gpu_backend import _run as run_backend
from test_gpu_track import I34, _run as run_track

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("huber", [1.345, float("inf")])
def test_cost_is_infinite(huber):
    print("infinite confidence", huber, flush=True)
    tp = synth.make_tracking(24, 32, 31, noise=1e-3, valid_frac=1.0)
    tp.Qk[5, 7] = np.inf
    T, info, _, ref = run_track(tp, I34, huber=huber, iters=2)
    assert info[0] == np.inf and int(info[1]) == ref["count"] and int(info[2]) == 0
    assert np.array_equal(T, I34.astype(np.float32))
    bp = synth.make_backend(3, 24, 32, 32, noise=1e-3, loops=0)
    bp.Q[1] = np.where(np.arange(32) == 9, np.inf, bp.Q[1])
    T, info, _, ref = run_backend(bp, huber=huber, iters=2)
    assert info[0] == np.inf and int(info[1]) == ref["count"] and int(info[2]) == 0
    assert np.array_equal(T, np.asarray(bp.T_init, np.float32))
