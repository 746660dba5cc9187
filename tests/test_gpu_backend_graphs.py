"""GPU parity of the backend solve over graph shapes that take each of its ways
through the factor: in LDS, in the workspace, and dense, with the limits between
them on either side.  Tolerances and their derivation are those of
test_gpu_backend.py (the solve itself is fp64 in every way)."""
import numpy as np
import pytest
import torch  # noqa: F401

import synth
from test_gpu_backend import _check_poses, _run

pytestmark = pytest.mark.gpu


def _full(N):
    return [(i, j) for j in range(N) for i in range(j)]


def _chain(N):
    return [(k - 1, k) for k in range(1, N)]


def _random(N, extra, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    more = rng.integers(0, N, size=(extra, 2)).tolist()
    return _chain(N) + [(a, b) for a, b in more if a != b]


GRAPHS = [
    # name, keyframes, edges
    ("one_free_keyframe", 2, [(0, 1), (1, 0)]),
    # No edge between free keyframes: one level, no products.
    ("star_on_the_gauge", 20, [(0, k) for k in range(1, 20)]),
    ("star_on_a_free_keyframe", 30, [(0, 1)] + [(1, k) for k in range(2, 30)]),
    ("two_chains", 33, _chain(17) + [(0, 17)] + [(k - 1, k) for k in range(18, 33)]),
    # Complete graphs: 300 blocks (LDS holds 320), 325 (workspace), 741 blocks with 9,139
    # products (8,192 at most: dense).
    ("complete_25", 25, _full(25)),
    ("complete_26", 26, _full(26)),
    ("complete_39", 39, _full(39)),
    ("random_100", 100, _random(100, 40, 3)),
    ("chain_128", 128, _chain(128)),
    # More edges per block than are read at once, more in all than LDS lists.
    ("repeated_edges", 30, (_chain(30) + [(j, i) for i, j in _chain(30)]) * 7),
]


@pytest.mark.parametrize("name,N,edges", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_backend_graph(name, N, edges):
    print("backend graph", name, N, len(edges), flush=True)
    H, W, E = 6, 8, len(edges)
    # Every keyframe sees every world point at the same pixel, so any pair is an edge.
    bp = synth.make_backend(N, H, W, 40 + N, noise=1e-3, loops=0, scramble=False)
    rng = np.random.Generator(np.random.PCG64(N))
    idx = np.tile(np.arange(H * W, dtype=np.int32).reshape(1, H, W), (E, 1, 1))
    valid = rng.uniform(size=(E, H, W)) < 0.95
    T, info, T_ref, ref = _run(bp, edges=np.array(edges, np.int32), idx=idx, valid=valid, iters=4)
    assert np.array_equal(T[0], np.asarray(bp.T_init[0], np.float32)), "keyframe 0 moved"
    _check_poses(T, T_ref)
    assert int(info[1]) == ref["count"] and int(info[2]) == ref["applied"] == 4
    assert abs(info[0] - ref["cost"]) <= 2e-3 * ref["cost"] + 1e-6 * max(ref["count"], 1)
