"""The ways of the backend solve (in LDS, in the workspace, dense) on graphs that
need each of them at its larger sizes, against the fp64 oracle, with the way that
the library took read back from the workspace and compared with a model of its
elimination order and limits.  Tolerances are those of test_gpu_backend.py (the
solve itself is fp64 in every way)."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

LDS, WORKSPACE, DENSE = 0, 1, 2


def _full(N):
    return [(i, j) for j in range(N) for i in range(j)]


def _chain(N):
    return [(k - 1, k) for k in range(1, N)]


def _band(N, b):
    return [(i, j) for j in range(N) for i in range(max(0, j - b), j)]


def _random(N, extra, seed):
    more = np.random.Generator(np.random.PCG64(seed)).integers(0, N, size=(extra, 2)).tolist()
    return _chain(N) + [(a, b) for a, b in more if a != b]


def _both_ways(edges, total):
    """`total` edges: the given ones and their reverses in turn, over and over."""
    e = edges + [(j, i) for i, j in edges]
    return (e * (total // len(e) + 1))[:total]


GRAPHS = [
    # name, keyframes, edges, expected way
    # The lists of the edges of every block are made in chunks of 512 edges.
    ("edges_512", 12, _both_ways(_chain(12), 512), LDS),
    ("edges_513", 12, _both_ways(_chain(12), 513), LDS),
    ("edges_1037", 12, _both_ways(_band(12, 3), 1037), LDS),
    ("edges_1600", 40, _both_ways(_chain(40), 1600), LDS),
    # More edge entries than the workspace way keeps in LDS (8,192), ids above 9 bits.
    ("workspace_3049_edges", 128, _both_ways(_chain(128), 3049), WORKSPACE),
    ("workspace_band", 64, _band(64, 8), WORKSPACE),
    # Past LDS but faster dense.
    ("dense_by_cost", 26, _full(26), DENSE),
    # More than 8,192 products, on both sides of the panel's limit in LDS (65 keyframes) ...
    ("dense_65", 65, _full(65), DENSE),
    ("dense_66", 66, _full(66), DENSE),
    # ... with more than 512 columns left of a tile, and more than 2,048 blocks.
    ("dense_90", 90, _full(90), DENSE),
    ("dense_random_128", 128, _random(128, 300, 3), DENSE),
    ("dense_128", 128, _full(128), DENSE),
]


def expected_way(N, edges):
    """The library's order (level by level, each an independent set of keyframes of nearly the
    least degree), the blocks and products of the factor in it, and the rule over them."""
    nb = N - 1
    near = [set() for _ in range(nb)]
    for i, j in edges:
        if i != j and i > 0 and j > 0:
            near[i - 1].add(j - 1)
            near[j - 1].add(i - 1)
    left, place, column, levels = list(range(nb)), {}, [], 0
    while left:
        degree = {x: len(near[x]) for x in left}
        top = max(min(degree.values()) + 1, 2)
        key = {x: (degree[x], (rank + levels) & 1, x) for rank, x in enumerate(left)}
        candidates, level = {x for x in left if degree[x] <= top}, []
        while candidates:
            take = {x for x in candidates if all(key[x] < key[y] for y in near[x] & candidates)}
            for x in sorted(take):
                place[x] = len(column)
                column.append(set(near[x]))
                level.append(x)
            candidates = {x for x in candidates - take if not near[x] & take}
        left = [x for x in left if x not in place]
        for x in left:
            for v in level:
                if v in near[x]:
                    near[x] |= column[place[v]]
            near[x] -= set(level) | {x}
        levels += 1
    rows = [{p for p in range(nb) if x in column[p]} for x in range(nb)]
    order = sorted(place, key=place.get)
    blocks = products = 0
    for p, z in enumerate(order):
        for x in [z] + sorted(column[p]):
            blocks += 1
            products += len(rows[x] & rows[z])
    if blocks <= 320 and products <= 3072:
        return LDS
    tiles = -(-7 * nb // 32)
    slow = tiles <= 14 and 390 * levels + 9 * products > 294 * tiles * tiles + 210 * tiles + 1200
    return DENSE if blocks > 2048 or products > 8192 or slow else WORKSPACE


@pytest.mark.parametrize("name,N,edges,way", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_model_of_the_order(name, N, edges, way):
    assert expected_way(N, edges) == way


def _way_taken(ws, N, H, W, E):
    """The way recorded in the workspace: the third word after the poses, the edges' relative
    poses, systems and blocks, and the accumulation's rows."""
    def groups(matches):
        return min(1024, -(-H * W // (256 * matches)))

    rows = max(groups(8) * E, min(groups(4) * E, 3072))
    at = 0
    for nbytes in (96 * N, 48 * E, 320 * E, 448 * E, 128 * rows):
        at = (at + nbytes + 255) // 256 * 256
    return int(ws[at + 8:at + 12].view(-1).cpu().numpy().view(np.int32)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("name,N,edges,way", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_solve(name, N, edges, way):
    import torch

    from paper_2412_12392_amd import _lib, backend_params
    from test_gpu_backend import _check_poses
    print("solve", name, N, len(edges), flush=True)
    H, W, E, iters = 5, 7, len(edges), 3
    bp = synth.make_backend(N, H, W, 80 + N, noise=1e-3, loops=0, scramble=False)
    rng = np.random.Generator(np.random.PCG64(E))
    idx = np.tile(np.arange(H * W, dtype=np.int32).reshape(1, H, W), (E, 1, 1))
    valid = rng.uniform(size=(E, H, W)) < 0.95
    edges = np.array(edges, np.int32)
    T0 = np.asarray(bp.T_init, np.float32)
    Xc, Q, ed, ix, va = (torch.from_numpy(a).cuda() for a in (bp.Xc, bp.Q, edges, idx, valid.astype(np.uint8)))
    T, info = torch.tensor(T0).cuda(), torch.empty(4, device="cuda")
    lib = _lib.load()
    ws = torch.empty(lib.m3s_backend_workspace_bytes(N, H, W, E), dtype=torch.uint8, device="cuda")
    prob = _lib.BackendProblem(N, H, W, E, Xc.data_ptr(), Q.data_ptr(), ed.data_ptr(), ix.data_ptr(), va.data_ptr())
    args = dict(oracle.BACKEND_DEFAULTS, iters=iters)
    st = lib.m3s_backend_gn(ctypes.byref(prob), ctypes.byref(backend_params(**args)), T.data_ptr(), info.data_ptr(),
                            ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    _lib.check(lib, "m3s_backend_gn", st)
    torch.cuda.synchronize()
    assert _way_taken(ws, N, H, W, E) == way
    T_ref, ref = oracle.backend_gn(bp.Xc, bp.Q, edges, idx, valid, T0.astype(np.float64), **args)
    T, info = T.cpu().numpy(), info.cpu().numpy()
    assert np.array_equal(T[0], T0[0]), "keyframe 0 moved"
    _check_poses(T, T_ref)
    assert int(info[1]) == ref["count"] and int(info[2]) == ref["applied"] == iters
    assert abs(info[0] - ref["cost"]) <= 2e-3 * ref["cost"] + 1e-6 * max(ref["count"], 1)
