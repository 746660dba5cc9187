"""Edges of the match statistics and of the tracking step's vector loads.

The statistics are whole numbers and exact.  The tracking tolerances and their
derivation are those of test_gpu_track.py."""
import numpy as np
import pytest
import torch

import synth
from paper_2412_12392_amd import MatchResult, match_stats
from test_gpu_track import I34, _check, _run

pytestmark = pytest.mark.gpu


# One pixel pair up to several workgroups (2,048 queries each), a span of matches wider than the
# 8,192 words of LDS (262,144 pixels), and images without a match.
@pytest.mark.parametrize("H,W,kind", [(2, 2, "shift"), (31, 33, "shift"), (64, 64, "shift"), (384, 512, "shift"),
                                      (520, 512, "scatter"), (600, 700, "scatter"), (45, 64, "none"), (48, 64, "one"),
                                      (48, 64, "wild")])
def test_stats_exact(H, W, kind):
    print("stats", H, W, kind, flush=True)
    n = H * W
    rng = np.random.Generator(np.random.PCG64(n))
    idx = {"shift": (np.arange(n) + 5) % n, "scatter": rng.integers(0, n, n), "none": np.arange(n),
           "one": np.full(n, n - 1), "wild": rng.integers(-n, 2 * n, n)}[kind].astype(np.int32)
    valid = np.zeros(n, bool) if kind == "none" else rng.uniform(size=n) < 0.7
    use = valid & (idx >= 0) & (idx < n)
    res = MatchResult(None, torch.from_numpy(idx.reshape(H, W)).cuda(),
                      torch.from_numpy(valid.astype(np.uint8).reshape(H, W)).cuda(), None, None)
    counts = match_stats(res).cpu().tolist()
    assert counts == [int(use.sum()), len(np.unique(idx[use]))]


# Pixel counts that leave 0, 1 and 3 over a lane's 4 matches, on both sides of the change from 1
# match a lane to 4 (131,072 pixels) and beyond what one pass of the grid covers (2,097,152).
@pytest.mark.parametrize("H,W", [(2, 2), (3, 3), (29, 53), (256, 512), (257, 511), (1449, 1449)])
def test_track_pixel_counts(H, W):
    print("track", H, W, flush=True)
    tp = synth.make_tracking(H, W, H + W, noise=1e-3, outlier_frac=0.05 if H > 3 else 0.0, valid_frac=0.9 if H > 3 else 1.0)
    T, info, T_ref, ref = _run(tp, I34, iters=4 if H > 3 else 0)
    _check(T, info, T_ref, ref)
