"""The refine where windows reach beyond the image: the unrolled scan slides
them inside.  Frames around the least size that allows it (2 r 2^l + 2^l) and
initial pixels in the corners, every output bit against the plain scan of global
memory (tile configuration 0), which has no windows to slide."""
import numpy as np
import pytest
import torch

import parity
import synth
from paper_2412_12392_amd import match, match_batched, params, set_launch, EdgeInput

pytestmark = pytest.mark.gpu

# H, W, r, levels
CASES = [(H, W, r, 1) for r in (2, 3, 4) for H, W in ((2 * r, 2 * r + 9), (2 * r + 1, 2 * r + 1), (2 * r + 2, 40), (33, 2 * r))]
CASES += [(13, 14, 3, 2), (14, 14, 3, 2), (14, 31, 3, 2), (40, 15, 3, 2), (27, 28, 3, 3), (37, 53, 2, 2), (37, 53, 5, 1)]
# Coarse levels whose regions are staged in bands of rows, and radii whose mask takes two words.
CASES += [(45, 60, 4, 2), (45, 60, 4, 3), (31, 36, 4, 3), (60, 90, 3, 3), (60, 90, 2, 4), (70, 96, 3, 4), (35, 120, 4, 4)]


@pytest.mark.parametrize("H,W,r,levels", CASES)
@pytest.mark.parametrize("tile", [5, 6])
def test_refine_windows_beyond_the_image(H, W, r, levels, tile):
    print("refine border", H, W, r, levels, tile, flush=True)
    t = parity.pair_tensors(synth.make_pair(H, W, 900 + H * W + r, conf=True))
    rng = np.random.Generator(np.random.PCG64(H * W))
    # Every query starts, and with K = 0 stays, at a pixel of the border or anywhere.
    corner = rng.integers(0, 2, size=(H, W, 2)) * np.array([W - 1.0, H - 1.0])
    some = rng.uniform(0, 1, size=(H, W, 2)) * np.array([W - 1.0, H - 1.0])
    p0 = torch.from_numpy(np.where(rng.uniform(size=(H, W, 1)) < 0.5, corner, some).astype(np.float32)).cuda()
    args = (t["Xii"], t["Xji"], t["Dii"], t["Dji"], t["Qii"], t["Qji"])
    for init, K in ((p0, 0), (None, 10)):
        prm = params(max_iter=K, refine_radius=r, refine_levels=levels, max_theta=10.0)
        got = []
        for cfg in (0, tile):
            set_launch(tile_config=cfg)
            try:
                res = match(*args, init, prm, want_xhat=True)
                out = match_batched([EdgeInput(*args, init)], prm, graph=False, want_xhat=True)[0]
                got += [parity.result_numpy(res), parity.result_numpy(out)]
            finally:
                set_launch()
        for g in got[1:]:
            for k in ("p", "idx", "valid", "theta", "xhat"):
                assert np.array_equal(got[0][k], g[k], equal_nan=True), (k, K)


@pytest.mark.parametrize("H,W,r,levels", [(256, 384, 3, 1), (256, 392, 4, 1), (8, 12288, 2, 1), (192, 256, 4, 2),
                                          (192, 264, 3, 2), (8, 9, 3, 2), (96, 128, 3, 3)])
def test_small_frame_tiles(H, W, r, levels):
    """The library's own choice of tiles, at the sizes where it changes (256
    CUs: 1,536 and 768 tiles of 8 x 8), against the scan of global memory."""
    print("small frame", H, W, r, levels, flush=True)
    t = parity.pair_tensors(synth.make_pair(H, W, 70 + H + W, conf=True))
    args = (t["Xii"], t["Xji"], t["Dii"], t["Dji"], t["Qii"], t["Qji"], None)
    prm = params(refine_radius=r, refine_levels=levels, max_theta=10.0)
    got = parity.result_numpy(match(*args, prm, want_xhat=True))
    set_launch(tile_config=0)
    try:
        ref = parity.result_numpy(match(*args, prm, want_xhat=True))
    finally:
        set_launch()
    for k in ("p", "idx", "valid", "theta", "xhat"):
        assert np.array_equal(ref[k], got[k], equal_nan=True), k
