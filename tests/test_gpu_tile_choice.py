"""Which tiles a single pair takes, by frame, radius and levels: the number of tiles
that leave the fp16 refine (all of them, with descriptors outside its range) tells.
Outputs are those of the plain scan of global memory, whatever the tiles."""
import numpy as np
import pytest

import parity
import synth
from paper_2412_12392_amd import match, params, path_counters, set_launch

pytestmark = pytest.mark.gpu


# At 256 CUs.  Radii up to 4 take 8 x 8 tiles up to six a CU (two levels: three); wider windows up
# to one and a half, and where one 16 x 16 tile a CU is not enough.
@pytest.mark.parametrize("H,W,r,levels,side", [
    (216, 288, 4, 1, 8), (256, 384, 4, 1, 8), (256, 392, 4, 1, 16),
    (128, 192, 5, 1, 8), (128, 200, 5, 1, 16), (216, 288, 5, 1, 16), (216, 288, 6, 1, 16), (256, 256, 8, 1, 16),
    (256, 272, 6, 1, 8), (256, 384, 8, 1, 8), (256, 392, 6, 1, 16),
    (192, 256, 5, 2, 8), (128, 192, 6, 2, 8), (128, 200, 6, 2, 16), (192, 256, 6, 2, 16), (48, 64, 3, 3, 16)])
def test_tiles_of_a_pair(H, W, r, levels, side):
    print("tiles", H, W, r, levels, flush=True)
    t = parity.pair_tensors(synth.make_pair(H, W, H + W + r, conf=True))
    args = (t["Xii"], t["Xji"], t["Dii"] * 1e4, t["Dji"], t["Qii"], t["Qji"], None)
    prm = params(refine_radius=r, refine_levels=levels, max_theta=10.0)
    path_counters(reset=True)
    got = parity.result_numpy(match(*args, prm, want_xhat=True))
    counts = path_counters(reset=True)
    assert counts["refine_global"] == levels * -(-H // side) * -(-W // side), counts
    set_launch(tile_config=0)
    try:
        ref = parity.result_numpy(match(*args, prm, want_xhat=True))
    finally:
        set_launch()
    for k in ("p", "idx", "valid", "theta", "xhat"):
        assert np.array_equal(ref[k], got[k], equal_nan=True), k
