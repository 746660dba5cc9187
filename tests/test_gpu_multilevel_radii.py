"""The coarse-to-fine refine over every radius, alone and mixed in one batch: the
launch takes the kernel of the batch's radius, or the one for any.  Every output
bit against the plain scan of global memory (tile configuration 0)."""
import numpy as np
import pytest

import parity
import synth
from paper_2412_12392_amd import EdgeInput, match, match_batched, params, set_launch

pytestmark = pytest.mark.gpu

FIELDS = ("p", "idx", "valid", "theta", "xhat")


def _same(a, b, what):
    for k in FIELDS:
        assert np.array_equal(a[k], b[k], equal_nan=True), (what, k)


# Every kind of kernel: 2, 3 and 4 alone, other radii together, and mixtures of them, over regions
# that fit LDS (the small frame), are staged in bands, and take too many bands (the wide frame).
@pytest.mark.parametrize("levels", [2, 3, 4])
@pytest.mark.parametrize("radii", [(2, 2), (3, 3), (4, 4), (0, 1, 5, 8), (3, 5), (0, 2), (4, 3, 2), (6, 4)], ids=str)
@pytest.mark.parametrize("tile", [5, 6])
def test_radii_of_a_batch(radii, levels, tile):
    print("radii", radii, levels, tile, flush=True)
    shapes = [(30, 41), (70, 96), (17, 200), (37, 53)]
    pairs = [parity.pair_tensors(synth.make_pair(*shapes[k % 4], 500 + k, conf=True)) for k in range(len(radii))]
    args = [(t["Xii"], t["Xji"], t["Dii"], t["Dji"], t["Qii"], t["Qji"]) for t in pairs]
    prm = params(refine_levels=levels, max_theta=10.0)
    edges = [EdgeInput(*a, refine_radius=r) for a, r in zip(args, radii)]
    ref = []
    set_launch(tile_config=0)
    try:
        for a, r in zip(args, radii):
            ref.append(parity.result_numpy(match(*a, None, params(refine_radius=r, refine_levels=levels, max_theta=10.0),
                                                 want_xhat=True)))
        set_launch(tile_config=tile)
        for k, (a, r) in enumerate(zip(args, radii)):
            one = match(*a, None, params(refine_radius=r, refine_levels=levels, max_theta=10.0), want_xhat=True)
            _same(ref[k], parity.result_numpy(one), ("pair", k))
        # Captured and replayed, and then with the radii the other way round, which is another graph.
        for rep in range(2):
            for k, o in enumerate(match_batched(edges, prm, graph=True, want_xhat=True)):
                _same(ref[k], parity.result_numpy(o), ("batch", rep, k))
        turned = [EdgeInput(*a, refine_radius=r) for a, r in zip(args, radii[::-1])]
        for k, o in enumerate(match_batched(turned, prm, graph=True, want_xhat=True)):
            set_launch(tile_config=0)
            one = match(*args[k], None, params(refine_radius=radii[::-1][k], refine_levels=levels, max_theta=10.0),
                        want_xhat=True)
            _same(parity.result_numpy(one), parity.result_numpy(o), ("turned", k))
    finally:
        set_launch()
