"""The pose solves in a view of one degree, where the rays of all matches nearly
coincide and the roll's curvature, sum w (1 - u_z^2), is 5e-5 of sum w.

Tolerance (derived before the first run): from a pose that is off by a roll of
0.5 rad, one Gauss-Newton step turns by about sin 0.5 = 0.48 rad.  Its relative
error is that of the roll's gradient and curvature: every term is rounded a few
times (each 2^-24 of the term, since neither is a difference of larger ones)
and summed over at most 1,024 matches in fp32, pairwise but for a lane's own 4
to 8: together below 25 * 2^-24 = 1.5e-6, or 7e-7 rad; rounding the pose to fp32
adds 1e-7.  The test allows 2e-6 rad.  Sums whose terms cancel leave 1e-5 to
1e-4 rad here.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_12392_amd import backend_gn, backend_params, track_params, track_pose

pytestmark = pytest.mark.gpu

ROLL_TOL = 2e-6
I34 = np.concatenate([np.eye(3), np.zeros((3, 1))], 1)


def _scene(H, W, seed, degrees=1.0):
    """Points of one surface seen through a narrow lens, fp32, with confidences."""
    rng = np.random.Generator(np.random.PCG64(seed))
    t = np.tan(np.radians(degrees) / 2)
    x, y = np.meshgrid((np.arange(W) - (W - 1) / 2) * 2 / W, (np.arange(H) - (H - 1) / 2) * 2 / W)
    z = 2.0 + 0.3 * np.sin(3 * x) * np.cos(2 * y) + 0.1 * x
    X = np.stack([z * x * t, z * y * t, z], -1).astype(np.float32)
    Q = rng.uniform(2.0, 5.0, size=(2, H, W)).astype(np.float32)
    return X, Q, rng.uniform(size=(H, W)) < 0.9


def _rolled(X, angle):
    c, s = np.cos(angle), np.sin(angle)
    R = np.array([[c, -s, 0], [s, c, 0], [0, 0, 1.0]])
    return (X.reshape(-1, 3).astype(np.float64) @ R.T).reshape(X.shape).astype(np.float32)


def _roll_between(Ta, Tb):
    """The roll of Ta's rotation after Tb's is taken off."""
    def rot(T):
        A = np.asarray(T, np.float64)[:, :3]
        return A / np.cbrt(np.linalg.det(A))
    D = rot(Ta) @ rot(Tb).T
    return abs(np.arctan2(D[1, 0] - D[0, 1], D[0, 0] + D[1, 1]))


# On both sides of the change of launch shape (131,072 matches).
@pytest.mark.parametrize("H,W", [(240, 320), (384, 512)])
def test_track_roll(H, W):
    print("narrow track", H, W, flush=True)
    Xf, Q, valid = _scene(H, W, H)
    Xk = _rolled(Xf, 0.5)
    idx = np.arange(H * W, dtype=np.int32).reshape(H, W)
    prm = dict(oracle.TRACK_DEFAULTS, iters=1, huber=float("inf"))
    dev = [torch.from_numpy(a).cuda() for a in (Xk, Xf, idx, valid.astype(np.uint8), Q[0], Q[1])]
    T = torch.tensor(I34, dtype=torch.float32, device="cuda").contiguous()
    track_pose(*dev, T, track_params(**prm))
    T_ref, ref = oracle.track_pose(Xk, Xf, idx, valid, Q[0], Q[1], I34, **prm)
    assert ref["solved"] == 1
    assert _roll_between(T_ref, I34) > 0.4
    assert _roll_between(T.cpu().numpy(), T_ref) <= ROLL_TOL


@pytest.mark.parametrize("H,W", [(240, 320), (384, 512)])
def test_backend_roll(H, W):
    print("narrow backend", H, W, flush=True)
    X, Q, valid = _scene(H, W, 7 + H)
    Xc = np.stack([_rolled(X, 0.5), X])
    edges = np.array([[0, 1], [1, 0]], np.int32)
    idx = np.tile(np.arange(H * W, dtype=np.int32).reshape(1, H, W), (2, 1, 1))
    v = np.stack([valid, valid[::-1]])
    T0 = np.stack([I34, I34])
    prm = dict(oracle.BACKEND_DEFAULTS, iters=1, huber=float("inf"))
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (Xc, Q, edges, idx, v.astype(np.uint8))]
    T = torch.tensor(T0, dtype=torch.float32, device="cuda").contiguous()
    backend_gn(*dev, T, backend_params(**prm))
    T_ref, ref = oracle.backend_gn(Xc, Q, edges, idx, v, T0, **prm)
    assert ref["applied"] == 1
    assert _roll_between(T_ref[1], I34) > 0.4
    assert _roll_between(T[1].cpu().numpy(), T_ref[1]) <= ROLL_TOL
