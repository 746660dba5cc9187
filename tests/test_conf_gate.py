"""The confidence gate of the pose solves: decided as in fp64 for every q_min, in
fp32 but for a narrow band of products."""
import subprocess

import numpy as np
import pytest

import synth
from paper_2412_12392_amd import build

# Open gates, and thresholds at the ends of the ranges that get a band.
THRESHOLDS = [0.0, -1.0, -1e-30, 1e-30, 1e-18, 2e-18, 1e-12, 1.5, 1e12, 9e17, 2e18]


@pytest.fixture(scope="module")
def bands(tmp_path_factory):
    """(lo, hi) of the host's gate for every threshold."""
    d = tmp_path_factory.mktemp("gate")
    src = d / "gate.hip"
    src.write_text('#include <stdio.h>\n#include <stdlib.h>\n#include "m3s_sim3.h"\n'
                   "int main(int n, char** v) {\n"
                   "  for (int i = 1; i < n; ++i) {\n"
                   "    const m3s::ConfGate g = m3s::conf_gate(strtof(v[i], 0));\n"
                   '    printf("%.9g %.9g\\n", g.lo, g.hi);\n  }\n  return 0;\n}\n')
    exe = str(d / "gate")
    subprocess.run([build.hipcc(), *build.flags(), str(src), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe, *["%.9g" % q for q in THRESHOLDS]], check=True, capture_output=True, text=True).stdout
    return dict(zip(THRESHOLDS, [tuple(float(x) for x in line.split()) for line in out.splitlines()]))


@pytest.mark.parametrize("q_min", THRESHOLDS)
def test_band(bands, q_min):
    lo, hi = bands[q_min]
    # No product of usual confidences falls into the band of an open gate or of a small threshold.
    if q_min < 1.0:
        assert 0.0 <= lo <= hi <= 1e-20
    # Outside the band fp32 and fp64 agree: thresholds and products around it.
    q32 = np.float32(q_min)
    rng = np.random.Generator(np.random.PCG64(5))
    near = np.abs(np.float64(q32)) * (1 + np.concatenate([[0.0], rng.normal(0, 1e-5, 2000), rng.normal(0, 1e-7, 2000)]))
    a = np.concatenate([near, 10.0 ** rng.uniform(-44, 38, 4000), [0.0, -0.0, 1e-45, 5.0]]).astype(np.float32)
    b = np.concatenate([near[::-1], 10.0 ** rng.uniform(-44, 38, 4000), [3.0, 2.0, 1e-45, -1e-30]]).astype(np.float32)
    with np.errstate(over="ignore", under="ignore", invalid="ignore"):
        p = a * b
        exact = np.sqrt(a.astype(np.float64) * b.astype(np.float64)) > np.float64(q32)
        flushed = np.where(np.abs(p) < np.float32(1.17549435e-38), np.float32(0), p)
    for prod in (p, flushed):  # with and without subnormal products
        assert exact[prod > np.float32(hi)].all()
        assert not exact[prod < np.float32(lo)].any()


@pytest.mark.gpu
@pytest.mark.parametrize("q_min", THRESHOLDS)
def test_match_counts(q_min):
    """Counts of the two solves equal the oracle's, over confidences that are zero, negative,
    not numbers, or so small or large that their product leaves the fp32 range."""
    from test_gpu_backend import _run as run_backend
    from test_gpu_track import I34, _check, _run as run_track
    print("gate", q_min, flush=True)
    rng = np.random.Generator(np.random.PCG64(11))
    tp = synth.make_tracking(31, 45, 21, noise=1e-3)

    def confidences(shape):
        q = 10.0 ** rng.uniform(-24, 18, size=shape)
        kind = rng.uniform(size=shape)
        q = np.where(kind < 0.3, rng.uniform(0.5, 5.0, size=shape), q)
        q = np.where(kind > 0.9, 0.0, q)
        q = np.where((kind > 0.8) & (kind < 0.85), -q, q)
        return np.where((kind > 0.85) & (kind < 0.87), np.nan, q).astype(np.float32)

    tp.Qf, tp.Qk = confidences(tp.Qf.shape), confidences(tp.Qk.shape)
    T, info, _, ref = run_track(tp, I34, iters=0, q_min=q_min)
    assert int(info[1]) == ref["count"]
    bp = synth.make_backend(3, 24, 31, 22, noise=1e-3, loops=0)
    bp.Q = confidences(bp.Q.shape)
    T, info, _, ref = run_backend(bp, iters=0, q_min=q_min)
    assert int(info[1]) == ref["count"]
    # An open gate over usual confidences keeps every valid match, and the poses are the oracle's.
    if q_min <= 0:
        tp = synth.make_tracking(31, 45, 23, noise=1e-3)
        T, info, T_ref, ref = run_track(tp, I34, q_min=q_min)
        assert ref["count"] == int(tp.valid.sum())
        _check(T, info, T_ref, ref)
