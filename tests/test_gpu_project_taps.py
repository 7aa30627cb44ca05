"""GPU: the staged projector at every tap count and weighting that reaches it.

Each case names the kernel it takes (turned images M, taps T, the three-tap shortcut), which
tests/test_project_routes_cpu.py holds it to, so that a change of the dispatch rule cannot
leave a form untested.  Sides odd and even, half detectors of 16 n - 1, 16 n and 16 n + 1
bins, lists whose windows hold eight and four angles, angle-gap weights.  Reference and
tolerance: the oracle's adjoint in FP64 and those of the projector's parity test (16 FP32
ulps of the largest pixel for each of the N (2 sqrt(2) dt + 1) terms of a bin).
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu

STAGED, LANE = "project_staged_kernel", "project_kernel"

# K, D, N, dt, list, weighting, kernel, its first template values: (M, T, FAST3), or (T, FAST3) of the one-lane kernel
CASES = [
    (720, 189, 112, 1.0, "uniform", "uniform", STAGED, [4, 3, 1]),      # the smallest staged image; half detector of 95 bins
    (720, 252, 131, 0.75, "uniform", "uniform", STAGED, [4, 3, 0]),     # 126
    (720, 255, 113, 0.75, "quarter", "uniform", STAGED, [4, 3, 0]),     # 128
    (1441, 257, 136, 0.75, "uniform", "uniform", STAGED, [2, 3, 0]),    # 129; the smallest of other lists, three taps
    (1601, 256, 141, 0.8, "golden", "uniform", STAGED, [2, 3, 0]),
    (720, 320, 130, 0.6, "uniform", "uniform", STAGED, [4, 2, 0]),
    (720, 513, 120, 0.4, "uniform", "uniform", STAGED, [4, 2, 0]),      # 257
    (1501, 321, 129, 0.6, "golden", "uniform", STAGED, [2, 2, 0]),
    (1501, 321, 112, 0.6, "golden", "uniform", STAGED, [2, 2, 0]),
    (720, 460, 400, 1.25, "uniform", "uniform", STAGED, [4, 4, 0]),     # four angles to a window
    (1601, 191, 137, 1.0, "golden", "angle-gaps", STAGED, [2, 3, 1]),
    (1600, 191, 130, 1.0, "uniform", "angle-gaps", STAGED, [4, 3, 1]),
    (1701, 250, 139, 0.75, "golden", "angle-gaps", STAGED, [2, 3, 0]),
    (720, 513, 150, 0.35, "uniform", "uniform", LANE, [1, 0]),          # one tap
    (1401, 509, 150, 0.34, "golden", "uniform", LANE, [1, 0]),          # other lists: two or three taps
    (1601, 150, 150, 1.25, "golden", "uniform", LANE, [4, 0]),
    (1601, 191, 135, 1.0, "golden", "uniform", LANE, [3, 1]),           # below the smallest staged images
    (720, 159, 111, 1.0, "uniform", "uniform", LANE, [3, 1]),
    (64, 183, 150, 1.0, "golden", "uniform", LANE, [3, 1]),             # too few angles to a window
    (100, 300, 300, 1.0, "uniform", "uniform", LANE, [3, 1]),
]


def angles(K, kind):
    if kind == "uniform":
        return ph.uniform_angles(K)
    if kind == "golden":
        return np.mod(np.arange(K) * math.pi * (math.sqrt(5.0) - 1.0) / 2.0, math.pi)
    h = np.sort(ph.rng_for(1950, K).uniform(-math.pi, math.pi, K // 2))
    return np.concatenate([h, h + 0.5 * math.pi])


@pytest.mark.parametrize("K,D,N,dt,kind,weighting", [c[:6] for c in CASES])
def test_projector_matches_oracle(K, D, N, dt, kind, weighting):
    ang = angles(K, kind)
    x = ph.rng_for(1951, K + N).normal(size=(2, N, N)).astype(np.float32)
    got = fbp.fbp_project(fbp.Geometry(K, D, N, dt, ang, weighting=weighting), torch.tensor(x, device="cuda")).cpu().numpy()
    ref = oracle.forward_splat(x.astype(np.float64), K, D, dt, ang)
    factor = 1.0
    if weighting == "angle-gaps":
        w = oracle.angle_weights(ang) * K / math.pi
        ref *= w[None, :, None]
        factor = float(np.max(w))
    terms = N * (2.0 * math.sqrt(2.0) * dt + 1.0)
    tol = (math.pi / K) * terms * 16 * 2.0 ** -24 * float(np.max(np.abs(x))) * factor
    assert np.max(np.abs(got - ref)) <= tol
