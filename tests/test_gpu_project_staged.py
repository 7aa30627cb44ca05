"""GPU: the staged forward projector at the edges of its tiles.

Workgroups own 16 bins of up to eight neighbouring base angles and stage 16 image
rows of at most 64 pixels at a time; a base angle serves two bins (any list) or four
(lists closed under +pi/2).  The cases sit on the edges of the bin blocks (half the
detector a multiple of 16, one more, one less; the middle bin of an odd detector),
of the row chunks, of the tap counts (detector spacings) and of the angle groups
(dense lists, lists too sparse to share a window, fewer angles than a group), and
detectors too coarse to stage.  Reference: the oracle's adjoint in FP64, with the
tolerance of the projector's own parity test (16 FP32 ulps of the largest pixel for
each of the N (2 sqrt(2) dt + 1) terms of a bin).
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


def _tol(x, N, dt, K):
    terms = N * (2.0 * math.sqrt(2.0) * dt + 1.0)
    return (math.pi / K) * terms * 16 * 2.0 ** -24 * float(np.max(np.abs(x))) + 1e-30


def _angles(K, kind, seed):
    if kind == "uniform":
        return ph.uniform_angles(K)
    if kind == "golden":
        return np.mod(np.arange(K) * math.pi * (math.sqrt(5.0) - 1.0) / 2.0, math.pi)
    if kind == "quarter":       # random angles over the whole turn, each with its quarter turn
        h = ph.rng_for(1600, seed).uniform(-math.pi, math.pi, K // 2)
        return np.concatenate([h, h + 0.5 * math.pi])
    return ph.rng_for(1601, seed).uniform(-2.0 * math.pi, 2.0 * math.pi, K)


@pytest.mark.parametrize("K,D,N,dt,B,kind", [
    (90, 31, 16, 1.0, 1, "uniform"),     # half detector of 16 bins, one chunk of rows
    (90, 32, 17, 1.0, 2, "uniform"),     # even detector; one row into a second chunk
    (92, 33, 15, 1.0, 1, "quarter"),     # half detector of 17 bins
    (64, 97, 64, 1.0, 1, "uniform"),
    (61, 96, 65, 1.0, 1, "uniform"),     # odd count: two bins per angle
    (400, 190, 130, 1.0, 1, "golden"),   # dense after sorting
    (2, 400, 260, 1.0, 1, "uniform"),    # one base angle
    (3, 400, 260, 1.0, 2, "random"),     # too far apart to share a window
    (6, 430, 300, 1.0, 1, "quarter"),
    (120, 181, 80, 0.6, 1, "uniform"),   # two taps
    (120, 190, 64, 0.45, 1, "golden"),   # one tap
    (120, 110, 100, 1.3, 1, "uniform"),  # four taps
    (37, 60, 70, 1.9, 1, "random"),      # too coarse to stage
    (36, 24, 90, 6.0, 1, "uniform"),
    (720, 181, 128, 1.0, 1, "uniform"),
    (720, 159, 112, 1.0, 1, "uniform"),  # the smallest staged image; half detector of 80 bins
    (720, 161, 113, 1.0, 2, "uniform"),  # one bin and one row more
    (720, 160, 111, 1.0, 1, "uniform"),  # one below the smallest
    (300, 183, 128, 1.0, 3, "uniform"),  # four angles share a window
    (1001, 190, 130, 1.0, 2, "golden"),  # eight, two bins per angle
    (1001, 190, 130, 1.0, 1, "uniform"),
    (720, 300, 112, 0.6, 1, "uniform"),  # two taps
    (720, 400, 113, 0.45, 1, "uniform"),   # one tap
    (720, 140, 127, 1.3, 1, "uniform"),  # four taps
])
def test_staged_projector_matches_oracle(K, D, N, dt, B, kind):
    ang = _angles(K, kind, K * D + N)
    x = ph.rng_for(1602, K + N).normal(size=(B, N, N)).astype(np.float32)
    got = fbp.fbp_project(fbp.Geometry(K, D, N, dt, ang), torch.tensor(x, device="cuda")).cpu().numpy()
    ref = oracle.forward_splat(x.astype(np.float64), K, D, dt, ang)
    assert np.max(np.abs(got - ref)) <= _tol(x, N, dt, K)


@pytest.mark.parametrize("K,D,N,kind", [(360, 183, 128, "uniform"), (301, 183, 128, "golden")])
def test_a_slice_alone_equals_its_place_in_a_stack(K, D, N, kind):
    """Short and long calls put different numbers of angles in a workgroup; the sums
    are the same."""
    g = fbp.Geometry(K, D, N, 1.0, _angles(K, kind, 0))
    x = torch.tensor(ph.rng_for(1603, N).normal(size=(24, N, N)).astype(np.float32), device="cuda")
    whole = fbp.fbp_project(g, x).cpu().numpy()
    for i in (0, 11, 23):
        assert np.array_equal(fbp.fbp_project(g, x[i:i + 1].contiguous()).cpu().numpy()[0], whole[i]), i
