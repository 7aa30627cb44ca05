"""GPU: the staged fan-beam projector at the edges of its tiles.

Workgroups own 16 bins of up to eight neighbouring base views and stage 8 image rows of
at most 96 pixels; a walk serves the four quarter turns of a view where the list is closed
under them, and two or four slices of a stack.  The cases sit on the edges of the bin
blocks, the row chunks, the tap counts (detector spacing, source distance), the view
groups and the slice sets, and on both sides of the rule that keeps coarse detectors and
close sources on the one-lane kernel.  Reference: the oracle's adjoint in FP64; tolerance
256 FP32 ulps of the largest term for each of a bin's terms, as in the projector's parity
test.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


def _tol(x, N, K, R, T=9):
    wmax = (R / (R - math.sqrt(2.0) * 0.5 * N)) ** 2
    return (2.0 * math.pi / K) * N * T * wmax * 256 * 2.0 ** -24 * float(np.max(np.abs(x))) + 1e-30


def _views(K, kind, seed):
    rng = ph.rng_for(1700, seed)
    if kind == "uniform":
        return np.arange(K) * (2.0 * math.pi / K)
    if kind == "quarter":         # unsorted first quarter, anywhere on the circle
        q = rng.uniform(-math.pi, math.pi, K // 4)
        return np.concatenate([q + i * 0.5 * math.pi for i in range(4)])
    return rng.uniform(-7.0, 7.0, K)


@pytest.mark.parametrize("K,D,N,dt,R,B,kind", [
    (96, 48, 32, 1.0, 80.0, 1, "uniform"),     # three blocks of bins, two chunks of rows
    (96, 49, 33, 1.0, 80.0, 2, "uniform"),     # one bin and one row more
    (100, 47, 31, 1.0, 80.0, 3, "quarter"),    # one fewer; a set of slices half full
    (45, 61, 40, 1.0, 100.0, 1, "random"),     # no quarter turns
    (45, 61, 40, 1.0, 100.0, 2, "random"),
    (46, 61, 40, 1.0, 100.0, 5, "random"),
    (720, 145, 100, 1.0, 400.0, 1, "uniform"),   # dense views: eight share a window
    (720, 145, 100, 1.0, 200.0, 3, "uniform"),   # four share one
    (723, 145, 100, 1.0, 200.0, 4, "uniform"),
    (4, 145, 100, 1.0, 400.0, 1, "uniform"),   # one base view
    (60, 260, 100, 0.55, 400.0, 2, "uniform"),   # two and three pixels per row
    (60, 360, 100, 0.4, 250.0, 1, "quarter"),  # one
    (60, 130, 100, 1.3, 400.0, 1, "uniform"),
    (360, 163, 100, 1.0, 150.0, 2, "uniform"),   # wide fan
    (64, 40, 64, 3.0, 130.0, 2, "uniform"),    # too coarse to stage
    (64, 90, 64, 1.0, 60.0, 1, "uniform"),     # source too close to stage
    (90, 1, 40, 1.0, 160.0, 1, "uniform"),     # one bin
    (8, 300, 260, 1.0, 1000.0, 1, "uniform"),  # detector shorter than the image
])
def test_staged_fan_projector_matches_oracle(K, D, N, dt, R, B, kind):
    b = _views(K, kind, K * D + N)
    x = ph.rng_for(1701, K + N).normal(size=(B, N, N)).astype(np.float32)
    got = fbp.fbp_project(fbp.Geometry(K, D, N, dt, b, source_distance=R), torch.tensor(x, device="cuda")).cpu().numpy()
    ref = oracle.fan_splat(x.astype(np.float64), K, D, dt, R, b)
    assert np.max(np.abs(got - ref)) <= _tol(x, N, K, R)


@pytest.mark.parametrize("K,D,N,R", [(360, 183, 128, 300.0), (301, 183, 128, 300.0)])
def test_a_slice_alone_equals_its_place_in_a_stack(K, D, N, R):
    """Short and long calls put different numbers of views and slices in a workgroup; the
    sums are the same."""
    g = fbp.Geometry(K, D, N, 1.0, source_distance=R)
    x = torch.tensor(ph.rng_for(1702, N).normal(size=(19, N, N)).astype(np.float32), device="cuda")
    whole = fbp.fbp_project(g, x).cpu().numpy()
    for i in (0, 11, 18):
        assert np.array_equal(fbp.fbp_project(g, x[i:i + 1].contiguous()).cpu().numpy()[0], whole[i]), i
