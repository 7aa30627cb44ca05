"""GPU: the forward projectors' error against 64 bits on an image of pixel noise.

Noise has no smoothness for a position error to hide in: moving every hat by e changes a
bin by about e times the root sum of squares of the pixel differences it meets.  Positions
are held to about 2^-26 of a pixel, so what remains is the rounding of each weight (once or
twice, 2^-24) and of the sums; a NumPy replay of the kernels' arithmetic gives 1.1 to 1.3
(parallel beam) and 1.7 to 1.9 (fan beam) times 2^-24 sqrt(3 N) of the noise, root mean
square over the bins.  FP32 positions over a window of 64 or 96 pixels would give 4.4 to 7.3
and 4.8 to 5.4.  The bounds are twice the replay's largest.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu

N = 512


def _image(seed):
    return ph.rng_for(1930, seed).normal(size=(1, N, N)).astype(np.float32)


@pytest.mark.parametrize("K,kind", [(720, "uniform"), (1201, "golden")])
def test_parallel_projector(K, kind):
    D = 725
    ang = ph.uniform_angles(K)
    if kind == "golden":
        ang = np.mod(np.arange(K) * math.pi * (math.sqrt(5.0) - 1.0) / 2.0, math.pi)
    x = _image(0)
    got = fbp.fbp_project(fbp.Geometry(K, D, N, 1.0, ang), torch.tensor(x, device="cuda")).cpu().numpy()[0]
    unit = (math.pi / K) * 2.0 ** -24 * math.sqrt(3.0 * N)
    for k in (1, K // 16, K // 5, K // 3, (2 * K) // 3, K - 7):
        ref = oracle.forward_splat(x[0].astype(np.float64), 1, D, 1.0, ang[k:k + 1])[0] / K
        assert np.sqrt(np.mean((got[k] - ref) ** 2)) <= 2.6 * unit, k


@pytest.mark.parametrize("K", [720, 721])
def test_fan_projector(K):
    D, R = 801, 1024.0
    b = np.arange(K) * (2.0 * math.pi / K)
    x = _image(1)
    got = fbp.fbp_project(fbp.Geometry(K, D, N, 1.0, b, source_distance=R), torch.tensor(x, device="cuda")).cpu().numpy()[0]
    unit = (2.0 * math.pi / K) * 2.0 ** -24 * math.sqrt(3.0 * N)
    for k in (1, K // 16, K // 5, K // 3, (2 * K) // 3, K - 7):
        ref = oracle.fan_splat(x[0].astype(np.float64), 1, D, 1.0, R, b[k:k + 1])[0] / K
        assert np.sqrt(np.mean((got[k] - ref) ** 2)) <= 3.8 * unit, k
