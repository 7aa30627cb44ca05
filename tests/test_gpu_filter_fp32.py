"""GPU: every FP32 filter row comes from the FP32 matrix product, whatever calls it.

A row's bits depend on the row, the detector and the kernel alone, not on how many angles,
slices or views the call has.  Its error against 64 bits is that of FP32 products and sums:
about 2^-24 of the row's root sum of squares (inputs times taps) for each of the D/2 terms
of a sum, adding like a random walk.  Measured in NumPy, a filter that multiplies bf16
pairs instead (three products: relative error 2^-16 a term) is 2 to 6 times past this
bound at the sizes below, FP32 sums at 0.15 to 0.43 of it.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu

FEW = 128            # rows of the small geometry that the same rows are filtered in again


def _rows(seed, n, D):
    return torch.tensor(ph.rng_for(1920, seed).normal(size=(n, D)).astype(np.float32), device="cuda")


def _few(rows, D, kind, dt=1.0):
    g = fbp.Geometry(FEW, D, 16, dt, filter=kind)
    return fbp.fbp_filter(g, rows.reshape(-1, FEW, D)).reshape(-1, D)


@pytest.mark.parametrize("kind", ["ramlak", "shepp-logan", "hann"])
@pytest.mark.parametrize("K,D,B", [(512, 200, 1), (640, 725, 1), (1024, 257, 30), (1408, 1451, 1), (512, 2100, 1)])
def test_rows_have_the_same_bits_in_any_geometry(kind, K, D, B):
    rows = _rows(K + D, B * K, D)
    got = fbp.fbp_filter(fbp.Geometry(K, D, 16, 1.0, filter=kind), rows.reshape(B, K, D))
    assert torch.equal(got.reshape(-1, D), _few(rows, D, kind))


def test_rows_of_fan_and_cone_geometries_too():
    """Fan-beam column weights and cone-beam pre-weights are FP32 products before the filter,
    and half the kernel is an exact halving after it."""
    K, D, R = 640, 385, 700.0
    rows = _rows(1, K, D)
    s = np.arange(D) - 0.5 * (D - 1)
    w = torch.tensor((R / np.sqrt(R * R + s * s)).astype(np.float32), device="cuda")
    got = fbp.fbp_filter(fbp.Geometry(K, D, 16, 1.0, source_distance=R), rows[None])[0]
    assert torch.equal(got, 0.5 * _few(rows * w, D, "ramlak"))
    views, Dv = 10, 64
    z = np.arange(Dv) - 0.5 * (Dv - 1)
    pw = torch.tensor((R / np.sqrt(R * R + s[None] ** 2 + z[:, None] ** 2)).astype(np.float32), device="cuda")
    got = fbp.fbp_cone_filter(fbp.ConeGeometry(views, D, Dv, 16, 8, R), rows.reshape(views, Dv, D))
    assert torch.equal(got.reshape(K, D), 0.5 * _few((rows.reshape(views, Dv, D) * pw).reshape(K, D), D, "ramlak"))


@pytest.mark.parametrize("kind", ["ramlak", "hann"])
@pytest.mark.parametrize("K,D", [(512, 200), (512, 725), (512, 1451)])
def test_error_against_64_bits_is_that_of_fp32_sums(kind, K, D):
    rows = _rows(K * D, K, D)
    got = fbp.fbp_filter(fbp.Geometry(K, D, 16, 1.0, filter=kind), rows[None])[0].cpu().numpy()
    P = rows[:64].cpu().numpy().astype(np.float64)
    ref = oracle.filter_rows(P[None], 1.0, kind)[0]
    unit = np.zeros((1, 1, 2 * D - 1))
    unit[0, 0, D - 1] = 1.0
    taps = oracle.filter_rows(unit, 1.0, kind)[0, 0]
    bound = 2.0 ** -24 * math.sqrt(0.5 * D) * math.sqrt(np.sum(taps ** 2))        # inputs of variance 1
    assert np.sqrt(np.mean((got[:64] - ref) ** 2)) <= bound


def test_an_infinite_sample_gives_infinities():
    """Its own bin and the bins of the other parity (all of whose taps are negative); the
    other bins of the row and the other rows stay as they are."""
    K, D = 512, 200
    g = fbp.Geometry(K, D, 16, 1.0)
    rows = _rows(3, K, D)
    clean = fbp.fbp_filter(g, rows[None])[0].cpu().numpy()
    rows[3, 50] = math.inf
    got = fbp.fbp_filter(g, rows[None])[0].cpu().numpy()
    want = clean.copy()
    want[3, 1::2] = -math.inf
    want[3, 50] = math.inf
    assert np.array_equal(got, want)
