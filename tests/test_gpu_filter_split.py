"""GPU: the FP32 filter through bf16 matrix products at the edges of its tiles.

Tiles of 16 and 32 rows by 32, 64 and 192 output bins of each parity, chunks of 32 inputs
per parity.  The cases sit on both sides of those (one bin, one row, a chunk or a tile
exactly, one more), take both kernels with and without even taps, fan-beam column weights,
rows too few for the tall tiles, and the detectors on both sides of the length the tap
copies allow.  Reference: the oracle in FP64; tolerance the FP32 dot product's, D ulps of
2^-24 of the largest input times the kernel's mass (1/(2 dt), fan beam half of it), as in
the filter's parity test.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ramlak", "hann"])
@pytest.mark.parametrize("K,D,B", [
    (511, 200, 1), (512, 200, 1), (512, 191, 1), (512, 192, 1),   # both sides of the sizes that take these kernels
    (512, 1, 1), (513, 255, 1), (528, 256, 1), (529, 257, 1), (543, 383, 1), (544, 384, 30), (527, 385, 1),
    (512, 385, 1), (600, 383, 30), (1001, 769, 13),      # tall tiles, ragged rows and bins
    (512, 2039, 1), (512, 2041, 1), (512, 4100, 1), (512, 5400, 1),   # longest detectors (even taps; odd taps only; past both)
])
def test_split_filter_matches_oracle(kind, K, D, B):
    g = fbp.Geometry(K, D, 16, 1.0, filter=kind)
    P = ph.rng_for(1900, K + D).normal(size=(B, K, D)).astype(np.float32)
    P[0, 0] *= 2.0 ** 40                                 # rows of very different size in one tile
    P[-1, -1] *= 2.0 ** -40
    got = fbp.fbp_filter(g, torch.tensor(P, device="cuda")).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(18), np.arange(K - 18, K), np.arange(0, K, 37)]))
    for b in {0, B // 2, B - 1}:
        ref = oracle.filter_rows(P[b:b + 1, rows].astype(np.float64), 1.0, kind)[0]
        bound = D * 2.0 ** -24 * np.max(np.abs(P[b, rows]), axis=-1, keepdims=True) / 2 * 4
        assert np.all(np.abs(got[b, rows] - ref) <= bound), b


@pytest.mark.parametrize("K,D,B", [(512, 201, 1), (600, 400, 20)])
def test_split_filter_with_column_weights(K, D, B):
    R = 500.0
    g = fbp.Geometry(K, D, 16, 1.0, source_distance=R)
    P = ph.rng_for(1901, K).normal(size=(B, K, D)).astype(np.float32)
    got = fbp.fbp_filter(g, torch.tensor(P, device="cuda")).cpu().numpy()
    s = np.arange(D) - 0.5 * (D - 1)
    w = (R / np.sqrt(R * R + s * s)).astype(np.float32)
    ref = 0.5 * oracle.filter_rows((P[-1:] * w).astype(np.float64), 1.0, "ramlak")[0]
    assert np.max(np.abs(got[-1] - ref)) <= D * 2.0 ** -24 * np.max(np.abs(P)) / 4 * 4


@pytest.mark.parametrize("K,D", [(512, 192), (600, 534)])
def test_shepp_logan_stays_on_fp32_products(K, D):
    """The same rows in a geometry of too few angles for the bf16 products: the same bits."""
    P = ph.rng_for(1903, K).normal(size=(1, K, D)).astype(np.float32)
    few = 128
    want = fbp.fbp_filter(fbp.Geometry(few, D, 16, 1.0, filter="shepp-logan"), torch.tensor(P[:, :few], device="cuda"))
    got = fbp.fbp_filter(fbp.Geometry(K, D, 16, 1.0, filter="shepp-logan"), torch.tensor(P, device="cuda"))
    assert torch.equal(got[:, :few], want)


def test_large_and_non_finite_inputs():
    """Values up to FLT_MAX stay finite where the sum is; a non-finite input makes its own
    bin and the bins of the other parity of its row non-finite, and no others."""
    K, D = 512, 200
    g = fbp.Geometry(K, D, 16, 1.0)
    P = ph.rng_for(1902, 0).normal(size=(1, K, D)).astype(np.float32)
    clean = fbp.fbp_filter(g, torch.tensor(P, device="cuda")).cpu().numpy()
    P[0, 3, 50] = np.inf
    P[0, 7, 51] = np.nan
    P[0, 9] = 0.0
    P[0, 9, 60] = np.finfo(np.float32).max
    got = fbp.fbp_filter(g, torch.tensor(P, device="cuda")).cpu().numpy()[0]
    j = np.arange(D)
    assert np.array_equal(np.isfinite(got[3]), (j % 2 == 0) & (j != 50))
    assert np.array_equal(np.isfinite(got[7]), (j % 2 == 1) & (j != 51))
    ref = oracle.filter_rows(P[:, 9:10].astype(np.float64), 1.0, "ramlak")[0, 0]
    assert np.all(np.abs(got[9] - ref) <= D * 2.0 ** -24 * np.finfo(np.float32).max / 2 * 4)
    rest = [k for k in range(K) if k not in (3, 7, 9)]
    assert np.array_equal(got[rest], clean[0][rest])
