"""GPU: fan-beam stacks in groups of two and four slices, the last group short.

A group past the end of the stack repeats its last slice and does not write it: every slice
equals the oracle's and, bit for bit, the same slice in a longer stack, and memory after
the image stays as it was.  Both kernels (quarter-turn lists and others, odd sides with the
centre pixel), stack lengths on both sides of a group, and images large enough for groups
of four.  Tolerance: that of the fan backprojection's parity test.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


def _bp_tol(Q, N, R):
    Q = np.asarray(Q, np.float64)
    M = R / (R - (N - 1) / math.sqrt(2.0))
    dq = np.max(np.abs(np.diff(Q, axis=-1)))
    return 2.0 * math.pi * M * M * (1e-5 * max(dq, np.max(np.abs(Q))) + 1e-6 * np.max(np.abs(Q))) + 1e-6


@pytest.mark.parametrize("N,K,D", [(48, 40, 73), (33, 40, 53), (48, 41, 73), (360, 16, 520), (361, 13, 520)])
def test_short_last_groups(N, K, D):
    R = 2.0 * N
    g = fbp.Geometry(K, D, N, 1.0, source_distance=R)
    Q = ph.rng_for(2000, N + K).normal(size=(19, K, D)).astype(np.float32)
    q = torch.tensor(Q, device="cuda")
    ref = oracle.fan_backproject(Q[:6].astype(np.float64), N, 1.0, R, g.angles)
    first = {}
    for n in (4, 5, 6, 7, 16, 17, 18, 19):
        out = torch.full((n + 1, N, N), 7.0, device="cuda")
        fbp.fbp_backproject(g, q[:n].contiguous(), out=out[:n])
        got = out.cpu().numpy()
        assert np.all(got[n] == 7.0), n
        assert np.max(np.abs(got[:min(n, 6)] - ref[:min(n, 6)])) <= _bp_tol(Q, N, R), n
        for s in range(n):
            assert np.array_equal(got[s], first.setdefault(s, got[s])), (n, s)
