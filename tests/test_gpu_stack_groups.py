"""GPU: stacks of other than quarter-turn lists on both sides of the rule that groups slices.

Slices go in groups of two or four per workgroup only where the groups outnumber the CUs;
small stacks go one slice per workgroup.  Copies of one slice must give the same bits at
every position either way, and the first equals the oracle's, with the tolerance of the
stack parity test.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,B", [(600, 7, 9), (300, 9, 4), (300, 9, 33), (200, 11, 37)])
def test_grouped_and_single_slices_agree(N, K, B):
    D = int(math.ceil(math.sqrt(2.0) * N)) + 2
    ang = ph.rng_for(2100, N + K).uniform(0.0, math.pi, K)
    g = fbp.Geometry(K, D, N, 1.0, ang)
    Q = ph.rng_for(2101, N).normal(size=(1, K, D)).astype(np.float32)
    q = torch.tensor(Q, device="cuda").expand(B, K, D).contiguous()
    ref = oracle.backproject(Q.astype(np.float64), N, 1.0, ang)[0]
    dq = np.max(np.abs(np.diff(Q, axis=-1)))
    tol = math.pi * (1e-4 * max(dq, np.max(np.abs(Q))) + 1e-5 * np.max(np.abs(Q))) + 1e-6
    for cfg in range(fbp.fbp_num_tile_configs()):
        if "slice stacks" not in fbp.fbp_tile_config_name(cfg):
            continue
        out = torch.full((B, N, N), float("nan"), device="cuda")
        fbp.fbp_backproject_with_config(g, q, cfg, out=out)
        got = out.cpu().numpy()
        assert np.max(np.abs(got[0] - ref)) <= tol, cfg
        for s in range(1, B):
            assert np.array_equal(got[0], got[s]), (cfg, s)
