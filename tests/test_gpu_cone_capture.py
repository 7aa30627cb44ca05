"""GPU: a captured cone-beam backprojection gives the bits of the eager call.

Small volumes split their views over partial volumes; a captured call cannot use them (its
replays would not wait for other calls) and adds the parts into the volume one after
another, in the same order.  Volumes with and without a split, quarter-turn lists (odd sides
with their centre column) and others.
"""
import numpy as np
import pytest
import torch

import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import phantom as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,Nz", [(40, 33, 20), (42, 33, 20), (64, 32, 33), (150, 17, 5), (4, 24, 20), (36, 200, 130),
                                    (36, 17, 300)])    # windows too large for LDS: direct reads
def test_replays_equal_the_eager_volume(K, N, Nz):
    R = 1.9 * N
    g = fbp.ConeGeometry(K, int(1.6 * N), int(1.4 * Nz) + 3, N, Nz, R)
    Q = ph.rng_for(1940, K + N).normal(size=(3, K, int(1.4 * Nz) + 3, int(1.6 * N))).astype(np.float32)
    q = torch.tensor(Q, device="cuda")
    ref = [fbp.fbp_cone_backproject(g, q[i]) for i in range(3)]
    buf, out = q[0].clone(), torch.full(g.volume_shape(), float("nan"), device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fbp.fbp_cone_backproject(g, buf, out=out, stream=torch.cuda.current_stream())
    for rep in range(3):
        buf.copy_(q[rep])
        out.fill_(float(rep))
        other = fbp.fbp_cone_backproject(g, q[(rep + 1) % 3])      # an eager call between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref[rep]), rep
        assert torch.equal(other, ref[(rep + 1) % 3]), rep
