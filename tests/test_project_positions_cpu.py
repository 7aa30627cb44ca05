"""CPU replay of the staged projectors' fixed-point positions: a lane's pixel and phase,
anchored in FP64 per chunk and stepped in integers, against the position in FP64."""
import math

import numpy as np
import pytest

from paper_2109_02174_amd import phantom as ph
from test_project_windows_cpu import BINS, CELLS, LINES, base_table, group_angles, ranges

ONE = 1 << 26


@pytest.mark.parametrize("K,D,N,dt,kind", [
    (720, 725, 512, 1.0, "uniform"), (1201, 725, 512, 1.0, "golden"), (719, 725, 511, 0.75, "uniform"),
    (400, 150, 130, 1.3, "uniform"), (300, 500, 112, 0.3, "uniform"), (60, 23171, 16384, 1.0, "uniform"),
])
def test_parallel_positions(K, D, N, dt, kind):
    ang = ph.uniform_angles(K) if kind == "uniform" else np.mod(np.arange(K) * math.pi * (math.sqrt(5.0) - 1.0) / 2.0, math.pi)
    tab, n0, quarter = base_table(ang, dt)
    rs = [1 / e[0] for e in tab]
    T = 3 if min(rs) >= 1.0 and max(rs) <= 1.5 else math.ceil(2 * max(rs))
    A = group_angles(tab, n0, T, N)
    assert A >= 1
    half, cd = 0.5 * (N - 1), 0.5 * (D - 1)
    l0 = np.arange(0, N, LINES)
    for a, b, *_ in tab[:: max(1, len(tab) // 23)]:
        inv, dl = 1 / a, -b / a
        for j0 in {0, ((D + 1) // 4) // BINS * BINS, (D - 1) // 2 // BINS * BINS}:
            j = np.arange(j0, j0 + BINS)[:, None]
            xj = (j - cd + b * half) * inv + half - inv
            own = np.floor(xj[0] + min(0.0, (LINES - 1) * dl) + l0 * dl) - 1
            for l in range(LINES):
                q, li = divmod(l, 4)
                anchor = ((xj + (l0 + li) * dl - own) * ONE).astype(np.int64)
                x = anchor + int(np.rint(4 * q * dl * ONE))
                assert np.all((x >> 26 >= 0) & ((x >> 26) + T < CELLS))
                phase = ((x & (ONE - 1)) << 6).astype(np.float32).astype(np.float64) * 2.0 ** -32
                exact = xj + (l0 + l) * dl - own
                assert np.max(np.abs((x >> 26) + phase - exact)) <= 2.0 ** -24
