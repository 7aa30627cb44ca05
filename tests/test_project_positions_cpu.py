"""CPU replay of the staged projectors' fixed-point positions: a lane's pixel and phase,
anchored in FP64 per chunk and stepped in integers, against the position in FP64."""
import math

import numpy as np
import pytest

from paper_2109_02174_amd import phantom as ph
import test_fan_staged_cpu as fan
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


@pytest.mark.parametrize("K,D,N,ds,R", [(720, 801, 512, 1.0, 1024.0), (721, 801, 512, 1.0, 1024.0), (96, 150, 90, 0.8, 130.0),
                                        (61, 9000, 4096, 1.0, 9000.0)])
def test_fan_positions(K, D, N, ds, R):
    one = 1 << 25
    b = np.arange(K) * (2.0 * math.pi / K)
    _, tab = fan.table(b)
    half, cd = 0.5 * (N - 1), 0.5 * (D - 1)
    chunks = np.arange(0, N, fan.LINES)
    for _, c0, s0, _, _ in tab[:: max(1, len(tab) // 23)]:
        for j0 in {0, (D // 3) // BINS * BINS, (D - 1) // BINS * BINS}:
            g0 = cd - j0
            c, s = fan.turn_by(fan.turns(c0, s0, R, ds, g0 - 0.5 * (BINS - 1)), c0, s0)
            below = [fan.ray(c, s, R, ds, half, g0 - i + 1.0) for i in range(BINS)]
            p0, dp = (np.array([r[i] for r in below])[:, None] for i in (0, 1))
            ends = [below[0][0] + l * below[0][1] for l in (chunks, chunks + fan.LINES - 1)]
            ends += [below[-1][0] + l * below[-1][1] for l in (chunks, chunks + fan.LINES - 1)]
            lo, hi = np.min(ends, axis=0), np.max(ends, axis=0)
            meets = (lo - 2.0 <= N) & (hi + fan.TAPS + 3.0 >= 0.0) & (hi - lo + 5.5 <= fan.CELLS)
            if not np.any(meets):
                continue
            own, l0 = np.floor(lo[meets]) - 1, chunks[meets]
            for l in range(fan.LINES):
                q, li = divmod(l, 4)
                anchor = ((p0 + (l0 + li) * dp - own) * one).astype(np.int64)
                x = anchor + np.rint(4 * q * dp * one).astype(np.int64)
                assert np.all((x >= 0) & (x >> 25 < fan.CELLS))
                phase = ((x & (one - 1)) << 7).astype(np.float32).astype(np.float64) * 2.0 ** -32
                exact = p0 + (l0 + l) * dp - own
                assert np.max(np.abs((x >> 25) + phase - exact)) <= 1.5 * 2.0 ** -24
