"""CPU replay of the staged fan-beam projector: the host's grouping rule and the kernel's
turns, windows, tap counts and positions, restated in NumPy.

Asserts that every LDS read of every lane stays inside the staged window (96 pixels a
row), and that the sums of the replay in FP64 equal the oracle's adjoint, for quarter-turn
and other view lists, odd sides, sources near the image and coarse and fine detectors.
No GPU is involved.
"""
import math

import numpy as np
import pytest

import oracle

BINS, LINES, CELLS, WAVES, TAPS, DEPTH = 16, 8, 96, 8, 6, 16.0


def turn_by(q, c, s):
    return [(c, s), (-s, c), (-c, -s), (s, -c)][q]


def turns(c, s, R, ds, g):
    dx, dy = g * ds * s - R * c, -g * ds * c - R * s
    if abs(dy) >= abs(dx):
        return 0 if dy > 0 else 2
    return 1 if dx > 0 else 3


def ray(c, s, R, ds, half, g):
    inv = 1.0 / (-R * s / ds - g * c)
    dp = -(R * c / ds - g * s) * inv
    return half - g * R * inv - dp * half, dp


def reach(c, s, R, ds, half, g0, r0, r1):
    at = {}
    for n, o in (("a", 1.0), ("b", -1.0), ("c", -(BINS - 2)), ("d", -BINS)):
        p0, dp = ray(c, s, R, ds, half, g0 + o)
        at[n] = np.array([p0 + r0 * dp, p0 + r1 * dp])
    ends = np.concatenate([at["a"], at["c"]])
    width = max(np.abs(at["b"] - at["a"]).max(), np.abs(at["d"] - at["c"]).max())
    return ends.min(), ends.max(), width


def quarter_turns(b):
    K = len(b)
    if K < 4 or K % 4:
        return False
    q = K // 4
    return all(abs(math.remainder(b[k + i * q] - b[k] - 0.5 * math.pi * i, 2 * math.pi)) <= 1e-12
               for k in range(q) for i in (1, 2, 3))


def table(b):
    quarter = quarter_turns(b)
    tab = []
    for k in range(len(b) // 4 if quarter else len(b)):
        c, s, t = math.cos(b[k]), math.sin(b[k]), 0
        while quarter and not (c > 0 and s >= 0) and t < 4:
            c, s, t = s, -c, t + 1
        tab.append((math.atan2(s, c), c, s, k, t & 3))
    return quarter, sorted(tab, key=lambda e: e[0])


def group_views(tab, N, D, R, ds):
    if N > 4096 or not (R - 0.70710678118654752 * N >= DEPTH + TAPS + 2.0):
        return 0
    half, cd = 0.5 * (N - 1), 0.5 * (D - 1)
    nch = (N + LINES - 1) // LINES

    def group_fits(ents, j0):
        g0 = cd - j0
        em = ents[len(ents) >> 1]
        q = turns(em[1], em[2], R, ds, g0 - 0.5 * (BINS - 1))
        walks = [turn_by(q, e[1], e[2]) for e in ents]
        for c, s in walks:
            for g in (g0 + 1.0, g0 - BINS):
                dx, dy = g * ds * s - R * c, -g * ds * c - R * s
                if dy < 0.5 * math.hypot(dx, dy):
                    return False

        def chunk(ch):
            fs = [reach(c, s, R, ds, half, g0, ch * LINES, ch * LINES + LINES - 1) for c, s in walks]
            lo, hi, width = min(f[0] for f in fs), max(f[1] for f in fs), max(f[2] for f in fs)
            taps = math.ceil(width)
            if lo - 2.0 > N or hi + taps + 3.0 < 0.0:
                return 0
            return 1 if width <= TAPS - 0.01 and hi - lo + taps + 4.5 <= CELLS else -1

        for order in (range(nch), range(nch - 1, -1, -1)):
            first = next((f for f in map(chunk, order) if f), 1)
            if first < 0:
                return False
        return True

    A = WAVES
    while A >= 1:
        if all(group_fits(tab[i0:i0 + A], j0) for i0 in range(0, len(tab), A) for j0 in range(0, D, BINS)):
            return A
        A >>= 1
    return 0


def replay(img, b, D, ds, R, per):
    """Sums of the kernel in FP64, and the bounds of its LDS reads."""
    N, K = img.shape[0], len(b)
    half, cd = 0.5 * (N - 1), 0.5 * (D - 1)
    quarter, tab = table(b)
    M = 4 if quarter else 1
    tr = img.T
    turned = [img, tr[::-1], img[::-1, ::-1], tr[:, ::-1]]
    nch = (N + LINES - 1) // LINES
    big = np.zeros((4, nch * LINES, N + 2 * CELLS))
    for m in range(4):
        big[m, :N, CELLS:CELLS + N] = turned[m]
    out = np.full((K, D), np.nan)
    lane_g = np.arange(BINS)
    for i0 in range(0, len(tab), per):
        ents = tab[i0:i0 + per]
        for j0 in range(0, D, BINS):
            g0 = cd - j0
            em = ents[len(ents) >> 1]
            q = turns(em[1], em[2], R, ds, g0 - 0.5 * (BINS - 1))
            acc = np.zeros((len(ents), M, BINS))
            for ch in range(nch):
                fs = [reach(*turn_by(q, e[1], e[2]), R, ds, half, g0, ch * LINES, ch * LINES + LINES - 1) for e in ents]
                owns = [math.floor(f[0]) - 1 for f in fs]
                wlo, T = min(owns), max(min(TAPS, math.ceil(f[2])) for f in fs)
                end = max(math.floor(f[1]) for f in fs) + T + 2
                if wlo >= N or end <= 0:
                    continue
                assert end - wlo <= CELLS
                for ie, e in enumerate(ents):
                    c, s = turn_by(q, e[1], e[2])
                    p0, dp = ray(c, s, R, ds, half, g0 - lane_g)
                    b0, db = ray(c, s, R, ds, half, g0 - lane_g + 1.0)
                    eq = (-R * s / ds - (g0 - lane_g) * c) / R
                    for l in range(ch * LINES, ch * LINES + LINES):
                        x = (b0 + l * db - owns[ie])
                        # FP32 as in the kernel, for the index bounds
                        x32 = x.astype(np.float32)
                        i32 = np.trunc(x32).astype(int)
                        assert i32.min() >= 0 and (owns[ie] - wlo) + i32.min() + 1 >= 0
                        assert (owns[ie] - wlo) + i32.max() + T < CELLS
                        i = np.floor(x).astype(int)
                        dep = np.maximum(1.0 - ((p0 + l * dp - half) * c + (l - half) * s) / R, DEPTH / R)
                        d0 = i + 1 - x - (p0 + l * dp - b0 - l * db)
                        for m in range(T):
                            d = d0 + m
                            inv = 1.0 / (dep - c / R * d)
                            w = np.clip(1.0 - np.abs(d) * eq * inv, 0.0, 1.0) * inv * inv
                            p = np.clip(owns[ie] + i + m + 1, -CELLS, N + CELLS - 1) + CELLS
                            for y in range(M):
                                acc[ie, y] += w * big[y if M == 4 else (4 - q) & 3, l, p]
            for ie, e in enumerate(ents):
                for y in range(M):
                    k = e[3] + ((q - e[4] + y) & 3) * (K // 4) if quarter else e[3]
                    n = min(BINS, D - j0)
                    assert np.all(np.isnan(out[k, j0:j0 + n]))
                    out[k, j0:j0 + n] = acc[ie, y, :n] * 2.0 * math.pi / K
    return out


def views(K, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        return np.arange(K) * (2.0 * math.pi / K)
    if kind == "quarter":         # unsorted first quarter, anywhere on the circle
        q = rng.uniform(-math.pi, math.pi, K // 4)
        return np.concatenate([q + i * 0.5 * math.pi for i in range(4)])
    return rng.uniform(-7.0, 7.0, K)


@pytest.mark.parametrize("N,K,D,ds,R,kind", [
    (40, 96, 61, 1.0, 80.0, "uniform"), (33, 40, 49, 1.1, 90.0, "random"), (48, 36, 97, 0.7, 70.0, "quarter"),
    (17, 25, 31, 0.7, 45.0, "random"), (64, 32, 80, 1.0, 72.0, "quarter"), (64, 31, 60, 1.2, 260.0, "random"),
    (1, 5, 3, 1.0, 90.0, "random"), (9, 4, 1, 1.0, 40.0, "uniform"), (130, 16, 15, 1.0, 600.0, "uniform"),
])
def test_replay_equals_the_oracle_adjoint(N, K, D, ds, R, kind):
    b = views(K, kind, N + K)
    _, tab = table(b)
    most = group_views(tab, N, D, R, ds)
    assert most > 0
    img = np.random.default_rng(N * K + D).normal(size=(N, N))
    ref = oracle.fan_splat(img, K, D, ds, R, b)
    per = most
    while True:
        got = replay(img, b, D, ds, R, per)
        assert np.max(np.abs(got - ref)) <= 1e-11 * max(np.max(np.abs(ref)), 1e-3)
        if per <= 2:
            break
        per >>= 1


@pytest.mark.parametrize("N,K,D,ds,R,fits", [
    (512, 720, 801, 1.0, 1024.0, True), (512, 720, 1100, 1.0, 768.0, True), (1024, 1440, 1500, 1.0, 4096.0, True),
    (64, 60, 40, 4.0, 130.0, False),      # too many pixels per row
    (64, 60, 90, 1.0, 60.0, False),       # source too close
    (512, 8, 801, 1.0, 1024.0, True),     # views too far apart to share a window
])
def test_grouping_rule(N, K, D, ds, R, fits):
    _, tab = table(np.arange(K) * (2.0 * math.pi / K))
    A = group_views(tab, N, D, R, ds)
    assert (A > 0) == fits
    print(N, K, A)
