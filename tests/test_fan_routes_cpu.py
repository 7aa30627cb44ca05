"""How fan-beam stacks are grouped, on a HIP runtime of host memory (fake_hip.cpp): slices
singly where groups of four would be fewer than the CUs, in twos below three groups of four a
CU, else in whole fours and the rest singly (a short last group of four costs a whole one)."""
import json

from fake_hip import run

CUS = 256

# side, angles, slices, launches as (slices per workgroup, workgroups per tile)
CASES = [
    (128, 360, 4, [(1, 4)]), (150, 361, 5, [(1, 5)]),
    (365, 540, 12, [(2, 6)]), (365, 540, 13, [(2, 7)]), (300, 361, 7, [(2, 4)]),
    (1024, 720, 4, [(4, 1)]), (1365, 500, 13, [(4, 3), (1, 1)]), (1254, 500, 15, [(4, 3), (1, 3)]),
    (188, 601, 33, [(4, 8), (1, 1)]), (343, 1000, 33, [(4, 8), (1, 1)]), (512, 721, 6, [(4, 1), (1, 2)]),
    (512, 720, 3, None), (1700, 722, 3, [(1, 3)]),
]


def test_groups():
    plain = [[N, K, n] for N, K, n, _ in CASES]
    got = run(f"""
result = []
for N, K, n in json.loads({json.dumps(json.dumps(plain))}):
    g = fbp.Geometry(K, int(1.6 * N), N, 1.0, source_distance=2.0 * N)
    fake.fake_reset()
    assert call("fbp_backproject", g, n, A, C) == 0
    result.append(launched())
""")
    for (N, K, n, want), launches in zip(CASES, got):
        rot = K % 4 == 0
        tiles = (((N + 1) // 2 + 15) // 16) * ((N // 2 + 15) // 16) if rot else ((N + 15) // 16) ** 2
        name = "fan_rot_kernel" if rot else "fan_bp_kernel"
        if want is None:                                 # fewer than four slices: one at a time, their views split
            assert [l[0] for l in launches] == [name, "combine_parts_kernel"] * n
            continue
        assert [(l[0], l[1][0], l[2]) for l in launches] == [(name, m, tiles * per) for m, per in want], (N, K, n)


def test_cases_lie_on_both_sides_of_the_rule():
    for N, K, n, want in CASES:
        if n < 4:
            continue
        tiles = (((N + 1) // 2 + 15) // 16) * ((N // 2 + 15) // 16) if K % 4 == 0 else ((N + 15) // 16) ** 2
        g = tiles * ((n + 3) // 4) / CUS
        assert want[0][0] == (1 if g < 1.0 else 2 if g < 3.0 else 4), (N, K, n, g)
