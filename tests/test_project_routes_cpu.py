"""Which projector kernel a geometry takes, on a HIP runtime of host memory (fake_hip.cpp)."""
import json

from fake_hip import run
from test_gpu_project_taps import CASES, angles


def test_every_case_takes_the_kernel_it_names():
    plain = [[K, D, N, dt, list(angles(K, kind)), weighting] for K, D, N, dt, kind, weighting, *_ in CASES]
    got = run(f"""
result = []
for K, D, N, dt, ang, weighting in json.loads({json.dumps(json.dumps(plain))}):
    g = fbp.Geometry(K, D, N, dt, np.array(ang), weighting=weighting)
    fake.fake_reset()
    assert call("fbp_project", g, 1, A, C) == 0
    result.append(launched()[-1])
""")
    for case, (kernel, values, blocks) in zip(CASES, got):
        assert kernel == case[6] and values[:len(case[7])] == case[7], (case, kernel, values)


def test_every_staged_form_is_among_the_cases():
    """M = 4 with two to four taps, M = 2 with two and three, each three-tap form twice."""
    forms = {tuple(c[7]) for c in CASES if c[6] == "project_staged_kernel"}
    assert forms == {(4, 2, 0), (4, 3, 0), (4, 3, 1), (4, 4, 0), (2, 2, 0), (2, 3, 0), (2, 3, 1)}


def test_laying_out_a_large_fan_projector_is_quick():
    """The first call of a geometry checks every staged window on the host: CPU time of the
    order of the one-lane kernel's own layout, which walks every view and line (here of bins too
    coarse to be staged).  Looked through one by one, the chunks that miss the
    image would take fifteen times that."""
    staged, lane = run("""
import time
result = []
for dt, kernel in ((1.0, "fan_staged_kernel"), (4.0, "fan_project_kernel")):
    times = []
    for i in range(3):
        g = fbp.Geometry(1441, int(1700 / dt), 1024, dt, np.arange(1441) * (2.0 * math.pi / 1441) + 0.001 * i, source_distance=2500.0)
        fake.fake_reset()
        t = time.thread_time()
        assert call("fbp_project", g, 1, A, C) == 0
        times.append(time.thread_time() - t)
        assert launched()[-1][0] == kernel
    result.append(min(times))
""")
    assert staged <= 10.0 * lane, (staged, lane)
