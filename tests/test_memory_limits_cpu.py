"""Calls for which device memory is short, on a HIP runtime of host memory (fake_hip.cpp):
buffers that only make a call faster are done without, and leave no error behind."""
import pytest

from fake_hip import run


@pytest.mark.parametrize("K,N,Nz,kernel,blocks", [
    (40, 33, 20, "cone_rot_kernel", 2 * 1 * 2 * 4),      # 2 x 1 base tiles, 2 blocks of 16 slices in fours
    (42, 33, 20, "cone_bp_kernel", 3 * 3 * 1 * 4),       # 3 x 3 tiles, one block of 32 slices in eights
])
def test_small_cone_volumes_without_partial_volumes(K, N, Nz, kernel, blocks):
    got = run(f"""
g = fbp.ConeGeometry({K}, 50, 40, {N}, {Nz}, 60.0)
part = 4 * {N} * {N} * {Nz}                  # the smallest set of partial volumes is two of these
fake.fake_fail_from(2 * part)
first = [call("fbp_cone_backproject", g, A, C), fake.hipPeekAtLastError(), launched()]
fake.fake_reset()
fake.fake_fail_from(1 << 62)
again = [call("fbp_cone_backproject", g, A, C), fake.hipPeekAtLastError(), launched()]
result = [first, again]
""")
    for status, error, launches in got:
        assert status == 0 and error == 0
        assert launches[0][0] == kernel and launches[0][2] == blocks
        assert not any(l[0].startswith("combine") for l in launches)


def test_an_earlier_error_of_the_caller_is_kept():
    got = run("""
g = fbp.ConeGeometry(40, 50, 40, 33, 20, 60.0)
p = ctypes.c_void_p()
fake.fake_fail_from(2 * 4 * 33 * 33 * 20)
assert fake.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 40)) == 2
result = [call("fbp_cone_backproject", g, A, C), fake.hipPeekAtLastError()]
""")
    assert got == [0, 2]


@pytest.mark.parametrize("K,D,N,R", [(360, 300, 200, 500.0), (721, 901, 512, 1024.0), (90, 6200, 4096, 12000.0)])
def test_fan_projector_takes_what_it_took_before_it_was_staged(K, D, N, R):
    """The one-lane kernel's copies took up to 16 slices of `copies` bytes (at most 256 MiB);
    where that much is free the call goes through, and with more it is staged."""
    pad = 2                                          # at least: two zeros on both sides of a line
    copies = 4 * 2 * (N + 1) * (N + 2 * pad)
    before = copies * max(1, min(16, (256 << 20) // copies))
    got = run(f"""
g = fbp.Geometry({K}, {D}, {N}, 1.0, source_distance={R})
result = []
fake.fake_fail_from({before} + {before} // 4)        # the copies' true padding included
result.append([call("fbp_project", g, 1, A, C), fake.hipPeekAtLastError(), [l[0] for l in launched()]])
g = fbp.Geometry({K}, {D}, {N}, 1.0, g.angles + 2.0 ** -12, source_distance={R})
fake.fake_reset()
fake.fake_fail_from(1 << 62)
result.append([call("fbp_project", g, 1, A, C), fake.hipPeekAtLastError(), [l[0] for l in launched()]])
""")
    assert [g[:2] for g in got] == [[0, 0], [0, 0]]
    assert got[1][2] == ["turn_kernel", "fan_staged_kernel"]
    assert got[0][2] in (["turn_kernel", "fan_staged_kernel"], ["pad_kernel", "fan_project_kernel"])
