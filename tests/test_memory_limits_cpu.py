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
