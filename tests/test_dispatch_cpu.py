"""Which kernels calls of few pixels take, on a HIP runtime without a GPU."""
import os

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="HIP headers not available")


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fakehip"))


@pytest.mark.parametrize("alpha,one,stack", [(1, 1 << 20, 1 << 20), (2, 9 << 16, 7 << 16),
                                             (3, 3 << 18, 3 << 18), (4, 7 << 17, 7 << 17)])
def test_small_adjoints_of_odd_rows_take_scalar_tiles(so, alpha, one, stack):
    """Up to `one` pixels in a frame, `stack` in a stack; rows of whole aligned
    groups keep their own line."""
    fake_hip.run(so, f"""
alpha, one, stack = {alpha}, {one}, {stack}
""" + r"""
p = bn.make_params(alpha)
intr = (bn.Intrinsics * 64)(*[bn.Intrinsics(500.0, 500.0, 50.0, 50.0)] * 64)
d, g, o = (1 << 30), (2 << 30), (3 << 30)
aligned = (3 << 17) if alpha <= 2 else (3 << 18)
for n in (0, 1, 2, 64):              # 0: the single-frame call
    for W in (129, 255, 256):
        most = aligned if W % 4 == 0 else one if n <= 1 else stack
        H = most // (max(n, 1) * W)  # the largest height up to the line
        for h, vec in ((H, False), (H + 1, True)):
            if n == 0:
                rc = L.bn_normals_vjp(d, h, W, W, 500.0, 500.0, 50.0, 50.0, p, g, o, None)
            else:
                rc = L.bn_normals_vjp_stack(d, n, h, W, W, h * W, intr, p, g, o, None)
            assert rc == 0
            (name, grid), = launches(log())
            assert ("k_vjp4" in name) == vec, (n, W, h, name)
""")


def test_few_partial_sums_of_the_angle_error_take_a_small_workgroup(so):
    fake_hip.run(so, r"""
a, b, ws, out = (1 << 30), (2 << 30), (3 << 30), (4 << 30)
for px, threads in ((1, 256), (1024 * 256, 256), (1024 * 256 + 1, 1024), (1 << 22, 1024)):
    assert L.bn_angle_mse(a, None, b, None, 1, px, ws, out, None) == 0
    names = [n for n, _ in launches(log())]
    assert "k_mse_partial" in names[0] and f"k_mse_finalILi{threads}E" in names[1], names
""")
