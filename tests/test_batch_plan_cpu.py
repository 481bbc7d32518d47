"""Host side of batch plans on a HIP runtime without a GPU: what a plan's calls
allocate, instantiate and launch."""
import os

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="HIP headers not available")


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return fake_hip.build(tmp_path_factory.mktemp("fakehip"))


def test_updates_within_a_plans_size_allocate_nothing(so):
    """A plan made of odd-sized frames holds the tiles of as many pixels in any
    layout: an update to such a list neither allocates nor waits."""
    fake_hip.run(so, r"""
h = create([(479, 637)] * 20)
log()
for shapes in ([(480, 640)] * 19, [(480, 636)] * 20, [(720, 1280)] * 20, [(479, 637)] * 20):
    assert update(h, shapes) == 0
    assert "alloc" not in log(), shapes
# normals and codes that start apart: scalar tiles
fr = frames([(479, 637)] * 20)
for f in fr:
    f.mask += 1
assert L.bn_batch_plan_update(h, fr, 20, None) == 0
assert "alloc" not in log()
""")


def test_a_failed_instantiation_is_tried_again(so):
    """A graph that could not be instantiated leaves nothing behind, and the
    next run makes it."""
    fake_hip.run(so, r"""
for odd in ((479, 637), (480, 640)):
    for small in (False, True):      # a table's graph, a small list's
        n = 3 if small else 20
        h = create([(480, 640)] * 20)
        shapes = [(480, 640)] * (n - 1) + [odd]
        if small:
            assert update(h, shapes) == 0
            fake.fake_fail_instantiate(1)
            assert L.bn_batch_run(h, None) != 0
        else:
            fake.fake_fail_instantiate(1)
            if update(h, shapes) == 0:
                L.bn_batch_run(h, None)
            fake.fake_fail_instantiate(0)
        log()
        assert L.bn_batch_run(h, None) == 0
        assert len(launches(log())) == (1 if small else 2)
        L.bn_batch_plan_destroy(h)
        assert fake.fake_graphs() == 0
""")


def test_a_run_instantiates_nothing(so):
    """The graph of another kind of list is made by the update that brings the
    list, once."""
    fake_hip.run(so, r"""
h = create([(480, 640)] * 20)
log()
made = 0
for odd in ((480, 640), (479, 637), (480, 640), (479, 637)):
    assert update(h, [(480, 640)] * 19 + [odd]) == 0
    made += log().count("instantiate")
    for _ in range(2):
        assert L.bn_batch_run(h, None) == 0
        lines = log()
        assert "instantiate" not in lines, odd
        name, grid = launches(lines)[0]
        assert ("Lb1E" in name) == (odd == (479, 637)), (name, odd)
assert made == 1
""")


def test_plan_info_reports_the_launch(so):
    """Workgroups are those of the launch, whatever tiles the frames take."""
    fake_hip.run(so, r"""
def info(h):
    px, tiles, wg = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int32()
    assert L.bn_batch_plan_info(h, ctypes.byref(px), ctypes.byref(tiles), ctypes.byref(wg)) == 0
    return px.value, tiles.value, wg.value

for shapes in ([(479, 637)] * 20, [(480, 640)] * 20, [(479, 637), (720, 1280)] * 12,
               [(1079, 1917)] * 3, [(480, 640)] * 16, [(0, 5), (479, 637)]):
    h = create(shapes)
    log()
    assert L.bn_batch_launch(h, None) == 0
    px, tiles, wg = info(h)
    assert px == sum(H * W for H, W in shapes)
    assert wg == launches(log())[0][1], shapes
    # the list's size: work items of four pixels in vector layouts, else of one
    assert tiles == sum((H * (W // 4 if W % 4 == 0 else W) + 255) // 256 for H, W in shapes)
""")


@pytest.mark.parametrize("H,W,kernel", [(1429, 2555, "k_flat"), (719, 1277, "k_scalar"),
                                        (1080, 1920, "k_vec4")])
def test_plain_autotuning_times_what_a_call_takes(so, H, W, kernel):
    """The kernels that the autotuner times are those that later calls with
    variant 0 choose among."""
    fake_hip.run(so, f"""
H, W, kernel = {H}, {W}, "{kernel}"
""" + r"""
L.bn_autotune_reset()
p = bn.make_params(2)
d, n, m = (1 << 30), (2 << 30), (3 << 30)
call = lambda: L.bn_estimate_normals(d, H, W, W, 500.0, 500.0, W / 2, H / 2, p, n, m, None, None)
assert call() == 0
(used, grid), = launches(log())
assert kernel in used
v, us = ctypes.c_int(), ctypes.c_float()
assert L.bn_autotune_plain(H, W, p, ctypes.byref(v), ctypes.byref(us)) == 0
timed = {name for name, _ in launches(log()) if "tune_scene" not in name and "zero" not in name}
assert used in timed and (W % 4 == 0 or len(timed) == 1), (used, timed)
assert call() == 0
assert launches(log())[0][0] in timed
""")


@pytest.mark.parametrize("method,scales,line", [("four_pair", 0, 1 << 18),
                                                ("pair_removal", 0, 3 << 17),
                                                ("multiscale", 6, 1 << 19),
                                                ("multiscale", 7, 1 << 20)])
def test_small_stacks_of_odd_frames_take_scalar_tiles(so, method, scales, line):
    """Up to `line` pixels in all (half as many again for a single frame)."""
    fake_hip.run(so, f"""
method, scales, line = "{method}", {scales}, {line}
""" + r"""
p = bn.make_params(2, method=method, scales=scales)
intr = (bn.Intrinsics * 64)(*[bn.Intrinsics(500.0, 500.0, 50.0, 50.0)] * 64)
d, n, m = (1 << 30), (2 << 30), (3 << 30)
for frames_, most in ((1, line * 3 // 2), (2, line), (64, line)):
    for W in (129, 255):
        H = most // (frames_ * W)       # the largest height up to the line
        for h, flat in ((H, False), (H + 1, True)):
            assert L.bn_estimate_normals_stack(d, frames_, h, W, W, h * W, intr, p, n, m, None,
                                               None) == 0
            (name, grid), = launches(log())
            assert ("k_stack_flat" in name) == flat, (frames_, h, W, name)
            if not flat:
                assert "k_stack" in name and grid == frames_ * ((h * W + 255) // 256)
""")


@pytest.mark.parametrize("method,scales,line", [("four_pair", 0, 1 << 19),
                                                ("pair_removal", 0, 3 << 18),
                                                ("multiscale", 6, 1 << 20),
                                                ("multiscale", 7, 1 << 21)])
def test_small_lists_of_odd_frames_take_scalar_tiles(so, method, scales, line):
    """Up to `line` pixels in the whole list: by a plan, for a small list and a
    table, and without one."""
    fake_hip.run(so, f"""
method, scales, line = "{method}", {scales}, {line}
""" + r"""
p = bn.make_params(2, method=method, scales=scales)
for n in (1, 3, 15, 16, 40):
    for W in (131, 255):
        H = line // (n * W)
        # a frame more of whole groups takes the list to the line, or over it
        rest = (line - n * H * W) // 4
        for extra, flat in ((rest, False), (rest + 1, True)):
            shapes = [(H, W)] * n + [(1, 4 * extra)]
            scalar = sum((h * w // (4 if w % 4 == 0 else 1) + 255) // 256 for h, w in shapes)
            h = create(shapes, p)
            log()
            assert L.bn_batch_launch(h, None) == 0
            (name, grid) = launches(log())[0]
            assert (grid < scalar) == flat, (shapes[0], n, extra, grid, scalar)
            if len(shapes) > 16:
                assert ("Lb1E" in name) == flat
            else:
                assert L.bn_estimate_normals_batch_noalloc(frames(shapes), len(shapes), p, None) == 0
                assert launches(log())[1] == (name, grid)
            L.bn_batch_plan_destroy(h)
""")
