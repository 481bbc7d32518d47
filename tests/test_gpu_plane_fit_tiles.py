"""The plane-fit kernel at the edges of its wavefronts (64 - 2R output columns,
1 or 4 rows) against the evaluation oracle, on scenes with holes, special
values, and windows whose two smallest eigenvalues nearly agree."""
import numpy as np
import pytest

import paper_2209_08241_amd as bn
from oracle import evaluation as oev
from synth import scenes

pytestmark = pytest.mark.gpu


def check(depth, fx, fy, cx, cy, r, pixels=None, pad=0):
    import torch
    H, W = depth.shape
    wide = torch.full((H, W + pad), float("nan"), device="cuda")
    wide[:, :W] = torch.from_numpy(np.ascontiguousarray(depth)).cuda()
    n, m = bn.plane_fit_normals(wide[:, :W], fx, fy, cx, cy, r)
    torch.cuda.synchronize()
    n, m = n.cpu().numpy(), m.cpu().numpy()
    fx, fy, cx, cy = (float(np.float32(v)) for v in (fx, fy, cx, cy))  # as the kernel gets them
    rn, rm, eigs = oev.plane_fit(depth, fx, fy, cx, cy, r, pixels=pixels)
    at = np.ones((H, W), bool)
    if pixels is not None:
        at[:] = False
        at[tuple(np.array([(y, x) for x, y in pixels]).T)] = True
    assert np.array_equal(m[at], rm[at])
    assert not n[at & (m != 0)].any()
    sel = at & (rm == 0)
    e = eigs[sel]
    gap = np.maximum((e[:, 1] - e[:, 0]) / e[:, 2], 1e-300)
    # binary32 rounding of a component (6e-8), the sensitivity of the vector to
    # FP64 rounding of the matrix (a few hundred ulp over the gap), and of the
    # closed forms' eigenvalue (an ulp over the gap squared)
    tol = 1e-7 + 1e-13 / gap + 4e-16 / gap ** 2
    err = np.abs(n[sel].astype(np.float64) - rn[sel]).max(axis=-1)
    assert np.all(err <= tol), f"{err.max():.3g} at gap {gap[np.argmax(err - tol)]:.3g}"
    return int(sel.sum())


@pytest.mark.parametrize("H,W", [(1, 1), (2, 70), (3, 3), (5, 5), (7, 7), (7, 59), (9, 60),
                                 (6, 61), (8, 62), (9, 64), (13, 65), (7, 125), (37, 180)])
@pytest.mark.parametrize("r", [1, 2, 3])
def test_small_frames(H, W, r):
    s = scenes.make_scene(H, W, fx=60.0, fy=63.0, cx=W / 2.3, cy=H / 1.7, seed=H * W + r,
                          hole_p=0.01)
    check(s.depth, s.fx, s.fy, s.cx, s.cy, r, pad=W % 3)


@pytest.mark.parametrize("r", [1, 2, 3])
def test_four_row_wavefronts(r):
    H, W = 773, 1021   # above the size from which a wavefront takes four rows
    s = scenes.make_scene(H, W, fx=700.0, seed=90 + r, hole_p=0.005)
    xs = sorted({min(max(k * (64 - 2 * r) + d, 0), W - 1) for k in (0, 1, 2, 9, 16, 17, 18)
                 for d in (-3, -1, 0, 1, 2)})
    ys = sorted({min(max(y + d, 0), H - 1) for y in (0, 4, 16, 400, 768, 772) for d in (-2, -1, 0, 1)})
    assert check(s.depth, *s.intrinsics, r, pixels=[(x, y) for y in ys for x in xs], pad=3) >= 250


def test_special_values_and_outliers():
    d = scenes.make_scene(40, 130, fx=120.0, seed=7, hole_p=0).depth
    for k, v in enumerate([0.0, -1.0, np.nan, np.inf, -np.inf, -0.0, 1e-40]):
        d[5 + 4 * k, 10 + 16 * k] = v
    d[20, 100] = 1e12      # a valid depth far from the others of its wavefront
    # away from the two extreme depths the windows are ordinary ones
    pts = [(x, y) for y in range(40) for x in range(130)
           if max(abs(x - 100), abs(y - 20)) > 2 and max(abs(x - 106), abs(y - 29)) > 2]
    assert check(d, 120.0, 120.0, 64.5, 19.5, 2, pixels=pts) > 3000


def test_close_eigenvalues_across_a_step():
    # two fronto planes: along the step the window's spread in depth dwarfs its
    # extent in x and y, whose eigenvalues nearly agree
    H, W = 24, 140
    rng = np.random.default_rng(3)
    d = np.full((H, W), 2.0)
    d[:, W // 2:] = 3.9
    d = (d * (1 + 1e-6 * rng.standard_normal((H, W)))).astype(np.float32)
    check(d, 2000.0, 2000.0, 70.0, 12.0, 2)
