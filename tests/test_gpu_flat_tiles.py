"""Flat tiles (frames whose layout or reach rules the vector tiles out) against
the oracle and, bit for bit, against the scalar tiles: odd widths, frames that
end anywhere in a tile, padded rows, output alignments, special depths, every
method and reach."""
import numpy as np
import pytest

import oracle
import paper_2209_08241_amd as bn
from gpu_util import assert_parity
from synth import scenes

pytestmark = pytest.mark.gpu

METHODS = [("four_pair", 1, 0), ("four_pair", 2, 0), ("four_pair", 8, 0), ("pair_removal", 2, 0),
           ("pair_removal", 5, 0), ("multiscale", 1, 1), ("multiscale", 3, 3), ("multiscale", 2, 5),
           ("multiscale", 8, 8)]


def run(depth, method, alpha, K, mode="rel", tau=4.0, variant=0, row_pad=0, shift=(0, 0, 0), f=90.0):
    """A stack of the frame and its mirror images (stacks take flat tiles at any
    size, and their later frames' outputs start anywhere), with the depth, the
    normals and the mask `shift` elements into larger buffers, whose
    surroundings must stay as they were."""
    import torch
    H, W = depth.shape
    host = np.stack([depth, depth[:, ::-1], depth[::-1]])
    N = len(host)
    wide = torch.full((N * H * (W + row_pad) + 64,), 3.25, device="cuda")
    d = wide[shift[0]:shift[0] + N * H * (W + row_pad)].view(N, H, W + row_pad)[:, :, :W]
    d.copy_(torch.from_numpy(np.ascontiguousarray(host)))
    nb = torch.full((3 * N * H * W + 64,), 7.0, device="cuda")
    mb = torch.full((N * H * W + 64,), 99, dtype=torch.uint8, device="cuda")
    n = nb[shift[1]:shift[1] + 3 * N * H * W].view(N, H, W, 3)
    m = mb[shift[2]:shift[2] + N * H * W].view(N, H, W)
    _, _, st = bn.estimate_normals_stack(d, (f, f + 2, (W - 1) / 2, (H - 1) / 2), alpha, mode, tau,
                                         method=method, scales=K, variant=variant, normals=n,
                                         mask=m)
    torch.cuda.synchronize()
    outside = torch.cat([nb[:shift[1]], nb[shift[1] + 3 * N * H * W:]])
    assert bool((outside == 7.0).all())
    outside = torch.cat([mb[:shift[2]], mb[shift[2] + N * H * W:]])
    assert bool((outside == 99).all())
    return host, n.cpu().numpy(), m.cpu().numpy(), st.cpu().numpy()


def depths(H, W, seed):
    s = scenes.make_scene(H, W, fx=90.0, fy=92.0, cx=(W - 1) / 2, cy=(H - 1) / 2, seed=seed)
    d = s.depth.copy()
    rng = np.random.default_rng(seed)
    for v in (np.nan, np.inf, -1.0, 1e-42, 1e30):
        d[rng.integers(0, H, 3), rng.integers(0, W, 3)] = v
    return d


@pytest.mark.parametrize("method,alpha,K", METHODS)
@pytest.mark.parametrize("H,W", [(1, 4), (1, 1023), (2, 5), (7, 6), (33, 7), (19, 9), (3, 257),
                                 (19, 131), (17, 253), (23, 511), (140, 767), (9, 1030),
                                 (70, 75)])
def test_flat_equal_scalar_tiles(method, alpha, K, H, W):
    d = depths(H, W, H + W + alpha)
    kw = dict(method=method, alpha=alpha, K=K, row_pad=W % 5, shift=(1 + W % 3, 3 * (H % 9), H % 9))
    a = run(d, variant=0, **kw)
    b = run(d, variant=1, **kw)
    for x, y in zip(a[1:], b[1:]):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8))


@pytest.mark.parametrize("shift", [(s, n, m) for s in (0, 3) for n in (0, 1, 4, 9) for m in (0, 2, 3, 7)])
@pytest.mark.parametrize("W", [254, 255, 256, 259])
@pytest.mark.parametrize("method", ["four_pair", "pair_removal"])
def test_output_alignments(W, shift, method):
    d = depths(11, W, W)
    a = run(d, method, 2, 0, shift=shift)
    b = run(d, method, 2, 0, shift=shift, variant=1)
    for x, y in zip(a[1:], b[1:]):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8))


@pytest.mark.parametrize("method,alpha,K", METHODS)
@pytest.mark.parametrize("mode,tau", [("rel", 4.0), ("abs", 2e-3), ("none", 1.0)])
def test_flat_against_the_oracle(method, alpha, K, mode, tau):
    H, W = 137, 389
    s = scenes.make_scene(H, W, fx=90.0, fy=92.0, cx=(W - 1) / 2, cy=(H - 1) / 2, seed=alpha + K)
    host, n, m, st = run(s.depth, method, alpha, K, mode, tau, shift=(1, 6, 2))
    for k, d in enumerate(host):
        ref = oracle.variant_f32(d, 90.0, 92.0, (W - 1) / 2, (H - 1) / 2, alpha, mode, tau,
                                 method=method, scales=K)
        assert_parity(ref, n[k], m[k], st[k], what=f"{method} {alpha} {K} {mode} frame {k}")


@pytest.mark.parametrize("method,alpha,K,W", [("four_pair", 2, 0, 1103), ("pair_removal", 1, 0, 1105),
                                              ("multiscale", 2, 3, 1102), ("multiscale", 5, 4, 1104)])
def test_single_frames_above_the_scalar_tiles_sizes(method, alpha, K, W):
    import torch
    d = torch.from_numpy(depths(1021, W, alpha)).cuda()
    a = bn.estimate_normals(d, 90.0, 92.0, 550.0, 510.0, alpha, method=method, scales=K)
    b = bn.estimate_normals(d, 90.0, 92.0, 550.0, 510.0, alpha, method=method, scales=K, variant=1)
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


@pytest.mark.parametrize("method,alpha,K", [("four_pair", 1, 0), ("pair_removal", 2, 0),
                                            ("multiscale", 1, 3), ("multiscale", 4, 6)])
@pytest.mark.parametrize("n", [5, 20])
def test_lists_of_mixed_layouts(method, alpha, K, n):
    """Vector, flat and scalar tiles in one launch (the last: codes that start
    elsewhere in a word than the normals), as single frames give them."""
    import torch
    shapes = [(24, 64), (33, 75), (7, 3), (40, 130), (61, 257)]
    frames = []
    for k in range(n):
        H, W = shapes[k % 5]
        d = torch.from_numpy(depths(H, W, k)).cuda()
        m = torch.zeros(H * W + 3, dtype=torch.uint8, device="cuda")[k % 4:k % 4 + H * W].view(H, W)
        frames.append(bn.BatchFrame(d, 90.0, 92.0, W / 2, H / 2, mask=m))
    with bn.BatchPlan(frames, alpha, method=method, scales=K) as plan:
        plan.run()
        torch.cuda.synchronize()
    for f in frames:
        want = bn.estimate_normals(f.depth, 90.0, 92.0, f.cx, f.cy, alpha, method=method, scales=K,
                                   variant=1)
        for x, y in zip((f.normals, f.mask, f.stats), want):
            assert torch.equal(x.reshape(-1).view(torch.uint8), y.reshape(-1).view(torch.uint8))
