"""Flat tiles at the edges of frames and tiles in launches large enough to take
them, bit for bit against the scalar tiles."""
import numpy as np
import pytest

import paper_2209_08241_amd as bn
from test_gpu_flat_tiles import METHODS, depths

pytestmark = pytest.mark.gpu


N = 64
# above six scales a stack's line is higher than these sizes
STACKS = [m for m in METHODS if m[2] <= 6] + [("multiscale", 8, 6)]


def stacks_agree(method, alpha, K, H, W, shift, pad):
    """64 frames, more than 2^19 pixels together, with padded rows, in flat tiles
    and in scalar ones; the depth, the normals (in pixels) and the codes start
    `shift` elements into larger buffers (alike in groups of four pixels, as
    flat tiles ask), whose surroundings stay as they were."""
    import torch
    assert N * H * W > 1 << 19 and (shift[1] - shift[2]) % 4 == 0
    one = np.stack([depths(H, W, H + k) for k in range(2)])
    wide = torch.full((N * H * (W + pad) + 8,), 3.25, device="cuda")
    d = wide[shift[0]:shift[0] + N * H * (W + pad)].view(N, H, W + pad)[:, :, :W]
    for k in range(N):   # frames differ: rolled rows
        d[k] = torch.from_numpy(np.ascontiguousarray(np.roll(one[k % 2], k, axis=0))).cuda()
    out = []
    for variant in (0, 1):
        nb = torch.full((3 * N * H * W + 128,), 7.0, device="cuda")
        mb = torch.full((N * H * W + 64,), 99, dtype=torch.uint8, device="cuda")
        n0 = 3 * shift[1]
        n = nb[n0:n0 + 3 * N * H * W].view(N, H, W, 3)
        m = mb[shift[2]:shift[2] + N * H * W].view(N, H, W)
        _, _, st = bn.estimate_normals_stack(d, (90.0, 92.0, (W - 1) / 2, (H - 1) / 2), alpha,
                                             method=method, scales=K, variant=variant, normals=n,
                                             mask=m)
        assert bool((torch.cat([nb[:n0], nb[n0 + 3 * N * H * W:]]) == 7.0).all())
        assert bool((torch.cat([mb[:shift[2]], mb[shift[2] + N * H * W:]]) == 99).all())
        out.append((n, m, st))
    for x, y in zip(*out):
        assert torch.equal(x.reshape(-1).view(torch.uint8), y.reshape(-1).view(torch.uint8))


@pytest.mark.parametrize("method,alpha,K", STACKS)
@pytest.mark.parametrize("H,W,shift", [(2053, 4, (1, 0, 0)), (1641, 5, (3, 1, 1)), (1367, 6, (0, 9, 1)),
                                       (1181, 7, (2, 4, 0)), (911, 9, (1, 3, 3)), (65, 131, (0, 2, 6)),
                                       (33, 257, (3, 2, 2)), (17, 511, (0, 1, 5)), (9, 1030, (1, 0, 4)),
                                       (2, 4111, (0, 7, 3)), (1, 8203, (2, 0, 4)), (40, 255, (1, 5, 1))])
def test_stacks_equal_scalar_tiles(method, alpha, K, H, W, shift):
    stacks_agree(method, alpha, K, H, W, shift, W % 4)


@pytest.mark.parametrize("W", [254, 255, 256, 259])
@pytest.mark.parametrize("n,m", [(0, 0), (0, 4), (1, 1), (1, 5), (2, 6), (4, 0), (7, 3), (9, 1),
                                 (31, 3)])
def test_output_alignments(W, n, m):
    stacks_agree("four_pair", 2, 0, 33, W, (n % 4, n, m), 1)


@pytest.mark.parametrize("method,alpha,K", METHODS)
@pytest.mark.parametrize("n", [9, 30])
def test_lists_of_small_frames_beside_a_large_one(method, alpha, K, n):
    """A list of more than 2^21 pixels: its small frames of any layout take flat
    tiles (and scalar ones where the codes start elsewhere in a word than the
    normals), as single frames give them."""
    import torch
    big = torch.from_numpy(depths(1032, 2064, 3)).cuda()
    frames = [bn.BatchFrame(big, 90.0, 92.0, 1000.0, 500.0)]
    shapes = [(1, 4), (7, 5), (33, 75), (3, 257), (61, 131), (2, 1030), (19, 9), (40, 255)]
    for k in range(n):
        H, W = shapes[k % 8]
        d = torch.from_numpy(depths(H, W, k)).cuda()
        out = torch.full((3 * H * W + 32,), 7.0, device="cuda")
        m = torch.full((H * W + 32,), 99, dtype=torch.uint8, device="cuda")
        at = k % 7
        frames.append(bn.BatchFrame(d, 90.0, 92.0, W / 2, H / 2,
                                    normals=out[3 * at:3 * at + 3 * H * W].view(H, W, 3),
                                    mask=m[at + k // 8:at + k // 8 + H * W].view(H, W)))
        frames[-1].buffers = (out, 3 * at, 7.0), (m, at + k // 8, 99)
    with bn.BatchPlan(frames, alpha, method=method, scales=K) as plan:
        plan.run()
        torch.cuda.synchronize()
    for f in frames[1:]:
        want = bn.estimate_normals(f.depth, 90.0, 92.0, f.cx, f.cy, alpha, method=method, scales=K,
                                   variant=1)
        for x, y in zip((f.normals, f.mask, f.stats), want):
            assert torch.equal(x.reshape(-1).view(torch.uint8), y.reshape(-1).view(torch.uint8))
        for (buf, at, v), x in zip(f.buffers, (f.normals, f.mask)):
            assert bool((buf[:at] == v).all()) and bool((buf[at + x.numel():] == v).all())
