"""Angle images and angle errors at their edges, against numpy in 64 bits:
sizes around the kernels' four pixels per thread, unaligned maps, axis and zero
vectors with either sign of zero, opposite and nearly equal vectors, infinities
and NaN."""
import numpy as np
import pytest

import paper_2209_08241_amd as bn

pytestmark = pytest.mark.gpu

ZEROS = [(x, y, z) for x in (0.0, -0.0) for y in (0.0, -0.0) for z in (0.0, -0.0, 1.0, -1.0)]
VECTORS = ZEROS + [(1, 0.0, 0), (1, -0.0, 0), (-1, 0.0, 0), (-1, -0.0, 0), (0.0, 1, 0), (-0.0, 1, 0),
                   (0.0, -1, 0), (-0.0, -1, 0), (0.6, 0.8, 0.1), (0.6, -0.8, 0.1), (-0.6, -0.8, -0.1),
                   (1, 1, 1), (-1, 1, -1), (1e-42, -1e-42, 1), (1, -1e-42, 0), (3e38, 3e38, -3e38),
                   (0.41421357, 1, 0.2), (1, 0.41421354, -2), (1e-30, 1e30, 1)]
ODD = [(np.inf, 1, 0), (-np.inf, -np.inf, 2), (0, np.inf, np.inf), (np.nan, 1, 1), (1, 1, np.nan)]


def angles(n):
    n = np.asarray(n, np.float32).astype(np.float64)
    phi = np.arctan2(n[..., 1], n[..., 0])
    phi = np.where(phi < 0, phi + 2 * np.pi, phi)
    return np.arctan2(np.hypot(n[..., 0], n[..., 1]), n[..., 2]), phi


def cuda(a, offset=0):
    import torch
    a = np.ascontiguousarray(a)
    flat = torch.empty(a.size + offset, dtype=torch.from_numpy(a).dtype, device="cuda")[offset:]
    flat.copy_(torch.from_numpy(a).reshape(-1))
    return flat.view(a.shape)


def test_angle_images_of_special_vectors():
    n = np.array(VECTORS + ODD, np.float32)[None]
    t, p = bn.normal_angles(cuda(n))
    for got, want in zip((t, p), angles(n)):
        # one rounding to binary32
        np.testing.assert_allclose(got.cpu().numpy(), want.astype(np.float32), rtol=1.2e-7,
                                   atol=0, equal_nan=True)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 255, 1023, 1024, 1025, 4099])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_sizes_and_alignments(n, offset):
    rng = np.random.default_rng(n)
    a = rng.normal(size=(1, n, 3)).astype(np.float32)
    b = (a + rng.normal(scale=0.1, size=a.shape)).astype(np.float32)
    ma = rng.integers(0, 2, size=(1, n)).astype(np.uint8)
    ma[0, -1] = 0
    t, p = bn.normal_angles(cuda(a, offset))
    (ta, pa), (tb, pb) = angles(a), angles(b)
    np.testing.assert_allclose(t.cpu().numpy(), ta, rtol=1.2e-7)
    np.testing.assert_allclose(p.cpu().numpy(), pa, rtol=1.2e-7)
    got = bn.angle_mse(cuda(a, offset), cuda(ma, offset), cuda(b, offset))
    use = ma == 0
    assert got[2] == use.sum()
    # each difference to a few 2^-53 of pi
    np.testing.assert_allclose(got[0], np.mean((ta - tb)[use] ** 2), rtol=1e-13, atol=1e-16)
    np.testing.assert_allclose(got[1], np.mean((pa - pb)[use] ** 2), rtol=1e-13, atol=1e-16)


def test_errors_of_every_pair_of_special_vectors():
    v = np.array(VECTORS + ODD, np.float32)
    for k, a in enumerate(v):
        n = np.repeat(a[None, None], len(v), axis=1)
        m = v[None]
        (ta, pa), (tb, pb) = angles(n), angles(m)
        na, nm = cuda(n), cuda(m)
        for j in range(len(v)):
            mask = np.ones((1, len(v)), np.uint8)
            mask[0, j] = 0
            got = bn.angle_mse(na, cuda(mask), nm)
            for g, d in ((got[0], (ta - tb)[0, j]), (got[1], (pa - pb)[0, j])):
                np.testing.assert_allclose(np.sqrt(g), abs(d), rtol=1e-14, atol=1e-14,
                                           equal_nan=True, err_msg=f"{a} {v[j]}")
