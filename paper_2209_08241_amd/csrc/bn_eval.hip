// Evaluation tools of Section 4 on the GPU: the spherical angle images of a
// normal map (Eqs. 14-15), their mean squared error between two maps over
// the pixels valid in both, and the local plane-fit normals that the paper
// uses as ground truth on real depth maps (25 neighbours: a 5x5 window).
//
// These are off the estimator's hot path and run in FP64 (on this GPU's
// vector units as fast as unpacked binary32), storing binary32 results.
#include <cmath>

#include "bn_internal.h"
#include "bn_tiles.h"
#include "bnormals.h"

namespace bn {

namespace {

constexpr uint32_t kMseBlocks = BN_MSE_WORKSPACE_DOUBLES / 3;  // partial sums per launch
constexpr double kPi = 3.1415926535897932384626433832795;
constexpr double kTwoPi = 6.283185307179586476925286766559;

struct Angles {
    double theta, phi;
};

// atan2(y, x) of finite arguments, within a few units of 2^-53 of the angle's
// range.  t = min / max of the magnitudes, or (min - max) / (min + max) with
// pi/4 added above tan(pi/8), so |t| <= tan(pi/8); atan(t) = t + t u Q(u), u =
// t^2, where 1 + u Q(u) interpolates atan(sqrt u) / sqrt u at the 11 Chebyshev
// nodes of [0, tan^2(pi/8)] (error 4e-17); then the octant.  Signed zeros as
// atan2 has them.  (One quotient and 10 polynomial steps, no branches.)
__device__ __forceinline__ double atan2_finite(double y, double x) {
    constexpr double kQ[10] = {
        -0x1.55555555551e4p-2,
        0x1.9999999934e46p-3,
        -0x1.24924900951a7p-3,
        0x1.c71c648aada59p-4,
        -0x1.745baa25fcbc9p-4,
        0x1.3afb01a2783e6p-4,
        -0x1.0ffbe59bee9f9p-4,
        0x1.d1fd50510a91ap-5,
        -0x1.64313e6c61e43p-5,
        0x1.5a4830043ba61p-6,
    };
    const double ay = __builtin_fabs(y), ax = __builtin_fabs(x);
    const bool steep = ay > ax, left = __builtin_signbit(x);
    const double mx = __builtin_fmax(ay, ax), mn = __builtin_fmin(ay, ax);
    // a 0 or 1 in FP64 is one select (of the high word), a selected value two
    const double big = mn > 0.41421356237309503 * mx ? 1.0 : 0.0;
    const double num = __builtin_fma(-big, mx, mn);
    const double den = __builtin_fmax(__builtin_fma(big, mn, mx), 1e-300);  // (the zero vector)
    double r = __builtin_amdgcn_rcp(den);
    r = __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
    double t = num * r;
    t = __builtin_fma(r, __builtin_fma(-t, den, num), t);
    const double u = t * t;
    double q = kQ[9];
#pragma unroll
    for (int k = 8; k >= 0; --k) q = __builtin_fma(q, u, kQ[k]);
    double a = __builtin_fma(t * u, q, t);
    a = __builtin_fma(big, 0.25 * kPi, a);
    // a, pi/2 - a, pi - a or pi/2 + a
    a = steep != left ? -a : a;
    a += steep ? 0.5 * kPi : (left ? kPi : 0.0);
    return __builtin_copysign(a, y);
}

// 1 / sqrt(v) for a positive v: the hardware estimate (good to about binary32)
// refined STEPS times, each step squaring its relative error (two: about 1
// ulp); every product stays near 1 whatever v's scale.
template <int STEPS>
__device__ __forceinline__ double rsqrt_d(double v) {
    double y = __builtin_amdgcn_rsq(v);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        const double e = __builtin_fma(-(v * y), y, 1.0);
        y = __builtin_fma(0.5 * y, e, y);
    }
    return y;
}

// |(x, y)| (the square root by Goldschmidt's steps on the hardware's estimate).
__device__ __forceinline__ double length2(double x, double y) {
    const double v = __builtin_fma(x, x, y * y);
    const double e0 = __builtin_amdgcn_rsq(v);
    double g = v * e0, h = 0.5 * e0;
    const double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    g = __builtin_fma(__builtin_fma(-g, g, v), h, g);
    return v > 0.0 ? g : 0.0;
}

__device__ __forceinline__ bool finite3(float x, float y, float z) {
    return __builtin_fabsf(x) + __builtin_fabsf(y) + __builtin_fabsf(z) < INFINITY;
}

// I_phi = atan2(ny, nx) taken into [0, 2 pi); I_theta = atan2(|(nx, ny)|, nz).
__device__ __forceinline__ Angles angles_finite(double x, double y, double r, double z) {
    Angles a;
    a.phi = atan2_finite(y, x);
    if (a.phi < 0.0) a.phi += kTwoPi;
    a.theta = atan2_finite(r, z);
    return a;
}

// v's part in a direction that holds an infinity: its sign where it is
// infinite, a zero of its sign otherwise.
__device__ __forceinline__ double at_infinity(float v) {
    return __builtin_copysign(__builtin_isinf(v) ? 1.0 : 0.0, (double)v);
}

__device__ __forceinline__ Angles angles_of(float x, float y, float z) {
    if (finite3(x, y, z)) return angles_finite(x, y, length2(x, y), z);
    const bool far = __builtin_isinf(x) | __builtin_isinf(y), up = __builtin_isinf(z);
    const bool bad = __builtin_isnan(x) | __builtin_isnan(y);
    Angles a = angles_finite(far ? at_infinity(x) : (double)x, far ? at_infinity(y) : (double)y,
                             far ? 1.0 : up ? 0.0 : length2(x, y),
                             far | up ? at_infinity(z) : (double)z);
    const double nan = __builtin_nan("");
    if (bad) a.phi = nan;
    if (bad | (bool)__builtin_isnan(z)) a.theta = nan;
    return a;
}

// One pixel per thread: FP64 arithmetic and traffic (12 bytes in, 8 out per
// pixel) about balance, and overlap best with many wavefronts in turn (four
// pixels per thread, with 16-byte loads and stores, 13.9 against 12.5 us).
// 1920x1080 14.4 -> 10.4 us, 640x480 4.05 -> 3.5 (with the library's atan2 and
// plain stores before).
__global__ __launch_bounds__(256) void k_angles(const float *__restrict__ normals, uint32_t npix,
                                                float *__restrict__ theta,
                                                float *__restrict__ phi) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= npix) return;
    const float *n = normals + 3 * (int64_t)i;
    const Angles a = angles_of(n[0], n[1], n[2]);
    const uint32_t i0 = blockIdx.x * 256u;  // streaming stores (out_store)
    const uint32_t bytes = 4u * min(256u, npix - i0);
    out_store((float)a.theta, out_buf(theta + i0, bytes), 4u * threadIdx.x);
    out_store((float)a.phi, out_buf(phi + i0, bytes), 4u * threadIdx.x);
}

// Block sum of three doubles, deterministic for a fixed block size: lane
// shuffles, then the wavefronts' totals in order.  Result in thread 0.
template <int TB>
__device__ __forceinline__ void block_sum3(double &a, double &b, double &c) {
    __shared__ double s[TB / 64][3];
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
        c += __shfl_xor(c, off);
    }
    const uint32_t w = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) {
        s[w][0] = a;
        s[w][1] = b;
        s[w][2] = c;
    }
    __syncthreads();
    // lane j sums the wavefronts' totals of quantity j
    if (threadIdx.x < 64u) {
        const uint32_t j = min(threadIdx.x, 2u);
        double v = s[0][j];
#pragma unroll
        for (int k = 1; k < TB / 64; ++k) v += s[k][j];
        a = __shfl(v, 0);
        b = __shfl(v, 1);
        c = __shfl(v, 2);
    }
}

// theta_a - theta_b and phi_a - phi_b of two vectors, each difference as one
// arc tangent (of the sine and cosine of the difference) instead of two.
// theta's difference lies in [-pi, pi], where atan2 has it.  phi's lies in
// (-2 pi, 2 pi): with each phi in [0, pi] (upper half) or (pi, 2 pi) (lower),
// two of the same half differ by atan2's value; a in the lower half and b in
// the upper differ by a value in (0, 2 pi), the other way in (-2 pi, 0).
// A vector on the axis (x = y = 0) has phi 0 or pi by the sign of x, the zero
// vector theta 0 or pi by that of z, as atan2 of zeros has them.
struct AngleDiff {
    double theta, phi;
};

__device__ __forceinline__ AngleDiff angle_diff(float ax, float ay, float az, float bx, float by,
                                                float bz) {
    AngleDiff d;
    if (!(finite3(ax, ay, az) && finite3(bx, by, bz))) {
        const Angles x = angles_of(ax, ay, az), y = angles_of(bx, by, bz);
        d.theta = x.theta - y.theta;
        d.phi = x.phi - y.phi;
        return d;
    }
    const double ra = length2(ax, ay), rb = length2(bx, by);
    const bool axis_a = (ax == 0.0f) & (ay == 0.0f), axis_b = (bx == 0.0f) & (by == 0.0f);
    const double za = axis_a & (az == 0.0f) ? (double)__builtin_copysignf(1.0f, az) : (double)az;
    const double zb = axis_b & (bz == 0.0f) ? (double)__builtin_copysignf(1.0f, bz) : (double)bz;
    // two rounded products: exactly 0 for equal vectors (lengths are inexact, so
    // a fused one would leave the other's rounding)
    d.theta = atan2_finite(ra * zb - rb * za, __builtin_fma(za, zb, ra * rb));
    const double xa = axis_a ? (double)__builtin_copysignf(1.0f, ax) : (double)ax;
    const double xb = axis_b ? (double)__builtin_copysignf(1.0f, bx) : (double)bx;
    const double ya = ay, yb = by;
    // the products are exact, so the sine's sign is too
    double p = atan2_finite(__builtin_fma(xb, ya, -(xa * yb)), __builtin_fma(xa, xb, ya * yb));
    const bool la = ay < 0.0f, lb = by < 0.0f;
    if (la & !lb & (p < 0.0)) p += kTwoPi;
    if (lb & !la & (p > 0.0)) p -= kTwoPi;
    d.phi = p;
    return d;
}

// Partial sums of (dtheta^2, dphi^2, count) over a grid-stride share of the
// pixels, one triple per workgroup (in three planes of kMseBlocks).  A null
// mask counts as all VALID.  1920x1080, both
// kernels: 30.6 us with four arc tangents of the library per pixel, now 21.7.
__global__ __launch_bounds__(256) void k_mse_partial(const float *__restrict__ na,
                                                     const uint8_t *__restrict__ ma,
                                                     const float *__restrict__ nb,
                                                     const uint8_t *__restrict__ mb,
                                                     uint32_t npix, double *__restrict__ part) {
    double st = 0.0, sp = 0.0, k = 0.0;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < npix; i += gridDim.x * 256u) {
        const bool in = (!ma || ma[i] == BN_VALID) && (!mb || mb[i] == BN_VALID);
        const float *a = na + 3 * (int64_t)i, *b = nb + 3 * (int64_t)i;
        const AngleDiff d = angle_diff(a[0], a[1], a[2], b[0], b[1], b[2]);
        st += in ? d.theta * d.theta : 0.0;
        sp += in ? d.phi * d.phi : 0.0;
        k += in ? 1.0 : 0.0;
    }
    block_sum3<256>(st, sp, k);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = st;
        part[kMseBlocks + blockIdx.x] = sp;
        part[2 * kMseBlocks + blockIdx.x] = k;
    }
}

// One workgroup: the partials in a fixed order, then the means.  TB threads: 256
// for up to kMseFew partials, 1024 above (16 partials 2.0 / 3.0 us, 312 2.0 /
// 2.8, 1200 3.0 / 3.3, 2048 4.6 / 3.8).
constexpr uint32_t kMseFew = 1024;

template <int TB>
__global__ __launch_bounds__(TB) void k_mse_final(const double *__restrict__ part,
                                                  uint32_t nparts, double *__restrict__ out) {
    double st = 0.0, sp = 0.0, k = 0.0;
#pragma unroll 2
    for (uint32_t j = threadIdx.x; j < nparts; j += TB) {
        st += part[j];
        sp += part[kMseBlocks + j];
        k += part[2 * kMseBlocks + j];
    }
    block_sum3<TB>(st, sp, k);
    if (threadIdx.x == 0) {
        out[0] = k > 0.0 ? st / k : 0.0;
        out[1] = k > 0.0 ? sp / k : 0.0;
        out[2] = k;
    }
}

// The null vector of B - mu I, unit length, for B = [b0 a1 a2; a1 b3 a4;
// a2 a4 b5] and mu near an eigenvalue: the adjugate of B - mu I is then a
// multiple of the vector's outer product with itself, so the column of its
// largest diagonal entry is the longest.  Returns that column's squared
// length (0, infinite or NaN: no vector).
__device__ __forceinline__ double adjugate_vec(const double a[6], double b0, double b3, double b5,
                                               double mu, double n[3]) {
    const double e0 = b0 - mu, e3 = b3 - mu, e5 = b5 - mu;
    const double m00 = __builtin_fma(e3, e5, -(a[4] * a[4]));
    const double m11 = __builtin_fma(e0, e5, -(a[2] * a[2]));
    const double m22 = __builtin_fma(e0, e3, -(a[1] * a[1]));
    const double m01 = __builtin_fma(a[2], a[4], -(a[1] * e5));
    const double m02 = __builtin_fma(a[1], a[4], -(a[2] * e3));
    const double m12 = __builtin_fma(a[1], a[2], -(a[4] * e0));
    const bool use1 = __builtin_fabs(m11) > __builtin_fabs(m00);
    double v0 = use1 ? m01 : m00;
    double v1 = use1 ? m11 : m01;
    double v2 = use1 ? m12 : m02;
    const bool use2 = __builtin_fabs(m22) > __builtin_fabs(use1 ? v1 : v0);
    v0 = use2 ? m02 : v0;
    v1 = use2 ? m12 : v1;
    v2 = use2 ? m22 : v2;
    const double best = __builtin_fma(v0, v0, __builtin_fma(v1, v1, v2 * v2));
    // the vector leaves as binary32: one refinement (about 1e-14) is ample
    const double inv = rsqrt_d<1>(best);
    n[0] = v0 * inv;
    n[1] = v1 * inv;
    n[2] = v2 * inv;
    return best;
}

// The root y in [0, 1] of y^2 (3 + y) = t, t in [0, 4] (clamped).  With s =
// sqrt(t), y is within 0.1% of s / sqrt(3 + 0.57735 s - 0.0387 s^2), and Newton's
// steps on y^2 (3 + y) - t double the relative accuracy for every t, also near
// the double root t = 0: one step in binary32 and two in FP64, no loop.
__device__ __forceinline__ double cubic_root(double t) {
    t = __builtin_fmin(__builtin_fmax(t, 1e-30), 4.0);
    const float tf = (float)t;
    const float sf = __builtin_amdgcn_sqrtf(tf);
    float yf = sf * __builtin_amdgcn_rsqf(
                        __builtin_fmaf(sf, __builtin_fmaf(sf, -0.0387f, 0.57735f), 3.0f));
    yf = __builtin_fmaf(-__builtin_fmaf(yf * yf, 3.0f + yf, -tf),
                        __builtin_amdgcn_rcpf(yf * __builtin_fmaf(3.0f, yf, 6.0f)), yf);
    double y = (double)yf;
    const double idh = (double)__builtin_amdgcn_rcpf(yf * __builtin_fmaf(3.0f, yf, 6.0f));
#pragma unroll
    for (int k = 0; k < 2; ++k) {  // one slope serves both steps
        const double h = __builtin_fma(y * y, 3.0 + y, -t);
        y = __builtin_fma(-h, idh, y);
    }
    return y;
}

// Smallest-eigenvalue eigenvector of the symmetric 3x3 matrix
// [a0 a1 a2; a1 a3 a4; a2 a4 a5].  With q = tr(A)/3, B = A - q I,
// p^2 = |B|^2 / 6 and
// r = det(B) / (2 p^3), lambda = q - p (1 + y) with y^2 (3 + y) = 2 - 2r
// (cubic_root; the trigonometric closed form costs an FP64 acos, a cos and
// three divisions).
// y is returned: half the gap between the two smallest eigenvalues, over p.
// False when the vector is not defined, or wanted is false.
__device__ __forceinline__ bool smallest_eigvec(const double a[6], bool wanted, double n[3],
                                                double &gap) {
    const double q = (a[0] + a[3] + a[5]) * (1.0 / 3.0);
    const double b0 = a[0] - q, b3 = a[3] - q, b5 = a[5] - q;
    const double off = __builtin_fma(a[1], a[1], __builtin_fma(a[2], a[2], a[4] * a[4]));
    const double dia = __builtin_fma(b0, b0, __builtin_fma(b3, b3, b5 * b5));
    const double p2 = __builtin_fma(2.0, off, dia) * (1.0 / 6.0);
    const double ip = rsqrt_d<2>(p2);
    const double p = p2 * ip;
    const double m0 = __builtin_fma(b3, b5, -(a[4] * a[4]));
    const double m1 = __builtin_fma(a[1], b5, -(a[4] * a[2]));
    const double m2 = __builtin_fma(a[1], a[4], -(b3 * a[2]));
    const double det = __builtin_fma(b0, m0, __builtin_fma(a[2], m2, -(a[1] * m1)));
    double t = __builtin_fma(-(det * ip), ip * ip, 2.0);
    const double y = cubic_root(t);
    gap = y;
    const double best = adjugate_vec(a, b0, b3, b5, -__builtin_fma(p, y, p), n);
    // Where the two smallest eigenvalues lie close (windows across a depth
    // step), lambda from the cubic carries the rounding of det over their
    // gap; the vector's Rayleigh quotient does not.  (Vectors of 640x480
    // scenes: mean error 4e-9..3e-8 without this step, like the trigonometric
    // form's, 2e-13 with it.)
    // Windows with a missing depth, which no one wants, mostly look like that
    // too: with them nearly every wavefront took the branch (1080p 32.9 us, now
    // 29.5; R = 3 at 1280x720 18.8, now 16.3).
    if (wanted & (y < 1e-4)) {
        const double g0 = __builtin_fma(b0, n[0], __builtin_fma(a[1], n[1], a[2] * n[2]));
        const double g1 = __builtin_fma(a[1], n[0], __builtin_fma(b3, n[1], a[4] * n[2]));
        const double g2 = __builtin_fma(a[2], n[0], __builtin_fma(a[4], n[1], b5 * n[2]));
        const double mu = __builtin_fma(n[0], g0, __builtin_fma(n[1], g1, n[2] * g2));
        double v[3];
        if (adjugate_vec(a, b0, b3, b5, mu, v) > 0.0) {
            n[0] = v[0];
            n[1] = v[1];
            n[2] = v[2];
        }
    }
    return wanted & (p2 > 0.0) & (best > 0.0) & (best < (double)INFINITY);
}

// The window's scatter matrix from the points' own products, for the few
// windows whose two smallest eigenvalues agree to kFitDirect of the spread
// (about one in 10^4, all across depth steps).  These keep the plain evaluation
// of the definition, up to r, in its order, because its vectors are the ones
// that this tool returns there, not because better ones don't exist: the
// closed form's eigenvalue is off by about an ulp over y, the vector by
// another y.  Largest component error of 5x5 step windows against 128-bit
// arithmetic, median / maximum, here and with a Rayleigh step instead: y in
// 3e-7 .. 1e-6 5e-6 / 2e-4 and 3e-11 / 2e-8, 1e-7 .. 3e-7 5e-5 / 2e-3 and
// 2e-10 / 3e-6, below 4e-4 / 4e-2 and 2e-8 / 3e-4.
constexpr double kFitDirect = 1e-6;

template <int R>
__device__ __forceinline__ bool fit_direct(const float *__restrict__ depth, int64_t stride,
                                           int32_t x, int32_t y, float cx, float cy, double ifx,
                                           double ify, double n[3]) {
    const double u0 = ((double)x - (double)cx) * ifx;
    const double v0 = ((double)y - (double)cy) * ify;
    const double d0 = depth[(int64_t)y * stride + x];
    const double X0[3] = {u0 * d0, v0 * d0, d0};
    double s[3] = {0.0, 0.0, 0.0}, m[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int dy = -R; dy <= R; ++dy) {
        const float *row = depth + (int64_t)(y + dy) * stride;
        const double v = ((double)(y + dy) - (double)cy) * ify;
        float t[2 * R + 1];
#pragma unroll
        for (int dx = -R; dx <= R; ++dx) t[R + dx] = row[x + dx];
#pragma unroll
        for (int dx = -R; dx <= R; ++dx) {
            const double d = t[R + dx];
            const double u = ((double)(x + dx) - (double)cx) * ifx;
            const double p0 = u * d - X0[0], p1 = v * d - X0[1], p2 = d - X0[2];
            s[0] += p0;
            s[1] += p1;
            s[2] += p2;
            m[0] += p0 * p0;
            m[1] += p0 * p1;
            m[2] += p0 * p2;
            m[3] += p1 * p1;
            m[4] += p1 * p2;
            m[5] += p2 * p2;
        }
    }
    const double N = (double)((2 * R + 1) * (2 * R + 1));
    const double c[3] = {s[0] / N, s[1] / N, s[2] / N};
    const double a[6] = {m[0] - N * c[0] * c[0], m[1] - N * c[0] * c[1], m[2] - N * c[0] * c[2],
                         m[3] - N * c[1] * c[1], m[4] - N * c[1] * c[2], m[5] - N * c[2] * c[2]};
    const double q = (a[0] + a[3] + a[5]) / 3.0;
    const double b0 = a[0] - q, b3 = a[3] - q, b5 = a[5] - q;
    const double p2 = (b0 * b0 + b3 * b3 + b5 * b5 +
                       2.0 * (a[1] * a[1] + a[2] * a[2] + a[4] * a[4])) / 6.0;
    const double p = sqrt(p2);
    const double det = b0 * (b3 * b5 - a[4] * a[4]) - a[1] * (a[1] * b5 - a[4] * a[2]) +
                       a[2] * (a[1] * a[4] - b3 * a[2]);
    const double r = det / (2.0 * p2 * p);
    const double gap = cubic_root(2.0 - 2.0 * r);
    const double best = adjugate_vec(a, b0, b3, b5, -__builtin_fma(p, gap, p), n);
    if (!(p2 > 0.0 && best > 0.0 && best < (double)INFINITY)) return false;
    if (n[0] * u0 + n[1] * v0 + n[2] > 0.0) {
        n[0] = -n[0];
        n[1] = -n[1];
        n[2] = -n[2];
    }
    return true;
}

// Plane fit over the (2R+1)^2 window of each pixel: points back-projected
// (Eqs. 8-9), scatter matrix about their mean, smallest-eigenvalue
// eigenvector turned towards the camera.
//
// The kernel is bound by FP64 instructions, so the window's moments are taken
// apart.  A window point at offset (j, i) is (u0 d + j d / fx, v0 d + i d /
// fy, d): its scatter matrix is L M L^T with M the scatter of (j d, i d, d)
// and L = [1/fx 0 u0; 0 1/fy v0; 0 0 1].  M needs sums of d and d^2 weighted
// by 1, j, j^2, i, i j, i^2: sums over a column of 2R+1 rows (weights 1, i,
// i^2), which a lane forms once for its column, combined over the 2R+1
// neighbouring lanes.  The depth's own scatter (near 0 on a plane that faces
// the camera) is summed from c = d - D with D the smallest valid depth of the
// wavefront's block: c is small on a surface and never larger than the
// depths themselves.
struct FitCol {
    double c0, c1, s0;  // sum of c, i c, c^2
    double q0, q1, q2;  // sum of d^2, i d^2, i^2 d^2
};

// The column centred on entry R of c, q (= d^2).
template <int R>
__device__ __forceinline__ FitCol fit_col(const double *c, const double *q) {
    FitCol f;
    f.c0 = c[R];
    f.s0 = c[R] * c[R];
    f.q0 = q[R];
#pragma unroll
    for (int i = 1; i <= R; ++i) {
        const double w = (double)i;
        const double cf = c[R + i], cb = c[R - i];
        const double pq = q[R + i] + q[R - i], mq = q[R + i] - q[R - i];
        f.c0 += cf + cb;
        f.s0 = __builtin_fma(cf, cf, __builtin_fma(cb, cb, f.s0));
        f.q0 += pq;
        if (i == 1) {
            f.c1 = cf - cb;
            f.q1 = mq;
            f.q2 = pq;
        } else {
            f.c1 = __builtin_fma(w, cf - cb, f.c1);
            f.q1 = __builtin_fma(w, mq, f.q1);
            f.q2 = __builtin_fma(w * w, pq, f.q2);
        }
    }
    return f;
}

// A wavefront's column sums, in LDS for the neighbouring lanes: three planes
// of pairs, R entries of slack at both ends (what the wavefront's first and
// last R lanes read there only reaches their own windows, which are not
// outputs).
constexpr int kFitPlane = 64 + 2 * BN_MAX_FIT_RADIUS;
struct FitLds {
    d2 v[3][kFitPlane];
};

// The scatter matrix of the lane's window: its own column m and its
// neighbours' from LDS.
template <int R>
__device__ __forceinline__ void fit_scatter(const FitCol &m, FitLds &lds, uint32_t lane, double D,
                                            double u0, double v0, double ifx, double ify,
                                            double a[6]) {
    constexpr double N = (double)((2 * R + 1) * (2 * R + 1));
    const uint32_t at = lane + BN_MAX_FIT_RADIUS;
    lds.v[0][at] = d2{m.c0, m.q0};
    lds.v[1][at] = d2{m.c1, m.q1};
    lds.v[2][at] = d2{m.s0, m.q2};
    wave_lds_sync();
    double c0 = m.c0, ic0 = m.c1, s0 = m.s0, iq = m.q1, BB = m.q2;
    double jc0 = 0.0, jq = 0.0, jjq = 0.0, ijq = 0.0;
#pragma unroll
    for (int j = 1; j <= R; ++j) {
        const double w = (double)j;
        const d2 f0 = lds.v[0][at + j], b0 = lds.v[0][at - j];
        const d2 f1 = lds.v[1][at + j], b1 = lds.v[1][at - j];
        const d2 f2 = lds.v[2][at + j], b2 = lds.v[2][at - j];
        c0 += f0.x + b0.x;
        ic0 += f1.x + b1.x;
        s0 += f2.x + b2.x;
        iq += f1.y + b1.y;
        BB += f2.y + b2.y;
        if (j == 1) {
            jc0 = f0.x - b0.x;
            jq = f0.y - b0.y;
            jjq = f0.y + b0.y;
            ijq = f1.y - b1.y;
        } else {
            jc0 = __builtin_fma(w, f0.x - b0.x, jc0);
            jq = __builtin_fma(w, f0.y - b0.y, jq);
            jjq = __builtin_fma(w * w, f0.y + b0.y, jjq);
            ijq = __builtin_fma(w, f1.y - b1.y, ijq);
        }
    }
    wave_lds_sync();
    // second moments of A = j d, B = i d, C = d - D about their means (the
    // sum of j d is that of j c, the sum of i d that of i c)
    const double ma = jc0 * (-1.0 / N), mb = ic0 * (-1.0 / N), mc = c0 * (-1.0 / N);
    const double AA = __builtin_fma(ma, jc0, jjq);
    BB = __builtin_fma(mb, ic0, BB);
    const double AB = __builtin_fma(ma, ic0, ijq);
    const double AC = __builtin_fma(ma, c0, __builtin_fma(-D, jc0, jq));
    const double BC = __builtin_fma(mb, c0, __builtin_fma(-D, ic0, iq));
    const double CC = __builtin_fma(mc, c0, s0);
    // X = A/fx + u0 C, Y = B/fy + v0 C, Z = C
    const double xa = ifx * AC, yb = ify * BC;
    const double xz = __builtin_fma(u0, CC, xa);
    const double yz = __builtin_fma(v0, CC, yb);
    a[0] = __builtin_fma(ifx * ifx, AA, u0 * (xa + xz));
    a[1] = __builtin_fma(ifx * ify, AB, __builtin_fma(v0, xa, u0 * yz));
    a[2] = xz;
    a[3] = __builtin_fma(ify * ify, BB, v0 * (yb + yz));
    a[4] = yz;
    a[5] = CC;
}

// The smallest v over the wavefront, as a scalar: DPP row shifts by 1, 2, 4, 8
// leave each row of 16 lanes' minimum in its last lane, two row broadcasts
// the wavefront's in lane 63 (a lane without a source keeps its own v).
template <int CTRL>
__device__ __forceinline__ float min_dpp(float v) {
    const int i = __float_as_int(v);
    return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ float wave_min(float v) {
    v = min_dpp<0x111>(v);
    v = min_dpp<0x112>(v);
    v = min_dpp<0x114>(v);
    v = min_dpp<0x118>(v);
    v = min_dpp<0x142>(v);
    v = min_dpp<0x143>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Each wavefront takes 64 columns, of which the middle 64 - 2R are outputs,
// and TY rows: TY = 4 shares the loads and the columns' conversions over four
// rows, TY = 1 makes four times the wavefronts of smaller frames.  About 290
// VALU instructions per output at R = 2 (FP64 ones issue at 30 T lane-op/s
// here): 1080p 84 -> 29 us, 640x480 15.7 -> 6.7 us, R = 3 at 1280x720 61 -> 16
// us against 25-tap sums per pixel with the trigonometric eigenvalue.  Row
// sums kept in a register ring down the rows (no LDS) took 27 us without the
// two branches on close eigenvalues, but spilled with them (41 us).
template <int R, int TY>
__global__ __launch_bounds__(256, 4) void k_plane_fit(const float *__restrict__ depth, int32_t H,
                                                      int32_t W, int64_t stride, double ifx,
                                                      double ify, float cx, float cy,
                                                      float *__restrict__ normals,
                                                      uint8_t *__restrict__ mask) {
    constexpr int NR = TY + 2 * R;   // rows a lane reads
    constexpr uint32_t OC = 64 - 2 * R;  // output columns of a wavefront
    __shared__ FitLds s_fit[4];
    __shared__ float s_n[4][64 * (TY > 3 ? TY : 3)];
    const uint32_t gx = ((uint32_t)W + OC - 1u) / OC;  // wavefronts per row of the frame
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = wave_id();
    const int32_t xb = (int32_t)((blockIdx.x % gx) * OC);
    const int32_t x = xb + (int32_t)lane - R;
    const int32_t y0 = (int32_t)((blockIdx.x / gx) * (4u * TY) + w * TY);
    // Loads are unconditional, clamped into the frame: what a clamped load
    // brings in only reaches windows that leave the frame.
    const int32_t xl = min(max(x, 0), W - 1);
    float d[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int32_t y = min(max(y0 - R + k, 0), H - 1);
        d[k] = depth[(int64_t)y * stride + xl];
    }
    float dmin = INFINITY;
    uint64_t good[NR];  // the lanes whose depth is valid
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const bool g = tap_ok(d[k]) != 0u;
        good[k] = __builtin_amdgcn_ballot_w64(g);
        dmin = fminf(dmin, g ? d[k] : INFINITY);
    }
    dmin = wave_min(dmin);
    const double D = dmin < INFINITY ? (double)dmin : 0.0;
    const double u0 = ((double)x - (double)cx) * ifx;
    const bool out_lane = (lane >= (uint32_t)R) & (lane < 64u - R);
    const bool x_in = out_lane & (x >= R) & (x + R < W);
    const uint32_t nx = min(OC, (uint32_t)(W - xb));  // pixels of this wavefront's rows
    float *st = s_n[w];
    uint32_t close = 0;  // bit r: the lane's window of row y0 + r goes to fit_direct
    double c[NR], q[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        c[k] = (double)d[k] - D;
        q[k] = (double)d[k] * (double)d[k];
        if (k < 2 * R) continue;
        const int32_t y = y0 + k - 2 * R;
        if (y >= H) break;  // uniform over the wavefront
        uint64_t all = good[k];
#pragma unroll
        for (int i = 1; i <= 2 * R; ++i) all &= good[k - i];
        uint64_t full = all;
#pragma unroll
        for (int j = 1; j <= R; ++j) full &= (all >> j) & (all << j);
        if (y < R || y + R >= H) full = 0;
        const double v0 = ((double)y - (double)cy) * ify;
        double a[6], n[3], gap;
        fit_scatter<R>(fit_col<R>(c + k - 2 * R, q + k - 2 * R), s_fit[w], lane, D, u0, v0, ifx,
                       ify, a);
        const bool in = ((full >> lane) & 1u) & x_in;
        const bool ok = smallest_eigvec(a, in, n, gap);
        close |= (uint32_t)(in & (gap < kFitDirect)) << (k - 2 * R);
        const bool away = __builtin_fma(n[0], u0, __builtin_fma(n[1], v0, n[2])) > 0.0;
        const int64_t i0 = (int64_t)y * W + xb;
        if (out_lane) {
            const uint32_t o = lane - R;
            const float sg = away ? -1.0f : 1.0f;
            st[3 * o + 0] = ok ? sg * (float)n[0] : 0.0f;
            st[3 * o + 1] = ok ? sg * (float)n[1] : 0.0f;
            st[3 * o + 2] = ok ? sg * (float)n[2] : 0.0f;
            out_store_byte(ok ? (uint8_t)BN_VALID : (uint8_t)BN_INVALID, out_buf(mask + i0, nx),
                           o);
        }
        wave_lds_sync();
        const OutBuf nb = out_buf(normals + 3 * i0, 12 * nx);
#pragma unroll
        for (int j = 0; j < 3; ++j) out_store(st[64 * j + lane], nb, 4 * lane + 256 * j);
        wave_lds_sync();
    }
    if (__builtin_amdgcn_ballot_w64(close != 0) == 0) return;
    // the wavefront's windows for fit_direct, one per lane: (row, column)
    // packed into the staging slice
    uint32_t *list = reinterpret_cast<uint32_t *>(st);
    uint32_t count = 0;
#pragma unroll
    for (int r = 0; r < TY; ++r) {
        const bool mine = ((close >> r) & 1u) != 0u;
        const uint64_t m = __builtin_amdgcn_ballot_w64(mine);
        const uint32_t before = (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
        if (mine) list[count + before] = ((uint32_t)r << 8) | lane;
        count += (uint32_t)__builtin_popcountll(m);
    }
    wave_lds_sync();
    // the stores above, by other lanes of this wavefront, come first
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    for (uint32_t k = lane; k < count; k += 64u) {
        const uint32_t e = list[k];
        const int32_t xk = xb + (int32_t)(e & 0xffu) - R;
        const int32_t yk = y0 + (int32_t)(e >> 8);
        double n[3];
        const bool ok = fit_direct<R>(depth, stride, xk, yk, cx, cy, ifx, ify, n);
        const int64_t i = (int64_t)yk * W + xk;
        normals[3 * i + 0] = ok ? (float)n[0] : 0.0f;
        normals[3 * i + 1] = ok ? (float)n[1] : 0.0f;
        normals[3 * i + 2] = ok ? (float)n[2] : 0.0f;
        mask[i] = ok ? (uint8_t)BN_VALID : (uint8_t)BN_INVALID;
    }
}

typedef void (*FitFn)(const float *, int32_t, int32_t, int64_t, double, double, float, float,
                      float *, uint8_t *);

// Rows per wavefront: 4, or 1 for frames below kFitSmall pixels, whose
// wavefronts of 4 rows would not fill the chip once (TY 4 against TY 1:
// 320x240 6.3 / 4.6 us, 640x480 8.2 / 6.7, 1000x600 10.6 / 9.7, 1280x720 12.9
// / 13.5, 1440x900 17.7 / 18.2, 1920x1080 29.3 / 32.2).
constexpr int64_t kFitSmall = 3 << 18;

FitFn fit_kernel(int r, bool small) {
    switch (r) {
        case 1: return small ? k_plane_fit<1, 1> : k_plane_fit<1, 4>;
        case 2: return small ? k_plane_fit<2, 1> : k_plane_fit<2, 4>;
        case 3: return small ? k_plane_fit<3, 1> : k_plane_fit<3, 4>;
    }
    return nullptr;
}

}  // namespace

}  // namespace bn

using namespace bn;

extern "C" {

int bn_normal_angles(const float *normals, int32_t height, int32_t width, float *theta,
                     float *phi, void *stream) {
    if (height < 0 || width < 0) return BN_ERR_INVALID_ARG;
    if ((int64_t)height * width > BN_MAX_PIXELS) return BN_ERR_UNSUPPORTED;
    if (height == 0 || width == 0) return BN_OK;
    if (!normals || !theta || !phi) return BN_ERR_INVALID_ARG;
    const uint32_t npix = (uint32_t)height * (uint32_t)width;
    hipLaunchKernelGGL(k_angles, dim3((npix + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       normals, npix, theta, phi);
    return hipGetLastError() == hipSuccess ? BN_OK : BN_ERR_DEVICE;
}

int bn_angle_mse(const float *normals_a, const uint8_t *mask_a, const float *normals_b,
                 const uint8_t *mask_b, int32_t height, int32_t width, double *workspace,
                 double *result, void *stream) {
    if (height < 0 || width < 0) return BN_ERR_INVALID_ARG;
    if ((int64_t)height * width > BN_MAX_PIXELS) return BN_ERR_UNSUPPORTED;
    if (!workspace || !result) return BN_ERR_INVALID_ARG;
    const uint32_t npix = (uint32_t)height * (uint32_t)width;
    if (npix > 0 && (!normals_a || !normals_b)) return BN_ERR_INVALID_ARG;
    uint32_t blocks = (npix + 255) / 256;
    if (blocks > kMseBlocks) blocks = kMseBlocks;
    if (blocks == 0) blocks = 1;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_mse_partial, dim3(blocks), dim3(256), 0, s, normals_a, mask_a,
                       normals_b, mask_b, npix, workspace);
    if (hipGetLastError() != hipSuccess) return BN_ERR_DEVICE;
    if (blocks <= kMseFew) {
        hipLaunchKernelGGL(k_mse_final<256>, dim3(1), dim3(256), 0, s, (const double *)workspace,
                           blocks, result);
    } else {
        hipLaunchKernelGGL(k_mse_final<1024>, dim3(1), dim3(1024), 0, s,
                           (const double *)workspace, blocks, result);
    }
    return hipGetLastError() == hipSuccess ? BN_OK : BN_ERR_DEVICE;
}

int bn_plane_fit_normals(const float *depth, int32_t height, int32_t width, int64_t depth_stride,
                         float fx, float fy, float cx, float cy, int32_t radius, float *normals,
                         uint8_t *mask, void *stream) {
    if (radius < 1) return BN_ERR_INVALID_ARG;
    if (radius > BN_MAX_FIT_RADIUS) return BN_ERR_UNSUPPORTED;
    int rc = check_frame_args(depth, height, width, depth_stride, fx, fy, cx, cy, normals, mask);
    if (rc != BN_OK) return rc;
    if (height == 0 || width == 0) return BN_OK;
    const bool small = (int64_t)height * width < kFitSmall;
    FitFn fn = fit_kernel(radius, small);
    const uint32_t cols = 64u - 2u * (uint32_t)radius, rows = small ? 4u : 16u;  // of a workgroup
    const uint64_t blocks = (uint64_t)(((uint32_t)width + cols - 1u) / cols) *
                            (uint64_t)(((uint32_t)height + rows - 1u) / rows);
    hipLaunchKernelGGL(fn, dim3((uint32_t)blocks), dim3(256), 0, (hipStream_t)stream, depth,
                       height, width,
                       depth_stride, 1.0 / (double)fx, 1.0 / (double)fy, cx, cy, normals, mask);
    return hipGetLastError() == hipSuccess ? BN_OK : BN_ERR_DEVICE;
}

}  // extern "C"
