// The cosine loss over the pixels valid in both of two normal maps, and its
// gradient (see bn_loss.h).
//
// Bound by HBM: 26 bytes in (and 1 out) per pixel forward, 13 in and 12 out
// backward.  As elementwise and reduction kernels of the tensor library the
// two take about 14 passes over [n][H][W] and [n][H][W][3] arrays (16 x
// 640x480: about 200 us of kernels); here one pass each way and a small sum
// (24.8 + 4 us and 19.3 us).
#include "bn_loss.h"

#include "bn_device.h"
#include "bn_internal.h"

#pragma clang fp contract(off)

namespace bn {
namespace {

// 1 - n . t of one pixel, each operation rounded as the tensor expressions
// (normals * target).sum(-1) and 1 - cos round theirs.
__device__ __forceinline__ float one_minus_cos(float nx, float ny, float nz, float tx, float ty,
                                               float tz) {
    const float p = nx * tx;
    const float q = ny * ty;
    const float r = nz * tz;
    return 1.0f - ((p + q) + r);
}

// Sums of (1 - cos) and of the pixels of U over the workgroup's
// BN_COSINE_TILE pixels: each thread takes groups of four consecutive pixels
// (the groups of a load instruction lie side by side), 16-byte loads where VEC
// (every array starts on a 16-byte line; masks and used on 4).
template <bool VEC>
__global__ __launch_bounds__(256) void k_cosine(const float *__restrict__ normals,
                                                const float *__restrict__ target,
                                                const uint8_t *__restrict__ mask,
                                                const uint8_t *__restrict__ target_mask,
                                                uint32_t npix, uint8_t *__restrict__ used,
                                                double *__restrict__ part) {
    constexpr int G = BN_COSINE_TILE / 1024;  // groups per thread
    double s = 0.0;
    uint32_t k = 0;
    f4 n[G][3], t[G][3];
    uint32_t m[G], mt[G];
    const uint32_t i0 = blockIdx.x * (uint32_t)BN_COSINE_TILE + 4u * threadIdx.x;
    if (VEC) {
        // every load of the thread before its arithmetic
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t i = i0 + 1024u * g;
            if (i + 4u > npix) continue;
            const f4 *np = reinterpret_cast<const f4 *>(normals + 3 * (int64_t)i);
            const f4 *tp = reinterpret_cast<const f4 *>(target + 3 * (int64_t)i);
            m[g] = *reinterpret_cast<const uint32_t *>(mask + i);
            mt[g] = *reinterpret_cast<const uint32_t *>(target_mask + i);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                n[g][c] = np[c];
                t[g][c] = tp[c];
            }
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t i = i0 + 1024u * g;
        if (VEC && i + 4u <= npix) {
            const float a[12] = {n[g][0].x, n[g][0].y, n[g][0].z, n[g][0].w, n[g][1].x, n[g][1].y,
                                 n[g][1].z, n[g][1].w, n[g][2].x, n[g][2].y, n[g][2].z, n[g][2].w};
            const float b[12] = {t[g][0].x, t[g][0].y, t[g][0].z, t[g][0].w, t[g][1].x, t[g][1].y,
                                 t[g][1].z, t[g][1].w, t[g][2].x, t[g][2].y, t[g][2].z, t[g][2].w};
            uint32_t u = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = (((m[g] >> (8 * j)) & 0xffu) == BN_VALID) &
                                (((mt[g] >> (8 * j)) & 0xffu) == BN_VALID);
                const float v = one_minus_cos(a[3 * j], a[3 * j + 1], a[3 * j + 2], b[3 * j],
                                              b[3 * j + 1], b[3 * j + 2]);
                s += in ? (double)v : 0.0;
                u |= (in ? 1u : 0u) << (8 * j);
            }
            k += (uint32_t)__builtin_popcount(u);
            if (used) *reinterpret_cast<uint32_t *>(used + i) = u;
            continue;
        }
        for (uint32_t j = i; j < i + 4u && j < npix; ++j) {
            const bool in = (mask[j] == BN_VALID) & (target_mask[j] == BN_VALID);
            const float *a = normals + 3 * (int64_t)j;
            const float *b = target + 3 * (int64_t)j;
            const float v = one_minus_cos(a[0], a[1], a[2], b[0], b[1], b[2]);
            s += in ? (double)v : 0.0;
            k += in ? 1u : 0u;
            if (used) used[j] = in ? 1 : 0;
        }
    }
    __shared__ double s_s[4];
    __shared__ uint32_t s_k[4];
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off);
        k += __shfl_xor(k, off);
    }
    if ((threadIdx.x & 63u) == 0) {
        s_s[threadIdx.x >> 6] = s;
        s_k[threadIdx.x >> 6] = k;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[2 * (int64_t)blockIdx.x + 0] = ((s_s[0] + s_s[1]) + s_s[2]) + s_s[3];
        part[2 * (int64_t)blockIdx.x + 1] = (double)(s_k[0] + s_k[1] + s_k[2] + s_k[3]);
    }
}

// One workgroup: the partial sums in a fixed order, then the mean.
__global__ __launch_bounds__(1024) void k_cosine_mean(const double *__restrict__ part,
                                                      uint32_t nparts, float *__restrict__ loss,
                                                      float *__restrict__ count) {
    double s = 0.0, k = 0.0;
    const d2 *p = reinterpret_cast<const d2 *>(part);
#pragma unroll 4
    for (uint32_t j = threadIdx.x; j < nparts; j += 1024u) {
        const d2 v = p[j];
        s += v.x;
        k += v.y;
    }
    __shared__ double s_s[16], s_k[16];
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off);
        k += __shfl_xor(k, off);
    }
    if ((threadIdx.x & 63u) == 0) {
        s_s[threadIdx.x >> 6] = s;
        s_k[threadIdx.x >> 6] = k;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        s = k = 0.0;
        for (int w = 0; w < 16; ++w) {
            s += s_s[w];
            k += s_k[w];
        }
        const float den = k > 1.0 ? (float)k : 1.0f;
        *loss = (float)s / den;
        *count = den;
    }
}

// grad_normals as a flat array of 3 npix floats.  VEC: three float4s per
// thread, each load and store instruction of a wavefront one contiguous KiB,
// the stores streaming (16 x 640x480: 24.0 us with plain stores, 19.3);
// float4 f covers the floats 4f .. 4f+3, of the pixels (4f)/3 and (4f)/3 + 1
// (and no third).  Otherwise three floats per thread, 64 apart.
template <bool VEC>
__global__ __launch_bounds__(256) void k_cosine_vjp(const float *__restrict__ target,
                                                    const uint8_t *__restrict__ used,
                                                    uint32_t npix, const float *__restrict__ grad,
                                                    const float *__restrict__ count,
                                                    float *__restrict__ out) {
    const float c = -(*grad / *count);
    const uint32_t nf = 3u * npix;  // floats
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = blockIdx.x * 4u + wave_id();
    if (VEC) {
        const uint32_t n4 = nf / 4u;
        f4 t[3];
        uint32_t ua[3], ub[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t f = 192u * w + 64u * k + lane;
            if (f >= n4) continue;
            const uint32_t p = 4u * f / 3u;
            t[k] = reinterpret_cast<const f4 *>(target)[f];
            ua[k] = used[p];
            ub[k] = used[min(p + 1u, npix - 1u)];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t f = 192u * w + 64u * k + lane;
            if (f >= n4) continue;
            const uint32_t at = 4u * f - 3u * (4u * f / 3u);  // first float's place in its pixel
            const float a = ua[k] ? c : 0.0f, b = ub[k] ? c : 0.0f;
            // floats of the first pixel: 3 - at of them
            const f4 v = f4{a * t[k].x, (at < 2u ? a : b) * t[k].y, (at < 1u ? a : b) * t[k].z,
                            b * t[k].w};
            const uint32_t fw = 192u * w + 64u * k;  // the wavefront's first
            out_store(v, out_buf(reinterpret_cast<f4 *>(out) + fw, 16u * min(64u, n4 - fw)),
                      16u * lane);
        }
        // the last nf % 4 floats
        if (blockIdx.x == 0 && threadIdx.x < nf % 4u) {
            const uint32_t f = 4u * n4 + threadIdx.x;
            out[f] = (used[f / 3u] ? c : 0.0f) * target[f];
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t f = 192u * w + 64u * k + lane;
        if (f < nf) out[f] = (used[f / 3u] ? c : 0.0f) * target[f];
    }
}

bool at(const void *p, uintptr_t a) { return ((uintptr_t)p % a) == 0; }

}  // namespace
}  // namespace bn

using namespace bn;

extern "C" {

int bn_cosine_loss(const float *normals, const float *target, const uint8_t *mask,
                   const uint8_t *target_mask, int64_t pixels, uint8_t *used, double *workspace,
                   float *loss, float *count, void *stream) {
    if (!normals || !target || !mask || !target_mask || !workspace || !loss || !count || pixels < 1)
        return BN_ERR_INVALID_ARG;
    if (pixels > BN_COSINE_MAX_PIXELS) return BN_ERR_UNSUPPORTED;
    if (!at(normals, 4) || !at(target, 4) || !at(loss, 4) || !at(count, 4) || !at(workspace, 16))
        return BN_ERR_INVALID_ARG;
    const bool vec = at(normals, 16) && at(target, 16) && at(mask, 4) && at(target_mask, 4) &&
                     at(used, 4);
    const uint32_t blocks = (uint32_t)((pixels + BN_COSINE_TILE - 1) / BN_COSINE_TILE);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(vec ? k_cosine<true> : k_cosine<false>, dim3(blocks), dim3(256), 0, s,
                       normals, target, mask, target_mask, (uint32_t)pixels, used, workspace);
    if (hipGetLastError() != hipSuccess) return BN_ERR_DEVICE;
    hipLaunchKernelGGL(k_cosine_mean, dim3(1), dim3(1024), 0, s, (const double *)workspace, blocks,
                       loss, count);
    return hipGetLastError() == hipSuccess ? BN_OK : BN_ERR_DEVICE;
}

int bn_cosine_loss_vjp(const float *target, const uint8_t *used, int64_t pixels,
                       const float *grad, const float *count, float *grad_normals,
                       void *stream) {
    if (!target || !used || !grad || !count || !grad_normals || pixels < 1)
        return BN_ERR_INVALID_ARG;
    if (pixels > BN_COSINE_MAX_PIXELS) return BN_ERR_UNSUPPORTED;
    if (!at(target, 4) || !at(grad, 4) || !at(count, 4) || !at(grad_normals, 4))
        return BN_ERR_INVALID_ARG;
    const bool vec = at(target, 16) && at(grad_normals, 16);
    // 768 float4s (1024 pixels) or 768 floats (256 pixels) per workgroup
    const int64_t per = vec ? 1024 : 256;
    const uint32_t blocks = (uint32_t)((pixels + per - 1) / per);
    hipLaunchKernelGGL(vec ? k_cosine_vjp<true> : k_cosine_vjp<false>, dim3(blocks), dim3(256), 0,
                       (hipStream_t)stream, target, used, (uint32_t)pixels, grad, count,
                       grad_normals);
    return hipGetLastError() == hipSuccess ? BN_OK : BN_ERR_DEVICE;
}

}  // extern "C"
