// The cosine loss of the differentiation path and its gradient, called by the
// Python binding through the library's exported symbols (not part of the
// estimator's interface, include/bnormals.h).  Device pointers, asynchronous
// on `stream`, nothing allocated; arrays dense, floats 4-byte aligned.
//   bn_cosine_loss: over the pixels U with mask == BN_VALID and target_mask ==
//     BN_VALID, *loss = sum of (1 - normals . target) / *count and *count =
//     max(|U|, 1), in binary32 (the sum in FP64, in a fixed order).  used
//     (nullable) receives 1 for a pixel of U and 0 for the others.  workspace:
//     BN_COSINE_WORKSPACE(pixels) doubles, 16-byte aligned.
//   bn_cosine_loss_vjp: grad_normals = -(*grad / *count) target at the
//     pixels of U, 0 times target at the others.
// normals, target, grad_normals [pixels][3]; masks, used [pixels]; pixels up
// to BN_COSINE_MAX_PIXELS.
#pragma once

#include <stdint.h>

#define BN_COSINE_TILE 2048 /* pixels of a workgroup */
#define BN_COSINE_WORKSPACE(pixels) (2 * (((pixels) + BN_COSINE_TILE - 1) / BN_COSINE_TILE))
#define BN_COSINE_MAX_PIXELS (1LL << 30)

extern "C" {
int bn_cosine_loss(const float *normals, const float *target, const uint8_t *mask,
                   const uint8_t *target_mask, int64_t pixels, uint8_t *used, double *workspace,
                   float *loss, float *count, void *stream);
int bn_cosine_loss_vjp(const float *target, const uint8_t *used, int64_t pixels,
                       const float *grad, const float *count, float *grad_normals,
                       void *stream);
}
