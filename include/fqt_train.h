/*
 * fqt_train.h -- the layer backward of a training step: fqt_layer_backward with what the
 * training loop does around it, in the same launches (fqt.h holds the conventions).
 */
#ifndef FQT_TRAIN_H
#define FQT_TRAIN_H

#include "fqt.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Workspace of fqt_train_backward: a FQT_WS_LAYER workspace (with its state in the first
 * FQT_WS_STATE_BYTES: run fqt_workspace_init once) followed by partial sums. */
int fqt_train_workspace_size(const fqt_layer_desc *desc, const fqt_quant_cfg *cfg, size_t *bytes);

/* For a layer H = Gamma_d * I, I the integer product of fqt_binary_forward (Section 5.1), and
 * the gradient dH [N][D][Ho][Wo] of its output, all float32 (FQT_E_DTYPE otherwise):
 *   dX, dW      fqt_layer_backward of dY = dH * gamma_d (one float32 product per element), with
 *               dX = 0 where |X| <= 1 does not hold (straight-through estimator, Section 3.1);
 *   dgamma[d] = sum over n, ho, wo of dH * I (float32 sums of at most a plane or a few 64-pixel
 *               tiles, added in float64 in a fixed order).
 * dH and I 16-byte aligned, gamma [D]; dX, dW and dgamma as X, W and gamma. */
int fqt_train_backward(const fqt_layer_desc *desc, const fqt_quant_cfg *cfg, const float *X,
                       const float *W, const float *gamma, const int32_t *I, const float *dH,
                       float *dX, float *dW, float *dgamma, void *ws, size_t ws_bytes,
                       void *hip_stream);

#ifdef __cplusplus
}
#endif
#endif /* FQT_TRAIN_H */
