// Host-side launchers of the ranker training kernels (sd3_mlp.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sd3_common.h"

namespace sd3 {

// Blocks the training kernels launch for n samples; a gradient needs
// MLP_NPARAM + 1 floats of scratch for each.
int mlp_blocks(int64_t n);
void mlp_forward(const float *params, const float *x, int64_t n, float *y, hipStream_t st);
void mlp_loss_grad(const float *params, const float *x, const float *t, int64_t n, float *part, float *loss,
                   float *grad, hipStream_t st);
void adam_step(float *p, const float *g, float *m, float *v, int64_t n, int step, float lr,
               float b1, float b2, float eps, hipStream_t st);

}  // namespace sd3
