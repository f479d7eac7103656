// Registry of the fused loss-and-gradient kernels (fused_loss.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "registry.hpp"

namespace mifft {

// loss[b] = sum_k w |(A x_b)_k|^2 and grad_b = A^H (2 w A x_b) for the
// batched FP32 transform A of sign `sign` and scale `scale`.  scaled_next: the
// next kernel scales grad (see keep_gradient).
using LaunchLossGrad = hipError_t (*)(const void* x, const float* w, void* grad, float* loss, const void* rows,
                                      int64_t batch, float scale, int64_t grid_limit, bool scaled_next,
                                      hipStream_t stream);

// Fused loss-gradient kernel (two transforms per group, so its own best
// shape differs from the plain transform's), per log2 N (index 1..11):
// the autotuner's pick on MI355X at 2^25 elements (log2 EPT, workgroup
// size; the kind field is unused).
constexpr Variant kDefaultLoss[12] = {
    {0, 0, 0},     // unused
    {1, 128, 0},   // N=2
    {2, 64, 0},    // N=4
    {3, 256, 0},   // N=8
    {2, 64, 0},    // N=16
    {2, 256, 0},   // N=32
    {2, 256, 0},   // N=64
    {3, 256, 0},   // N=128
    {4, 64, 0},    // N=256
    {3, 256, 0},   // N=512
    {4, 256, 0},   // N=1024
    {4, 128, 0},   // N=2048
};

struct KernelLossGrad {
    int log2n, log2ept, wg, sign;
    LaunchLossGrad fn;
    int (*occupancy)();
    int rows;  // twiddle-row entries needed (0: one thread per transform)
};

void register_loss_grad(const KernelLossGrad& k);
const KernelLossGrad* find_loss_grad(int log2n, int log2ept, int wg, int sign);

}  // namespace mifft
