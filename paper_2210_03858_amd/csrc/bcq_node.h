// Calls of the autograd node (bcq_torch.cpp) into the kernels' library: the two halves of a training step as it has them in
// hand.  Both compute what the entry points of bcq.h compute, bit for bit, in fewer launches; they are no part of the C ABI.
#pragma once
#include "../../include/bcq.h"

extern "C" {

// Forward with the scales in two tensors: alpha_first[q_first][N][K/g] and alpha_rest[q - q_first][N][K/g].  alpha[q][N][K/g]
// receives them all, as the backward pass wants them.
bcq_status bcq_node_forward(const uint32_t* packed, const float* alpha_first, int q_first, const float* alpha_rest, float* alpha,
                            const void* x, int dtype, int64_t T, int64_t N, int64_t K, int64_t g, int q, void* y, void* workspace,
                            size_t workspace_bytes, void* stream);

// Both gradients in one call, where bcq_node_backward_joint (1 or 0, from the sizes alone) says that this saves a launch; other calls
// are the two entry points of bcq.h.  The two workspaces are those of bcq_linear_bwd_input_grouped and bcq_linear_bwd_alpha_grouped, in
// use at once.
int bcq_node_backward_joint(int with_twin, int dtype, int64_t T, int64_t N, int64_t K, int64_t g, int q);
bcq_status bcq_node_backward(const uint32_t* packed, const float* alpha, const void* x, const void* dy, int dtype, int64_t T, int64_t N,
                             int64_t K, int64_t g, int q, int q_train, float grad_scale, void* dx, void* input_workspace,
                             size_t input_bytes, float* dalpha, void* alpha_workspace, size_t alpha_bytes, void* stream);

}  // extern "C"
