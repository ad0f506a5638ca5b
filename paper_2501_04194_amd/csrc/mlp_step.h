// The combined kernels that the network binding (mlp.py) composes a training
// step of, beside the building blocks of include/stlmi_mlp.h.  Same conventions
// (caller-owned device memory, asynchronous on `stream`, no allocation, negative
// stl_status with a message in stl_last_error()).  Not part of the public ABI.
#pragma once
#include "../../include/stlmi_mlp.h"

extern "C" {

/*
 * The gradient of a hidden layer's pre-activation in one product: g16 =
 * bf16((A * B) * (h > 0)), h the BF16 post-activation (M x N, h[m*ldh + n]),
 * g16 M x N (g16[m*ldg + n]); A and B as in stl_bf16_gemm.  The same bits as
 * stl_bf16_gemm into FP32 followed by stl_relu_grad_bf16.
 */
stl_status stl_bf16_gemm_relu_grad(const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B, int64_t sbk,
                                   int64_t sbn, int32_t M, int32_t N, int32_t K, const uint16_t* h, int64_t ldh,
                                   uint16_t* g16, int64_t ldg, void* stream);

/* stl_colsum over BF16 x (widened exactly, FP32 sums). */
stl_status stl_colsum_bf16(const uint16_t* x, int32_t rows, int32_t cols, int64_t ld, float* out, void* stream);

/* stl_adam_step for several tensors (host array; one launch per 16 of them). */
typedef struct {
    float* w;
    const float* g;
    float* m;
    float* v;
    uint16_t* w16;
    int64_t n;
} stl_adam_tensor;
stl_status stl_adam_step_multi(const stl_adam_tensor* tensors, int32_t n_tensors, float lr, float b1, float b2,
                               float eps, int32_t step, void* stream);
}
