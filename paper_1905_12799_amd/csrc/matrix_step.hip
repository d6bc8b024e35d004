// One matrix instruction of the distances on operands as they are given: a test measures with it what the instruction leaves out of a
// sum, which is part of the bound that decides the close calls (pair_error_of).
#include "lloyd_device.h"

namespace rls {

namespace {

// A wave per product.  a, b: eight elements per lane, of row (column) lane % 32 and of its half of K; acc: result 4 q + e of lane l is
// element (8 q + 4 (l / 32) + e, l % 32).
__global__ void __launch_bounds__(64) matrix_step_kernel(int bf16, const uint4 *a, const uint4 *b, const float *acc_in, float *acc_out)
{
    const int64_t at = (int64_t)blockIdx.x * 64 + threadIdx.x;
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = acc_in[at * 16 + i];
    if (bf16) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[at]), as_bf16x8(b[at]), acc, 0, 0, 0);
    else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a[at]), as_f16x8(b[at]), acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) acc_out[at * 16 + i] = acc[i];
}

}  // namespace

}  // namespace rls

extern "C" int32_t rls_matrix_step(int32_t bf16, const void *a_dev, const void *b_dev, const float *acc_dev, float *acc_out_dev, int32_t n, void *stream)
{
    if (!a_dev || !b_dev || !acc_dev || !acc_out_dev) return RLS_ERR_NULL;
    if (n < 1) return RLS_ERR_INVALID_ARG;
    hipLaunchKernelGGL(rls::matrix_step_kernel, dim3(n), dim3(64), 0, (hipStream_t)stream, (int)bf16, static_cast<const uint4 *>(a_dev),
                       static_cast<const uint4 *>(b_dev), acc_dev, acc_out_dev);
    RLS_HIP_TRY(hipGetLastError());
    return RLS_OK;
}
