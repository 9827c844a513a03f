// The batched FP32 kernel: plans of FP32 instances only (gfx950); its body is in batched_valu.hpp, which the
// kernel for plans with MFMA instances (demap_batched.hip) has too.
#include "batched_valu.hpp"

namespace dm {

namespace {

__global__ __launch_bounds__(kBatchThreads) void demap_batched_valu_kernel(const BatchArgs a) {
    extern __shared__ __align__(16) float lds[];
    batched_valu(a, lds);
}

}  // namespace

hipError_t prepare_batched_valu() {
    return hipFuncSetAttribute((const void*)demap_batched_valu_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kBatchedLdsBytes);
}

hipError_t launch_demap_batched_valu(const BatchArgs& a, int grid, hipStream_t st) {
    hipLaunchKernelGGL(demap_batched_valu_kernel, dim3(grid), dim3(kBatchThreads), a.lds_bytes, st, a);
    return hipGetLastError();
}

}  // namespace dm
