// Launchers of the mean-state kernel, one translation unit per slab type.
// prm == nullptr: only raise the kernels' dynamic-LDS limit to `lds`.
// Returns hipErrorInvalidValue when no kernel is instantiated for the number of row slots.
#pragma once
#include <hip/hip_runtime.h>

#include "fda_mean_kernel.hpp"

namespace fda {
// Sketch-row slots of one workgroup.  Each row group repeats the stream of the slab, so a sketch that fits one
// workgroup should not be split for want of a kernel (9 x 250: 30 x 7M fp32 233 -> 162 us, 8 x 40M bf16 401 -> 279).
// Nine is where 128 registers (two workgroups per CU on bf16 slabs) end: nine rows take 120, ten 147.
constexpr int kMeanMaxLR = kMaxLR;
constexpr int kMeanBatchF32 = 4;             // slab rows per batch: 4 x 16 bytes per lane ...
constexpr int kMeanBatchBF16 = 4;            // ... or 4 x 8 bytes

// FB: bits per field of the tabulated hash (field_bits_for(m)): 11 or 16
hipError_t launch_mean_f32(int LR, int FB, const MeanParams* prm, size_t lds, hipStream_t st);
hipError_t launch_mean_bf16(int LR, int FB, const MeanParams* prm, size_t lds, hipStream_t st);

template <typename T, int KB, int LR, int FB>
hipError_t launch_mean_kernel(const MeanParams* prm, size_t lds, hipStream_t st) {
  auto kern = mean_state_kernel<T, KB, LR, FB>;
  if (prm == nullptr)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(prm->R * prm->P), dim3(kStateThreads), lds, st, *prm);
  return hipGetLastError();
}
}  // namespace fda
