// Launchers of the state kernel.  The instantiations are spread over many translation units so
// that they compile in parallel: one per (slab type, worker-slot count).
// prm == nullptr: only raise the kernel's dynamic-LDS limit to `lds`.
// Returns hipErrorInvalidValue when no kernel is instantiated for the shape.
#pragma once
#include <hip/hip_runtime.h>

#include "fda_kernels.hpp"

namespace fda {
// Worker slots KC in kKCSet, row slots LR in 1..kMaxLR, KC * LR <= max_slots(KC): what the registers hold (fp32 slabs, with
// the library's own compiler options: 4 x 9 and 6 x 5 take 251 of 256, 6 x 6 would spill; 8 x 4 spills 50 to 54).  Nine rows in one workgroup instead of groups of five and four with six worker slots:
// 9 x 250, 30 x 7M fp32 378 -> 293 us a step, 8 x 40M bf16 553 -> 433.
// Kernels with sign-split LDS rows exist for the even KC, kernels with plain rows for KC <= 2 (with
// more slots, half the slots per workgroup and split rows need the same LDS and less work).
constexpr int kKCSet[] = {1, 2, 4, 6, 8};
constexpr int max_slots(int KC) { return KC == 4 ? 36 : 32; }
constexpr bool narrow_kernel_exists(int KC, bool split) { return split ? KC % 2 == 0 : KC <= 2; }
// ... and kernels for a table with placed rows (fields of kPlacedFieldBits bits) for the even KC: there a
// field is a bucket number in a whole group of rows
constexpr bool placed_kernel_exists(int KC) { return KC % 2 == 0; }

// FB: bits per field of the tabulated hash (field_bits_for(m): 11 or 16; kPlacedFieldBits with placed rows); split: sign-split LDS rows
// (even worker-slot counts only)
#define FDA_NARROW_LAUNCHER(t, kc) \
  hipError_t launch_narrow_##t##_kc##kc(int LR, int FB, int split, const StateParams* prm, size_t lds, hipStream_t st)
FDA_NARROW_LAUNCHER(f32, 1); FDA_NARROW_LAUNCHER(f32, 2); FDA_NARROW_LAUNCHER(f32, 4);
FDA_NARROW_LAUNCHER(f32, 6); FDA_NARROW_LAUNCHER(f32, 8);
FDA_NARROW_LAUNCHER(bf16, 1); FDA_NARROW_LAUNCHER(bf16, 2); FDA_NARROW_LAUNCHER(bf16, 4);
FDA_NARROW_LAUNCHER(bf16, 6); FDA_NARROW_LAUNCHER(bf16, 8);

template <typename T, int KC, int LR, int FB, bool SPLIT = false, bool SKETCH = true>
hipError_t launch_state_kernel(const StateParams* prm, size_t lds, hipStream_t st) {
  auto kern = state_kernel<T, KC, LR, FB, SPLIT, SKETCH>;
  if (prm == nullptr)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(prm->G * prm->R * prm->P), dim3(kStateThreads), lds, st, *prm);
  return hipGetLastError();
}
}  // namespace fda
