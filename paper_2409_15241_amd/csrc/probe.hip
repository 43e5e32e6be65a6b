// MFMA-only probe: what the matrix pipes of this chip sustain on the layer's kind of data when nothing else
// competes (no LDS, no memory traffic).  Under matrix load the clock is power-limited and depends on how many
// operand bits toggle, so the figure is measured on caller-provided fragments, not taken from the data sheet.
#include "probe.h"
#include <type_traits>
#include "common.h"

namespace {

// Every wave issues iters x 8 x 16384 multiply-adds back to back on one A and one B fragment per lane, read once from memory:
// 8 MFMAs 32x32x16 or 16 of 16x16x32 on as many independent accumulators.  The 16x16x32 form, which the products are
// made of, reads and writes half the accumulator bytes per flop.
template <bool WIDE>
__global__ __launch_bounds__(256)
void mfma_probe_kernel(const bf16x8* __restrict__ a, const bf16x8* __restrict__ b, float* __restrict__ out, int iters) {
  constexpr int N = WIDE ? 8 : 16, V = WIDE ? 16 : 4;
  using acc_t = std::conditional_t<WIDE, f32x16, f32x4>;
  const bf16x8 fa = a[threadIdx.x], fb = b[threadIdx.x];
  acc_t c[N];
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int v = 0; v < V; ++v) c[j][v] = 0.0f;
  for (int it = 0; it < iters; ++it)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if constexpr (WIDE) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, c[j], 0, 0, 0);
      else c[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, c[j], 0, 0, 0);
    }
  float t = 0.0f;
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int v = 0; v < V; ++v) t += c[j][v];
  out[(long)blockIdx.x * 256 + threadIdx.x] = t;
}

}  // namespace

hipError_t mfma_probe_launch(int shape, const void* a, const void* b, float* out, int blocks, int iters, hipStream_t st) {
  auto kern = shape == MFMA_PROBE_32x32x16 ? mfma_probe_kernel<true> : mfma_probe_kernel<false>;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, st, static_cast<const bf16x8*>(a), static_cast<const bf16x8*>(b), out, iters);
  return hipGetLastError();
}
