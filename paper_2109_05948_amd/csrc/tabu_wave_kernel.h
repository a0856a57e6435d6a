// The WAVE8 kernel and its dispatch over row widths, for one entry width and
// number of waves.
#pragma once

#include "tabu_wave.h"
#include "tabu_wave_launch.h"

namespace dlm {

// again: null, or the start colourings of a second run of those individuals
// that 4-bit entries had no room for.
template <int BITS, int NW, int RW>
__global__ __launch_bounds__(64 * NW) void tabucol_w8_kernel(TabuArgs a, int32_t acap, const int16_t* again) {
  extern __shared__ __align__(16) unsigned char smem[];
  if constexpr (BITS == 8) {
    if (again) {
      if ((int)rfl((uint32_t)a.iters[blockIdx.x]) != kW8GaveUp) return;
      const size_t row = (size_t)blockIdx.x * (size_t)a.n;
      for (int v = threadIdx.x; v < a.n; v += 64 * NW) a.colors[row + v] = again[row + v];
      __syncthreads();
    }
  }
  // dwords of a row that lie in it for every k of the bucket
  constexpr int RLO = RW <= 12 ? RW : RW == 16 ? 12 : RW == 24 ? 16 : RW == 32 ? 24 : 32;
  tabu_w8_individual<BITS, NW, RW, RLO>(a, blockIdx.x, acap, smem, [] { return late_args<TabuArgs>(); });
}

template <int BITS, int NW, int RW>
static int launch_w8_rows(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s, const int16_t* again) {
  auto kern = tabucol_w8_kernel<BITS, NW, RW>;
  DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kern, dim3(pop), dim3(64 * NW), lds, s, a, acap, again);
  DLM_HIP(hipGetLastError());
  return DLM_OK;
}

template <int BITS, int NW>
static int launch_w8_waves(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s,
                           const int16_t* again = nullptr) {
  switch (w8_bucket(a.k, BITS)) {
#define DLM_W8(RW) \
  case RW:         \
    return launch_w8_rows<BITS, NW, RW>(a, pop, acap, lds, s, again);
    DLM_W8(1) DLM_W8(2) DLM_W8(3) DLM_W8(4) DLM_W8(5) DLM_W8(6) DLM_W8(7) DLM_W8(8)
    DLM_W8(9) DLM_W8(10) DLM_W8(11) DLM_W8(12) DLM_W8(16) DLM_W8(24) DLM_W8(32)
    case 64:
      if constexpr (BITS == 8) return launch_w8_rows<BITS, NW, 64>(a, pop, acap, lds, s, again);
#undef DLM_W8
  }
  return set_error(DLM_E_UNSUPPORTED, "dlm_tabu_batch: k=%d too large for the wave table", a.k);
}

}  // namespace dlm
