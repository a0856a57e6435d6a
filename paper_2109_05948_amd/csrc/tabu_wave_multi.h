// Uneven batches on the WAVE8 search: one workgroup per (graph, individual)
// pair, one launch per number of waves.
#pragma once

#include "tabu_wave.h"
#include "tabu_wave_launch.h"

namespace dlm {

// Row widths an instance serves: RW dwords read, RLO..RW dwords long.  A few
// coarser ones than the single-graph launch's beyond 8 dwords; with only 4, 8,
// 12, ... a batch of 9 graphs of 85 to 257 vertices took 10.4 ms instead of 9.9.
#define DLM_W8_MULTI(X) \
  X(0, 4, 1, 1) \
  X(1, 4, 2, 2) \
  X(2, 4, 3, 3) \
  X(3, 4, 4, 4) \
  X(4, 4, 5, 5) \
  X(5, 4, 6, 6) \
  X(6, 4, 7, 7) \
  X(7, 4, 8, 8) \
  X(8, 4, 10, 9) \
  X(9, 4, 12, 11) \
  X(10, 4, 16, 13) \
  X(11, 4, 20, 17) \
  X(12, 4, 24, 21) \
  X(13, 4, 32, 25) \
  X(14, 8, 4, 1) \
  X(15, 8, 8, 5) \
  X(16, 8, 12, 9) \
  X(17, 8, 16, 13) \
  X(18, 8, 24, 17) \
  X(19, 8, 32, 25) \
  X(20, 8, 64, 33)

// instance of a row of k entries, or -1
inline int w8_multi_instance(int k, int bits) {
  const int w = w8_row_dwords(k, bits);
#define DLM_X(I, BITS, RW, RLO) \
  if (bits == BITS && w >= RLO && w <= RW) return I;
  DLM_W8_MULTI(DLM_X)
#undef DLM_X
  return -1;
}

// Items are ordered longest first, so that the long chains start at once: a
// batch lasts as long as its longest individual if the card holds them all.
// AGAIN: only the individuals that 4-bit entries had no room for, from their
// saved start (their descriptors here have 8-bit instances).
template <int NW, bool AGAIN>
__global__ __launch_bounds__(64 * NW) void tabu_multi_w8_kernel(const WaveDesc* __restrict__ descs, int32_t ndesc,
                                                                int32_t base) {
  extern __shared__ __align__(16) unsigned char smem[];
  typedef const __attribute__((address_space(4))) uint32_t* words;
  const int32_t item = base + (int32_t)blockIdx.x;
  int g = 0;
  while (g + 1 < ndesc && descs[g + 1].first_item <= item) ++g;
  g = (int)rfl((uint32_t)g);
  // the descriptor by scalar loads, whatever the search has stored before
  const uint64_t at = own_u64((uint64_t)(descs + g));
  WaveDesc d;
  static_assert(sizeof(WaveDesc) % 4 == 0, "read in words");
#pragma unroll
  for (size_t i = 0; i < sizeof(WaveDesc) / 4; ++i) reinterpret_cast<uint32_t*>(&d)[i] = ((words)at)[i];
  const int li = item - d.first_item;
  // the start waits for a rerun, or this is one
  if (AGAIN && (int)rfl((uint32_t)d.a.iters[li]) != kW8GaveUp) return;
  {
    const size_t row = (size_t)li * (size_t)d.a.n;
    for (int v = threadIdx.x; v < d.a.n; v += 64 * NW) {
      if (AGAIN)
        d.a.colors[row + v] = d.start[row + v];
      else
        d.start[row + v] = d.a.colors[row + v];
    }
  }
  auto late = [at] { return (const TabuArgs*)own_u64(at); };  // a is the descriptor's first member
  switch (d.instance) {
#define DLM_X(I, BITS, RW, RLO)                                           \
  case I:                                                                 \
    if constexpr (!AGAIN || BITS == 8)                                    \
      tabu_w8_individual<BITS, NW, RW, RLO>(d.a, li, d.acap, smem, late); \
    break;
    DLM_W8_MULTI(DLM_X)
#undef DLM_X
  }
}

template <int NW, bool AGAIN>
static int launch_multi_w8(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s) {
  auto kern = tabu_multi_w8_kernel<NW, AGAIN>;
  DLM_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kern, dim3(items), dim3(64 * NW), lds, s, descs, ndesc, base);
  DLM_HIP(hipGetLastError());
  return DLM_OK;
}

}  // namespace dlm
