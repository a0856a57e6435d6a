// WAVE8: 4-bit entries, 1 wave per individual.
#include "tabu_wave_kernel.h"

namespace dlm {

int launch_w4_1(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s) {
  return launch_w8_waves<4, 1>(a, pop, acap, lds, s);
}

}  // namespace dlm
