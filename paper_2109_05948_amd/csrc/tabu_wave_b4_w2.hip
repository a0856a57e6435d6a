// WAVE8: 4-bit entries, 2 waves per individual.
#include "tabu_wave_kernel.h"

namespace dlm {

int launch_w4_2(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s) {
  return launch_w8_waves<4, 2>(a, pop, acap, lds, s);
}

}  // namespace dlm
