// WAVE8: 8-bit entries, 4 waves per individual.
#include "tabu_wave_kernel.h"

namespace dlm {

int launch_w8_4(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s, const int16_t* again) {
  return launch_w8_waves<8, 4>(a, pop, acap, lds, s, again);
}

}  // namespace dlm
