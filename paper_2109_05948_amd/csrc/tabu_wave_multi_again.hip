// WAVE8 of an uneven batch: reruns with 8-bit entries, 4 waves per individual.
#include "tabu_wave_multi.h"

namespace dlm {

int launch_multi_w8_again(const WaveDesc* descs, int ndesc, int items, size_t lds, hipStream_t s) {
  return launch_multi_w8<4, true>(descs, ndesc, 0, items, lds, s);
}

}  // namespace dlm
