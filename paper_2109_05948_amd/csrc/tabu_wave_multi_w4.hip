// WAVE8 of an uneven batch: 4 waves per individual.
#include "tabu_wave_multi.h"

namespace dlm {

int launch_multi_w8_4(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s) {
  return launch_multi_w8<4, false>(descs, ndesc, base, items, lds, s);
}

}  // namespace dlm
