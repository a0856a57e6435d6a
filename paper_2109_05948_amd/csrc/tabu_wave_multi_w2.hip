// WAVE8 of an uneven batch: 2 waves per individual.
#include "tabu_wave_multi.h"

namespace dlm {

int launch_multi_w8_2(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s) {
  return launch_multi_w8<2, false>(descs, ndesc, base, items, lds, s);
}

}  // namespace dlm
