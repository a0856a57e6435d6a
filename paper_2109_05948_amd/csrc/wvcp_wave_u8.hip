// The weighted search, one wave per individual, 8-bit gammas.
#include "wvcp_wave.h"

namespace dlm {

int launch_wvcp_wave8(const WvcpArgs& a, int pop, hipStream_t s) {
  return launch_wv_gamma<uint8_t>(a, pop, wv_layout((a.n + 63) / 64, a.k, (int)sizeof(uint8_t)).bytes, s);
}

}  // namespace dlm
