// The weighted search, one wave per individual, 16-bit gammas.
#include "wvcp_wave.h"

namespace dlm {

int launch_wvcp_wave16(const WvcpArgs& a, int pop, hipStream_t s) {
  return launch_wv_gamma<uint16_t>(a, pop, wv_layout((a.n + 63) / 64, a.k, (int)sizeof(uint16_t)).bytes, s);
}

}  // namespace dlm
