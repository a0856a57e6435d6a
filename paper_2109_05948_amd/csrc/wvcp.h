// Arguments of the weighted search, and the launches of its wave form
// (wvcp_wave.h), one translation unit per gamma width.
#pragma once

#include "dlm_common.h"

namespace dlm {

struct WvcpArgs {
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const int32_t* erow;
  const int32_t* weights;
  int16_t* colors;
  int32_t* best_legal;
  int64_t* stats;
  uint64_t* hash;
  Key key;
  int32_t n, k, T, R, ten_rand, frz, shift, ind_base, max_w, max_deg;
  const uint32_t* adj;  // adjacency bits (dlm_graph)
};

int launch_wvcp_wave8(const WvcpArgs& a, int pop, hipStream_t s);
int launch_wvcp_wave16(const WvcpArgs& a, int pop, hipStream_t s);

}  // namespace dlm
