// Launches of the WAVE8 search (tabu_wave.h): table entries of 4 or 8 bits,
// 1, 2 or 4 waves.  One translation unit each, so that their instances
// compile side by side.
#pragma once

#include "tabu_body.h"

namespace dlm {

int launch_w4_1(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w4_2(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w4_4(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w8_1(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w8_2(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w8_4(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);

}  // namespace dlm
