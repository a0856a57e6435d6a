// Launches of the WAVE8 search (tabu_wave.h): table entries of 4 or 8 bits,
// 1, 2 or 4 waves.  One translation unit each, so that their instances
// compile side by side.
#pragma once

#include "tabu_body.h"

namespace dlm {

// again (8 bits): null, or the start colourings for a second run of what 4-bit
// entries had no room for
int launch_w4_1(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w4_2(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w4_4(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s);
int launch_w8_1(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s, const int16_t* again);
int launch_w8_2(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s, const int16_t* again);
int launch_w8_4(const TabuArgs& a, int pop, int acap, size_t lds, hipStream_t s, const int16_t* again);

// One graph's share of an uneven batch on the WAVE8 search: items
// [first_item, first_item + pop) of the batch are its individuals.
struct WaveDesc {
  TabuArgs a;
  int16_t* start;  // pop * n: the start colourings, for a rerun
  int32_t first_item, pop, acap, instance;
};

// items [base, base + items) of descs[0 .. ndesc)
int launch_multi_w8_1(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s);
int launch_multi_w8_2(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s);
int launch_multi_w8_4(const WaveDesc* descs, int ndesc, int base, int items, size_t lds, hipStream_t s);

// items [0, items): those that 4-bit entries had no room for, with four waves
int launch_multi_w8_again(const WaveDesc* descs, int ndesc, int items, size_t lds, hipStream_t s);

// A CU hands out its LDS in granules: workgroups of 53,760 bytes fit three to
// a CU, workgroups of 53,776 two (timed with a kernel of fixed length; the
// occupancy query of the runtime does not know the granule).
constexpr int64_t kLdsGranule = 1280;

constexpr int64_t kW8SideMax = 16384;  // side-list entries of one individual
// ... beyond what a random start needs, where 8-bit entries would take over:
// thousands of entries that outgrew 4 bits are walked in every iteration
// before the LDS is full
constexpr int64_t kW4Spare = 256;

// How a graph's individuals are searched: entry width, waves per individual
// and the side-list entries a random start needs.
struct W8Pick {
  int bits, waves;
  int64_t side;
};

// whether the wave table holds an individual of an automatic call, and whether
// the 16-bit block table in LDS is the faster one for pop of them all the same
bool w8_auto(const dlm_graph* g, const dlm_tabu_params* p);
bool block_faster(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop);
W8Pick w8_pick(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop);
// the same with 8-bit entries, for what 4-bit ones have no room for; false if
// the LDS does not hold them
bool w8_pick_bytes(const dlm_graph* g, const dlm_tabu_params* p, int64_t pop, W8Pick& r);

}  // namespace dlm
