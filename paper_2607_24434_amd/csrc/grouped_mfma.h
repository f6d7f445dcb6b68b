// The grouped passes on the matrix cores: launchers (internal).
#pragma once

#include "de_common.h"

namespace de {

// Largest number of columns (reduction length) of a source.
constexpr int kMfmaMaxK = 2048;

// log2 of the column slices of a pass over sources of at most K columns and
// `rows` rows in all (gate/up: (G, U) row pairs).
int mfma_lkw(int wdtype, bool gateup, int K, int rows);

// True when a layer's tables (T positions, top k of N experts) fit a block's
// LDS beside the staged weights and the partials.
bool mfma_fits(int wdtype, int T, int N, int k);

// DE_BF16 or DE_Q4_0 weights; GroupedArgs::lkw set, every source's columns (a
// down source's: cw) a multiple of 8 (32) and at most kMfmaMaxK.
hipError_t launch_gateup_mfma(const GroupedArgs& a, int wdtype, hipStream_t s);
hipError_t launch_down_mfma(const GroupedArgs& a, int wdtype, hipStream_t s);

}  // namespace de
