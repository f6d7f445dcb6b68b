// The grouped passes on the matrix cores: launchers (internal).
#pragma once

#include "de_common.h"

namespace de {

// Largest number of columns (reduction length) of a source.
constexpr int kMfmaMaxK = 2048;

// log2 of the column slices of a pass over sources of at most K columns and
// `rows` rows in all (gate/up: (G, U) row pairs), `per` rows per row group
// of a tile (16 gate/up pairs, 32 down rows).
int mfma_lkw(int K, int rows, int per);

// True when a layer's tables (T positions, top k of N experts) fit a block's
// LDS beside the staged weights and the partials.
bool mfma_fits(int T, int N, int k);

// GroupedArgs::lkw set, every source's columns a multiple of 8 and at most
// kMfmaMaxK.
hipError_t launch_gateup_mfma(const GroupedArgs& a, hipStream_t s);
hipError_t launch_down_mfma(const GroupedArgs& a, hipStream_t s);

}  // namespace de
