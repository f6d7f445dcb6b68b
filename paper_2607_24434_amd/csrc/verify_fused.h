// The verify layer in one launch: argument block and launcher (internal).
#pragma once

#include "de_common.h"

namespace de {

struct FusedArgs {
  GroupedArgs gu;      // the gate/up launch's arguments (fused selection and union)
  GroupedArgs dn;      // the down launch's
  CombineArgs c;       // the combine's
  uint64_t* flags;     // [grid] arrival words, never decreasing
  uint32_t epoch;      // this launch's; the words of earlier launches are smaller
  int32_t* status;     // device status word
  uint32_t* done;      // host word that receives the epoch once no block waits any more
};

// Blocks of 2 to 9 positions of a matrix-core layer (a draft of up to eight tokens).
// It is slower than the separate launches at every one of them (V2-Lite layer, us:
// T = 2 63 against 59, T = 5 99 against 93, T = 9 136 against 127), so longer blocks
// are not served.
constexpr int kVerifyFusedMinT = 2, kVerifyFusedMaxT = 9;

hipError_t launch_verify_fused(const FusedArgs& f, hipStream_t s);

// Host side (api.cpp): true only when DE_VERIFY_FUSED is "1".
bool verify_fused_enabled();

}  // namespace de
