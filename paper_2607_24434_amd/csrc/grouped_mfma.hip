// The grouped gate/up and down launches of a block of positions on the matrix
// cores (bf16 and Q4_0 weights); mfma_core.h holds the passes.
#include "mfma_core.h"

namespace de {
namespace {

template <typename WT, int KS, bool GATEUP, bool REREAD>
__global__ __launch_bounds__(kBlock, 2) void grouped_mfma_kernel(GroupedArgs a) {
  const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
  __shared__ int s_absent, s_nms;
  const MfmaTables mt = mfma_tables<WT, KS, GATEUP>(a, lane, wave, &s_absent, &s_nms);
  if constexpr (!GATEUP) {
    if (s_absent && !a.r.absent_ok) absent_rows_zero(a, mt.tb, mt.nu);
  }
  mfma_pass<WT, KS, GATEUP, REREAD>(a, 0, mt.tb, mt.slc, mt.nms, lane, wave);
}

// True when the blocks of a launch can be cut into one run per position group
// that reads the same rows at the same time through the same L2: workgroups go
// to the eight XCDs in turn, so a run is a multiple of eight blocks.  (Three
// groups would leave CUs idle: their weights pass the L2 by.)
bool shares_rows(const GroupedArgs& a, int cus) {
  const int G = a.geo.groups;
  return !a.has_routed && a.n_dense == 1 && G > 1 && cus % G == 0 && cus / G % 8 == 0 &&
         a.geo.ndt >= cus;
}

template <typename WT, int KS, bool GATEUP, bool REREAD = false>
hipError_t launch_ks(const GroupedArgs& a, int tiles, hipStream_t s) {
  if constexpr (!REREAD && !kQ4<WT>)
    if (shares_rows(a, dev_info().num_cus)) return launch_ks<WT, KS, GATEUP, true>(a, tiles, s);
  const auto kernel = grouped_mfma_kernel<WT, KS, GATEUP, REREAD>;
  const size_t lds = mfma_lds<WT, KS>(a);
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kernel), lds);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return note_hip(e);
  }
  const int cus = dev_info().num_cus;
  hipLaunchKernelGGL(kernel, dim3(tiles < cus ? tiles : cus), dim3(kBlock), lds, s, a);
  return note_hip(hipGetLastError());
}

template <typename WT, bool GATEUP>
hipError_t launch_typed(const GroupedArgs& in, hipStream_t s) {
  const GroupedArgs a = with_geometry<WT, GATEUP>(in);
  int K = GATEUP ? a.H : (a.has_routed ? a.r.inter : 0);
  if (!GATEUP)
    for (int i = 0; i < a.n_dense; ++i) K = a.dense[i].cw > K ? a.dense[i].cw : K;
  const int tiles =
      a.geo.ndt + (a.has_routed ? (a.r.max_union + a.r.pairs_max / kXP) * a.geo.tr : 0);
  if (tiles == 0) return hipSuccess;
  const int ks = cdiv(cdiv(K, 32), 1 << a.lkw);
  if (ks <= 2) return launch_ks<WT, 2, GATEUP>(a, tiles, s);
  if (ks <= 4) return launch_ks<WT, 4, GATEUP>(a, tiles, s);
  if (ks <= 6) return launch_ks<WT, 6, GATEUP>(a, tiles, s);
  if (ks <= 8) return launch_ks<WT, 8, GATEUP>(a, tiles, s);
  return note_hip(hipErrorInvalidValue);
}

template <bool GATEUP>
hipError_t launch_pass(const GroupedArgs& a, int wdtype, hipStream_t s) {
  if (wdtype == DE_Q4_0) return launch_typed<q4_t, GATEUP>(a, s);
  if (wdtype == DE_BF16) return launch_typed<uint16_t, GATEUP>(a, s);
  return note_hip(hipErrorInvalidValue);
}

}  // namespace

// The fewest column slices whose waves hold at most 8 steps each, then more
// (smaller tiles) while the rows make fewer tiles than the chip has CUs.
int mfma_lkw(int wdtype, bool gateup, int K, int rows) {
  const int per = wdtype == DE_Q4_0
                      ? (gateup ? group_rows<q4_t, true>() : group_rows<q4_t, false>())
                      : (gateup ? group_rows<uint16_t, true>() : group_rows<uint16_t, false>());
  const int S = (K + 31) / 32;
  int l = 0;
  while (l < 3 && cdiv(S, 1 << l) > 8) ++l;
  while (l < 3 && S >= (2 << l) && cdiv(rows, (kWavesPB >> l) * per) < dev_info().num_cus) ++l;
  return l;
}

bool mfma_fits(int wdtype, int T, int N, int k) {
  GroupedArgs a{};
  a.T = T;
  a.has_routed = a.fuse_route = 1;
  a.sel.k = k;
  a.sel.N = N;
  a.r.pairs_max = T * k;
  a.r.max_union = T * k < N ? T * k : N;
  const size_t lds = wdtype == DE_Q4_0 ? mfma_lds<q4_t, 8>(a) : mfma_lds<uint16_t, 8>(a);
  return lds <= (size_t)160 * 1024 - 256;
}

hipError_t launch_gateup_mfma(const GroupedArgs& a, int wdtype, hipStream_t s) {
  return launch_pass<true>(a, wdtype, s);
}
hipError_t launch_down_mfma(const GroupedArgs& a, int wdtype, hipStream_t s) {
  return launch_pass<false>(a, wdtype, s);
}

}  // namespace de
