// The verify layer of a block of positions (Eq. 4 over the expert union of
// Eq. 2-3, with the shared path) in one launch: one block per CU runs the
// gate/up pass, the down pass and the combine of the separate launches, with
// two device-wide points between them.
//
// The passes are the functions of the separate launches (mfma_core.h) and the
// combine sums in theirs' order, so the results are bit-identical to theirs.
// The member tables stay in LDS from the gate/up pass to the down pass.
//
// What blocks hand on (A, the partials, the pairs' places) is stored and loaded at
// agent scope, past the XCDs' own L2 caches.  (With a cache-wide write-back and
// invalidation per block and point instead, a V2-Lite layer took 196 us at T = 2 and
// 270 at T = 9; now 63 and 136, the separate launches 59 and 127.)
//
// A block arrives at a point by storing (launch epoch, point) to its word and
// waits until no block's word is smaller.  The grid is one block per CU (each
// takes more than half of a CU's LDS), and the host sends no such launch beside
// another one whose blocks wait (nor into a graph, whose replays would find their
// own epoch in the words), so every block gets its CU; every wait is bounded in
// any case, and one that runs out records kStatusSyncTimeout.
#include "verify_fused.h"

#include <algorithm>

#include "mfma_core.h"

namespace de {
namespace {

constexpr int kFKS = kMfmaMaxK / 32 / kWavesPB;  // steps per wave: serves both passes
constexpr unsigned kSpinLimit = 1u << 20;         // polls before a wait gives up
constexpr int kVT = kCombThreads / kBlock;        // combine: virtual threads per thread

__device__ __forceinline__ void grid_point(const FusedArgs& f, unsigned n, int* s_abort) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's stores have completed
  __syncthreads();
  const uint64_t target = ((uint64_t)f.epoch << 32) | n;
  if (threadIdx.x == 0)
    __hip_atomic_store(f.flags + blockIdx.x, target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x < kWave && !*(volatile int*)s_abort) {
    bool ok = false;
    for (unsigned i = 0; i < kSpinLimit && !ok; ++i) {
      uint64_t mn = ~0ull;
      for (int j = threadIdx.x; j < (int)gridDim.x; j += kWave) {
        const uint64_t w =
            __hip_atomic_load(f.flags + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mn = w < mn ? w : mn;
      }
      ok = __builtin_amdgcn_ballot_w64(mn < target) == 0ull;
      if (!ok) __builtin_amdgcn_s_sleep(2);
    }
    if (!ok && threadIdx.x == 0) {
      *(volatile int*)s_abort = 1;
      __hip_atomic_fetch_or(f.status, kStatusSyncTimeout, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  asm volatile("" ::: "memory");
}

template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load((const DE_GLOBAL T*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The combine of position t, its kCombThreads threads played by kBlock (thread
// i as the virtual threads i + j kBlock): combine_row's element, summation
// and reduction order.
__device__ __forceinline__ void combine_position(const CombineArgs& a, int t, float* red) {
  const size_t rowoff = (size_t)t * a.H;
  float ss[kVT], v[kVT][kCombPer];
  const auto element = [&](int j, int i) {
    return (int)threadIdx.x + j * kBlock + i * kCombThreads;
  };
#pragma unroll
  for (int j = 0; j < kVT; ++j)
#pragma unroll
    for (int i = 0; i < kCombPer; ++i) {
      v[j][i] = 0.f;
      if (element(j, i) >= a.H) continue;
#pragma unroll
      for (int s = 0; s < 3; ++s)
        if (s < a.n_dense) v[j][i] += ld_agent(a.dense_p[s] + rowoff + element(j, i));
    }
  // Eight list entries' partials in flight at a time.
  for (int q0 = 0; q0 < a.kk; q0 += 8) {
    int pp[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      pp[q] = ld_agent(a.pair_pos + (size_t)t * a.kk + min(q0 + q, a.kk - 1));
#pragma unroll
    for (int j = 0; j < kVT; ++j)
#pragma unroll
      for (int i = 0; i < kCombPer; ++i) {
        const int h = element(j, i);
        if (h >= a.H) continue;
        float p[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool ok = q0 + q < a.kk && pp[q] >= 0 && pp[q] < a.pairs_max;
          p[q] = ok ? ld_agent(a.p_r + (size_t)pp[q] * a.H + h) : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool ok = q0 + q < a.kk && pp[q] >= 0 && pp[q] < a.pairs_max;
          if (ok) v[j][i] += p[q];
        }
      }
  }
#pragma unroll
  for (int j = 0; j < kVT; ++j) {
    ss[j] = 0.f;
#pragma unroll
    for (int i = 0; i < kCombPer; ++i) {
      const int h = element(j, i);
      if (h >= a.H) continue;
      if (a.residual) v[j][i] = a.residual[rowoff + h] + v[j][i];
      a.y[rowoff + h] = v[j][i];
      ss[j] = fmaf(v[j][i], v[j][i], ss[j]);
    }
  }
  if (a.normed == nullptr) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < kVT; ++j) {
    const float w = wave_sum(ss[j]);
    if (lane == 0) red[wave + j * kWavesPB] = w;
  }
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < kCombThreads / kWave; ++w) tot += red[w];
  const float r = 1.0f / sqrtf(tot / (float)a.H + a.eps);
#pragma unroll
  for (int j = 0; j < kVT; ++j)
#pragma unroll
    for (int i = 0; i < kCombPer; ++i) {
      const int h = (int)threadIdx.x + j * kBlock + i * kCombThreads;
      if (h < a.H) a.normed[rowoff + h] = v[j][i] * r;
    }
}

__global__ __launch_bounds__(kBlock, 2) void verify_fused_kernel(FusedArgs f) {
  const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
  __shared__ int s_abort, s_absent, s_nms;
  __shared__ float s_red[kCombThreads / kWave];
  if (threadIdx.x == 0) s_abort = 0;
  const MfmaTables mt =
      mfma_tables<uint16_t, kFKS, true, true>(f.gu, lane, wave, &s_absent, &s_nms);
  mfma_pass<uint16_t, kFKS, true, false, true>(f.gu, offsetof(FusedArgs, gu), mt.tb, mt.slc, mt.nms,
                                               lane, wave);
  grid_point(f, 1, &s_abort);
  if (s_absent) absent_rows_zero<true>(f.dn, mt.tb, mt.nu);
  mfma_pass<uint16_t, kFKS, false, false, true>(f.dn, offsetof(FusedArgs, dn), mt.tb, mt.slc,
                                                mt.nms, lane, wave);
  grid_point(f, 2, &s_abort);
  // Every block is past its work for the others: another stream's launch may follow.
  if (blockIdx.x == 0 && threadIdx.x == 0 && !*(volatile int*)&s_abort)
    __hip_atomic_store(f.done, f.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  for (int t = blockIdx.x; t < f.c.T; t += gridDim.x) {
    combine_position(f.c, t, s_red);
    __syncthreads();  // s_red is reused
  }
}

}  // namespace

hipError_t launch_verify_fused(const FusedArgs& f, hipStream_t s) {
  const size_t lds = std::max(mfma_lds<uint16_t, kFKS>(f.gu), (size_t)84 * 1024);
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(verify_fused_kernel), lds);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return note_hip(e);
  }
  FusedArgs a = f;
  a.gu = with_geometry<uint16_t, true>(f.gu);
  a.dn = with_geometry<uint16_t, false>(f.dn);
  hipLaunchKernelGGL(verify_fused_kernel, dim3(dev_info().num_cus), dim3(kBlock), lds, s, a);
  return note_hip(hipGetLastError());
}

}  // namespace de
