// Top-k selection with gates (Eq. 1, Eq. 4) and the block union with
// per-expert position lists (Eq. 2, Eq. 3), as device functions over LDS
// arrays.  The routing launch selects; the union kernel and the prologue of
// the grouped gate/up kernel (in every block, from the selected lists) build
// the union.
//
// Selection: one wave per position, k rounds of a wave-wide argmax (largest
// key, ties to the lower id).  Gates are normalised in list order.  It runs in
// the prologue of every gate/up block, so its latency is the layer's: with up
// to 64 experts a lane holds one candidate and a round is one wave max of
// whole numbers and one ballot (with four float candidates per lane and a wave
// min for the id, two positions took 2.8 us).
//
// Union: integer work only.  Every (position, slot) entry sets its position
// bit in the expert's 64-bit mask with an LDS atomic OR (a bit already set
// means the id repeats within a position); a wave scan over the experts in
// ascending id gives each member's list offset and union index; the rank of
// a position in its expert's list is the popcount of the mask below it.
#pragma once

#include "de_common.h"

#include <climits>

namespace de {

// LDS arrays of the selection and union (sizes: T*k, T*k, N, N, N, 4), the masks
// first: behind the lists, at an odd multiple of 8 bytes, a layer of five positions and
// 22 us took 0.1 us more.
struct SelView {
  int32_t* idx;              // ordered top-k ids [T, k]
  float* gate;               // their gates
  unsigned long long* mask;  // position mask per expert [N]
  int32_t* off;              // list offset per expert
  int32_t* upos;             // union index per expert
  int32_t* misc;             // [0] bad, [1] n_union, [2] pairs
};

__host__ __device__ inline size_t sel_view_bytes(int T, int k, int N) {
  const size_t tk = (size_t)T * k;
  return tk * 8 + (size_t)N * 16 + 16;
}

__device__ inline SelView sel_view_at(char* p, int T, int k, int N) {
  SelView v;
  const size_t tk = (size_t)T * k;
  v.mask = reinterpret_cast<unsigned long long*>(p);
  v.off = reinterpret_cast<int32_t*>(v.mask + N);
  v.upos = v.off + N;
  v.misc = v.upos + N;
  v.idx = v.misc + 4;
  v.gate = reinterpret_cast<float*>(v.idx + tk);
  return v;
}

// Loads a position's N logits into the lane layout of the selection: lane l
// holds candidates l, l + 64, ... (N <= 256; zrow in LDS or global memory).
__device__ __forceinline__ void topk_load(const TopkUnionArgs& a, const float* zrow,
                                          float (&z)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = lane + q * kWave;
    z[q] = e < a.N ? zrow[e] : 0.f;
  }
}

// Inclusive sum over the lanes of a wave (no LDS): four shifts inside the
// 16-lane rows, then the rows' totals.
__device__ __forceinline__ int wave_scan_i32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// Set bits of `mask` below the lane.
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Largest value of a wave (0: smaller than every key).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  int v = (int)x;
  const auto mx = [](int p, int q) { return (int)max((uint32_t)p, (uint32_t)q); };
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));
  v = mx(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}

// Order-preserving whole number of a selection key, never 0; -0 and 0 are the
// same key, a NaN counts as -inf.
__device__ __forceinline__ uint32_t key_bits(float v) {
  if (!(v == v)) v = -INFINITY;
  const uint32_t u = __float_as_uint(v + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Ordered top-k of R positions at once from their logits in registers (R
// independent chains interleaved, so their latencies overlap), for
// N <= 64 NQ: lane j < k receives entry j's id and score.  Each of the k
// rounds takes the largest remaining key, ties to the lower id: a wave max
// finds the key and ballots find who holds it (candidate q of lane l is expert
// l + 64 q, so the first set bit of the first ballot is the lowest id).  A
// candidate id >= N never competes.  With a.rounds set, only that many leading
// entries are selected.  first(id): called once the leading entry is known
// (R = 1).  One wave.
template <int R, int NQ, class First>
__device__ __forceinline__ void topk_rounds(const TopkUnionArgs& a, const float (&z)[R][4],
                                            int (&id)[R], float (&sv)[R], const First& first) {
  const int lane = threadIdx.x & 63;
  const int N = a.N, k = a.k;
  float key[R][NQ], sc[R][NQ];
  uint32_t kb[R][NQ];  // the remaining candidates' keys; 0: none
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = lane + q * kWave;
      const float b = (e < N && a.bias != nullptr) ? a.bias[e] : 0.f;
      float kk;
      if (a.score_func == 0) {  // softmax(z + b): key z + b
        kk = z[r][q] + b;
        sc[r][q] = 0.f;
      } else {                  // sigmoid(z): key sigmoid(z) + b
        sc[r][q] = 1.0f / (1.0f + expf(-z[r][q]));
        kk = sc[r][q] + b;
      }
      if (!(kk == kk)) kk = -INFINITY;  // a NaN never wins
      key[r][q] = e < N ? kk : -INFINITY;
      kb[r][q] = e < N ? key_bits(kk) : 0u;
    }
    id[r] = 0;
  }
  float top[R];  // the largest key
  const int kr = a.rounds > 0 ? min(a.rounds, k) : k;
  for (int j = 0; j < kr; ++j) {
    uint32_t m[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      m[r] = kb[r][0];
#pragma unroll
      for (int q = 1; q < NQ; ++q) m[r] = max(m[r], kb[r][q]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) m[r] = wave_max_u32(m[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int win = 0;
#pragma unroll
      for (int q = NQ - 1; q >= 0; --q) {
        const unsigned long long b = __builtin_amdgcn_ballot_w64(kb[r][q] == m[r]);
        if (b != 0ull) win = q * kWave + (int)__builtin_ctzll(b);
      }
      if (j == 0) {
        first(win);
        const uint32_t u = (m[r] & 0x80000000u) ? (m[r] & 0x7fffffffu) : ~m[r];
        top[r] = __uint_as_float(u);
      }
      if (lane == j) id[r] = win;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (lane + q * kWave == win) kb[r][q] = 0u;
    }
  }
  if (a.score_func == 0) {
    float ex[R][NQ], sum[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      sum[r] = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        ex[r][q] = lane + q * kWave < N ? expf(key[r][q] - top[r]) : 0.f;
        sum[r] += ex[r][q];
      }
    }
    // (Candidates that no lane holds add zeros, as every NQ does.)
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] = wave_sum(sum[r]);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < NQ; ++q) sc[r][q] = ex[r][q] / sum[r];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    sv[r] = 0.f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float s = __shfl(sc[r][q], id[r] & 63, kWave);
      if (id[r] >> 6 == q) sv[r] = s;
    }
  }
}

struct NoFirst {
  __device__ __forceinline__ void operator()(int) const {}
};

template <int R, class First = NoFirst>
__device__ __forceinline__ void topk_regs(const TopkUnionArgs& a, const float (&z)[R][4],
                                          int (&id)[R], float (&sv)[R],
                                          const First& first = First()) {
  if (a.N <= kWave)
    topk_rounds<R, 1>(a, z, id, sv, first);
  else
    topk_rounds<R, 4>(a, z, id, sv, first);
}

// Gate of list entry `lane` of a position from the list's scores (lane j:
// entry j): score (/ sum of the k scores in list order) * routed_scale.
__device__ __forceinline__ float topk_gate(const TopkUnionArgs& a, float sv) {
  float g = sv;
  if (a.norm_topk) {
    float gsum = 0.f;
    for (int i = 0; i < a.k; ++i)
      gsum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sv), i));
    g = g / gsum;
  }
  return g * a.routed_scale;
}

// Union of the first a.ucols entries of every position's list in s.idx /
// s.gate.  s.misc[1] receives n_union (-1 for an id outside [0, N) or an id
// that repeats within a position) and s.misc[2] the number of pairs; the lists go
// to a.n_union / union_ids / offsets / tok_list / gate_list / pair_pos.  All
// threads of the block; ends with a barrier.
__device__ inline void build_union(const TopkUnionArgs& a, const SelView& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nthreads = blockDim.x;
  const int T = a.T, N = a.N, k = a.k, uc = a.ucols;
  for (int e = tid; e < N; e += nthreads) s.mask[e] = 0ull;
  if (tid == 0) s.misc[0] = 0;
  __syncthreads();
  for (int i = tid; i < T * uc; i += nthreads) {
    const int t = i / uc, j = i - t * uc;
    const int e = s.idx[t * k + j];
    if (e < 0 || e >= N) {
      s.misc[0] = 1;
    } else {
      const unsigned long long bit = 1ull << t;
      const unsigned long long old = atomicOr(&s.mask[e], bit);
      if (old & bit) s.misc[0] = 1;
    }
  }
  __syncthreads();
  if (s.misc[0]) {
    if (tid == 0) {
      s.misc[1] = -1;
      s.misc[2] = 0;
      *a.n_union = -1;
    }
    __syncthreads();
    return;
  }
  // Exclusive scans over the experts in ascending id (wave 0, four per lane).
  if (wave == 0) {
    int cnt[4], flg[4], csum = 0, fsum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane * 4 + q;
      const unsigned long long m = e < N ? s.mask[e] : 0ull;
      cnt[q] = __popcll(m);
      flg[q] = m != 0ull;
      csum += cnt[q];
      fsum += flg[q];
    }
    int ci = csum, fi = fsum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int cu = __shfl_up(ci, o, kWave);
      const int fu = __shfl_up(fi, o, kWave);
      if (lane >= o) {
        ci += cu;
        fi += fu;
      }
    }
    int cbase = ci - csum, fbase = fi - fsum;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = lane * 4 + q;
      if (e < N) {
        s.off[e] = cbase;
        s.upos[e] = fbase;
      }
      cbase += cnt[q];
      fbase += flg[q];
    }
    if (lane == kWave - 1) {
      s.misc[1] = fi;
      s.misc[2] = ci;
    }
  }
  __syncthreads();
  const int nu = s.misc[1], total = s.misc[2];
  for (int e = tid; e < N; e += nthreads) {
    if (s.mask[e] != 0ull) {
      a.union_ids[s.upos[e]] = e;
      a.offsets[s.upos[e]] = s.off[e];
    }
  }
  for (int u = nu + tid; u < N; u += nthreads) a.union_ids[u] = -1;
  for (int u = nu + tid; u <= N; u += nthreads) a.offsets[u] = total;
  if (tid == 0) *a.n_union = nu;
  for (int i = tid; i < T * uc; i += nthreads) {
    const int t = i / uc, j = i - t * uc;
    const int e = s.idx[t * k + j];
    const unsigned long long below = t == 0 ? 0ull : (s.mask[e] & (~0ull >> (64 - t)));
    const int p = s.off[e] + __popcll(below);
    a.tok_list[p] = t;
    a.gate_list[p] = s.gate[t * k + j];
    a.pair_pos[i] = p;
  }
  __syncthreads();
}

// Router logit of one expert (Eq. 1) by one wave: the dot product of the
// expert's fp32 router row w (H4 float4s) with x (xf(h) returns float4 h of
// the position's input), lane-strided in chunks of 8 float4 per lane whose
// loads are in flight together, then summed over the wave.  Every lane
// receives the same bits, whichever memory xf reads.
template <typename XF>
__device__ __forceinline__ float router_dot(const float4* w, int H4, int lane, XF xf) {
  float acc = 0.f;
  for (int h0 = 0; h0 < H4; h0 += kWave * 8) {
    float4 v0[8], xv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int h = min(h0 + lane + j * kWave, H4 - 1);  // clamped: in bounds, skipped below
      v0[j] = w[h];
      xv[j] = xf(h);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (h0 + lane + j * kWave < H4) {
        acc = fmaf(v0[j].x, xv[j].x, acc);
        acc = fmaf(v0[j].y, xv[j].y, acc);
        acc = fmaf(v0[j].z, xv[j].z, acc);
        acc = fmaf(v0[j].w, xv[j].w, acc);
      }
    }
  }
  return wave_sum(acc);
}

// router_dot for rows of at most kWave * 8 float4 (H <= 2048) with the row
// already loaded (w[j] = float4 lane + j * kWave, clamped as in router_dot):
// the same arithmetic, so the same bits.
template <typename XF>
__device__ __forceinline__ float router_dot_pre(const float4 (&w)[8], int H4, int lane, XF xf) {
  float acc = 0.f;
  float4 xv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) xv[j] = xf(min(lane + j * kWave, H4 - 1));
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (lane + j * kWave < H4) {
      acc = fmaf(w[j].x, xv[j].x, acc);
      acc = fmaf(w[j].y, xv[j].y, acc);
      acc = fmaf(w[j].z, xv[j].z, acc);
      acc = fmaf(w[j].w, xv[j].w, acc);
    }
  }
  return wave_sum(acc);
}

}  // namespace de
