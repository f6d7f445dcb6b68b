// Self-distillation signals as by-products of a verify pass (Section 3.3,
// Eqs. 6-10): the residual target from the layer's routed partials, and row
// divergences between target and draft distributions (router agreement,
// temperature-scaled logit KL, token cross entropy).
#include "de_common.h"

#include <climits>
#include <type_traits>

namespace de {
namespace {

constexpr int kResThreads = 256;

// m*[t] = sum_{j = 1 .. kk-1} P[pair_pos[t, j]]: the routed partials of
// position t without its top-1 expert's, in list order (entries outside the
// partial rows are skipped).  Grid (T, column chunks).
__global__ __launch_bounds__(kResThreads) void residual_kernel(ResidualArgs a) {
  const int t = blockIdx.x;
  const int h = blockIdx.y * kResThreads + threadIdx.x;
  if (h >= a.H) return;
  float m = 0.f;
  for (int j = 1; j < a.kk; ++j) {
    const int p = a.pair_pos[(size_t)t * a.kk + j];
    if (p >= 0 && p < a.pairs_max) m += a.p_r[(size_t)p * a.H + h];
  }
  a.out[(size_t)t * a.H + h] = m;
}

// Threads of a row's block, and the values of a row that a thread has in flight.
// One value at a time on 256 threads, each with a load and an exponential behind
// the last, a row of 102400 logits took 253 us (now 91).
constexpr int kKlWide = 1024, kKlNarrow = 256, kKlBatch = 8;
// The longest rows of the narrow block: the wide one has four times the waves but
// four times the partial results to merge.  us, narrow and wide, a row of softmax
// (three sums): 2048 11 and 22, 12288 28 and 30, 16384 35 and 32; of sigmoids (whose
// logarithms weigh more): 2056 27 and 28, 3072 34 and 33, 8192 78 and 59.
constexpr int kKlNarrowSoftmax = 12288, kKlNarrowSigmoid = 2560;

// Running (max, sum exp(v - max)).
struct Lse {
  float m, s;
};

// a with the values v (-inf adds nothing), rescaled once.
__device__ __forceinline__ Lse lse_add(Lse a, const float (&v)[kKlBatch]) {
  float m = a.m;
#pragma unroll
  for (int j = 0; j < kKlBatch; ++j) m = fmaxf(m, v[j]);
  float s = a.m == m ? a.s : a.s * expf(a.m - m);
#pragma unroll
  for (int j = 0; j < kKlBatch; ++j)
    s += v[j] == -INFINITY ? 0.f : (v[j] == m ? 1.f : expf(v[j] - m));
  return Lse{m, s};
}
// One value: one exponential.
__device__ __forceinline__ Lse lse_add(Lse a, const float (&v)[1]) {
  const float e = expf(-fabsf(v[0] - a.m));
  if (v[0] > a.m) return Lse{v[0], a.s * e + 1.f};
  if (v[0] != -INFINITY) a.s += v[0] == a.m ? 1.f : e;
  return a;
}

__device__ __forceinline__ Lse lse_merge(Lse a, Lse b) {
  if (b.s == 0.f) return a;
  if (a.s == 0.f) return b;
  const float m = fmaxf(a.m, b.m);
  return Lse{m, a.s * expf(a.m - m) + b.s * expf(b.m - m)};
}

__device__ __forceinline__ float lse_val(Lse a) { return a.m + logf(a.s); }

// log sigmoid(z) without overflow.
__device__ __forceinline__ float log_sigmoid(float z) {
  return z < 0.f ? z - log1pf(expf(z)) : -log1pf(expf(-z));
}

// Reduces v over the block with op (every thread receives the result); the
// members of V are floats.
template <int NTH, typename V, typename Op>
__device__ __forceinline__ V block_reduce(V v, V* red, Op op, V zero) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    V w;
    w = v;
    // Shuffle each float member.
    float* pv = reinterpret_cast<float*>(&w);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(V) / 4); ++i) pv[i] = __shfl_xor(pv[i], o, kWave);
    v = op(v, w);
  }
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  V t = zero;
  for (int w = 0; w < NTH / 64; ++w) t = op(t, red[w]);
  return t;
}

struct LseOp {
  __device__ Lse operator()(Lse a, Lse b) const { return lse_merge(a, b); }
};

struct Best {
  float v;
  float i;  // index as float bits (shuffled as a float)
};

// Larger value, then lower index; index INT_MAX marks "none".
struct BestOp {
  __device__ Best operator()(Best a, Best b) const {
    const int ia = __float_as_int(a.i), ib = __float_as_int(b.i);
    if (ib == INT_MAX) return a;
    if (ia == INT_MAX) return b;
    return (b.v > a.v || (b.v == a.v && ib < ia)) ? b : a;
  }
};

struct Sum {
  float s;
};
struct SumOp {
  __device__ Sum operator()(Sum a, Sum b) const { return Sum{a.s + b.s}; }
};

// One block per row r: a = target row, b = draft row (n values each).
// softmax mode (sigmoid == 0): p = softmax((a + bias) / tau), q likewise from
// b; kl = tau^2 KL(p || q).  sigmoid mode: p = sigmoid(a) normalised to sum
// one, q likewise; kl = KL(p || q).  ce (optional) = -log softmax(b + bias)
// at the argmax of a + bias (ties to the lower index).
template <int NTH>
__global__ __launch_bounds__(NTH) void rowkl_kernel(RowKlArgs a) {
  __shared__ Lse rl[NTH / 64];
  __shared__ Best rb[NTH / 64];
  __shared__ Sum rs[NTH / 64];
  const float* pa = a.a + (size_t)blockIdx.x * a.lda;
  const float* pb = a.b + (size_t)blockIdx.x * a.ldb;
  const float it = 1.f / a.tau;
  Lse la{-INFINITY, 0.f}, lb{-INFINITY, 0.f}, lb1{-INFINITY, 0.f};
  Best best{-INFINITY, __int_as_float(INT_MAX)};
  // A thread's B values from i0 on: a + bias and b + bias (sigmoid: log sigmoid of a
  // and b in x and y, and a + bias in c).  All of them exist.
  const auto load = [&](auto& x, auto& y, auto& c, int i0) __attribute__((always_inline)) {
    constexpr int B = sizeof(x) / sizeof(float);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int i = i0 + j * NTH;
      c[j] = a.bias ? a.bias[i] : 0.f;
      x[j] = pa[i];
      y[j] = pb[i];
    }
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const float bias = c[j];
      c[j] = x[j] + bias;
      x[j] = a.sigmoid ? log_sigmoid(x[j]) : c[j];
      y[j] = a.sigmoid ? log_sigmoid(y[j]) : y[j] + bias;
    }
  };
  const auto add = [&](auto b, int i0) __attribute__((always_inline)) {
    constexpr int B = decltype(b)::value;
    float x[B], y[B], c[B];
    load(x, y, c, i0);
    if (!a.sigmoid) lb1 = lse_add(lb1, y);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      // Argmax of a + bias; a NaN counts as -infinity, as in the argmax.
      const float vc = c[j] == c[j] ? c[j] : -INFINITY;
      if (__float_as_int(best.i) == INT_MAX || vc > best.v)
        best = Best{vc, __int_as_float(i0 + j * NTH)};
      if (!a.sigmoid) {
        x[j] *= it;
        y[j] *= it;
      }
    }
    la = lse_add(la, x);
    lb = lse_add(lb, y);
  };
  float lsa = 0.f, lsb = 0.f, acc = 0.f;
  const auto divergence = [&](auto b, int i0) __attribute__((always_inline)) {
    constexpr int B = decltype(b)::value;
    float x[B], y[B], c[B];
    load(x, y, c, i0);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const float xa = (a.sigmoid ? x[j] : x[j] * it) - lsa;
      const float xb = (a.sigmoid ? y[j] : y[j] * it) - lsb;
      acc += expf(xa) * (xa - xb);
    }
  };
  // The row: whole batches of the block, then what is left value by value (a router's
  // row is all of that: a padded batch, or code unrolled for one, costs it 1 to 10 us).
  const auto sweep = [&](const auto& f) __attribute__((always_inline)) {
    constexpr int kStep = NTH * kKlBatch;
    const int whole = a.n / kStep * kStep;
#pragma unroll 1
    for (int i0 = threadIdx.x; i0 < whole; i0 += kStep)
      f(std::integral_constant<int, kKlBatch>{}, i0);
#pragma unroll 1
    for (int i0 = whole + threadIdx.x; i0 < a.n; i0 += NTH) f(std::integral_constant<int, 1>{}, i0);
  };
  sweep(add);
  la = block_reduce<NTH>(la, rl, LseOp{}, Lse{-INFINITY, 0.f});
  lb = block_reduce<NTH>(lb, rl, LseOp{}, Lse{-INFINITY, 0.f});
  lb1 = block_reduce<NTH>(lb1, rl, LseOp{}, Lse{-INFINITY, 0.f});
  best = block_reduce<NTH>(best, rb, BestOp{}, Best{-INFINITY, __int_as_float(INT_MAX)});
  lsa = lse_val(la);
  lsb = lse_val(lb);
  sweep(divergence);
  const Sum tot = block_reduce<NTH>(Sum{acc}, rs, SumOp{}, Sum{0.f});
  if (threadIdx.x == 0) {
    a.kl[blockIdx.x] = a.sigmoid ? tot.s : a.tau * a.tau * tot.s;
    if (a.ce != nullptr) {
      const int t = __float_as_int(best.i);
      const float bias = (a.bias && t != INT_MAX) ? a.bias[t] : 0.f;
      a.ce[blockIdx.x] = t == INT_MAX ? __int_as_float(0x7fc00000)
                                      : lse_val(lb1) - (pb[t] + bias);
    }
  }
}

}  // namespace

hipError_t launch_residual(const ResidualArgs& a, hipStream_t s) {
  const dim3 grid(a.T, (a.H + kResThreads - 1) / kResThreads);
  hipLaunchKernelGGL(residual_kernel, grid, dim3(kResThreads), 0, s, a);
  return note_hip(hipGetLastError());
}

hipError_t launch_rowkl(const RowKlArgs& a, hipStream_t s) {
  if (a.n <= (a.sigmoid ? kKlNarrowSigmoid : kKlNarrowSoftmax))
    hipLaunchKernelGGL(rowkl_kernel<kKlNarrow>, dim3(a.rows), dim3(kKlNarrow), 0, s, a);
  else
    hipLaunchKernelGGL(rowkl_kernel<kKlWide>, dim3(a.rows), dim3(kKlWide), 0, s, a);
  return note_hip(hipGetLastError());
}

}  // namespace de
