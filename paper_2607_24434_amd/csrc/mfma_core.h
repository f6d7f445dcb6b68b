// The grouped gate/up and down passes of a block of positions on the matrix
// cores, for bf16 weights (the LM head's row-dot is a down pass of one
// source): the device functions of the separate launches and of the
// single-launch verify layer, which therefore write the same bits.
//
// Every weight byte meets |T_e| positions, so the passes should be bound by
// HBM; on the vector ALU each weight costs a conversion and one FMA per
// position, and the block's fp32 positions have to come from LDS.  Here
// v_mfma_f32_16x16x32_bf16 takes 16 positions x 32 columns against 32 columns
// x 16 weight rows, and the weights go from memory to the matrix cores as they
// are.
//
// fp32 activations: x = hi + mid + lo exactly, three bf16 values of 8 mantissa
// bits each (truncation splits), and every weight fragment meets all three, so
// each product is exact and only the order of the fp32 sums differs from the
// vector-ALU path.
//
// Split: a block is 8 waves, one block per CU.  The waves cut the columns
// into kw slices (kw = 8 for 2048 columns) and the block's rows into 8 / kw
// groups of 16 (gate/up: 16 (G, U) row pairs) or 32 (down).  A wave holds the
// activation fragments of its 256 columns and 16 positions in registers
// (3 x 32 VGPRs) for as long as the block stays with one expert, so the inner
// loop reads nothing but weights; its partial sums meet the other slices' in
// LDS once per tile.  Every step of 32 columns is summed from zero and added
// to the wave's sums, and the slices' sums are added last: against 64 bits the
// results are closer than the vector ALU's (V2-Lite LM head: 1.0e-7 against
// 1.2e-7 relative; one chain through all steps gave 1.7e-7).
//
// Streaming: what a load instruction covers decides the rate.  Loaded in
// operand order (16 rows x 64 bytes) a 461 MB stream ran at 4.2 to 4.8 TB/s,
// in runs of 512 bytes (2 rows) at 5.9 to 6.3, the same as linear reads.  So a
// wave loads its 16-row fragment in memory order into registers, puts it in
// its own LDS rows and reads it back in operand order (no block barrier; the
// LDS moves twice the weight bytes, a sixth of its rate).  The registers hold
// one fragment per wave (64 KB in flight per CU; two measured no faster) and
// each is refilled from the next fragment as soon as it is stored, across
// tiles and experts.  A block owns a contiguous range of the launch's tiles
// and meets one or two experts; the activations of the next expert are loaded
// the same way, into the registers of the step just finished, and are split
// when the step is used.
//
// Measured (rocprofv3, V2-Lite layer): T = 9 gate/up 82 us (vector ALU 88),
// down 42 (47); T = 17 99 (131) and 50 (80); T = 64 163 (554) and 79 (248);
// dense layer of 10944 at T = 9 21 and 15 (78 us with the combine before, 41
// now); LM head of 102400 at T = 9 72 (101).
//
// More than 16 positions are several slices of 16 over the same rows.  Blocks
// at the same place of two slices' ranges run side by side, so the second
// reading is served by the caches.
#pragma once

#include "grouped_core.h"
#include "grouped_mfma.h"
#include "topk_union.h"

namespace de {
namespace {

constexpr int kXP = 16;                       // positions per slice
constexpr int kRedLd = 20;                    // LDS partials: row stride (4 extra: no bank conflicts)
constexpr int kRedTile = kXP * kRedLd;        // one 16 x 16 tile of partials
constexpr int kRedBuf = kWavesPB * 2 * kRedTile;
constexpr int kRedFloats = 2 * kRedBuf;       // double buffered: one barrier per tile

// LDS of a wave's staged weight fragment: 16 rows of 4 KS units of 16 bytes,
// one unit of padding per row (no bank conflicts in the fragment reads).
template <int KS>
constexpr int kRowUnits = 4 * KS + 1;
template <int KS>
constexpr int kStageFloats = kWavesPB * 16 * kRowUnits<KS> * 4;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A slice: up to 16 positions against the rows of one source (the same in
// every lane).
struct Slice {
  const char* w;      // gate/up: G; down: the matrix
  int64_t w2;         // gate/up: bytes from a G row to its U row
  int rows, K;        // rows (gate/up: pairs), columns
  uint32_t rb;        // bytes per row
  const float* act;   // activations, row stride astride
  int astride;
  int nt, p0;         // positions, first output row
  int listed;         // gate/up of a member: activation rows come from the token list
  float* out;
  int ostride;
  int goff;           // down of a member: gate-list index of the first position; else -1
  float gscalar;
  int tiles;
};

typedef __attribute__((address_space(4))) const char kchar;

// Dense source s of the GroupedArgs at byte `arg` of the kernel arguments
// (uniform run-time index: scalar loads).
__device__ __forceinline__ DenseSrc dense_arg(int arg, int s) {
  kchar* p = (kchar*)__builtin_amdgcn_kernarg_segment_ptr() + arg + offsetof(GroupedArgs, dense) +
             (size_t)s * sizeof(DenseSrc);
  DenseSrc d{};
#define DE_KARG(f) d.f = *(__attribute__((address_space(4))) const decltype(d.f)*)(p + offsetof(DenseSrc, f))
  DE_KARG(w);
  DE_KARG(inter);
  DE_KARG(ld);
  DE_KARG(rows);
  DE_KARG(gate);
  DE_KARG(vin);
  DE_KARG(vin_stride);
  DE_KARG(out);
  DE_KARG(out_stride);
  DE_KARG(chunks);
  DE_KARG(cw);
  DE_KARG(chunk_out);
#undef DE_KARG
  return d;
}

// Tiles of a launch: each dense source's slices (position groups of 16), then
// the members' slices, every slice's tiles in row order.
template <bool GATEUP>
struct Tiles {
  const GroupedArgs& a;
  int arg;              // where the kernel arguments hold a
  Tables tb;
  const int32_t* slc;   // member slices: (member << 8) | position group
  int groups;           // position groups of a dense source
  int nds;              // dense slices
  int nms;              // member slices
  int rpt;              // rows (gate/up: pairs) per tile
  int tr;               // tiles per member slice

  __device__ __forceinline__ int dense_tiles(const DenseSrc& d) const {
    return uni(cdiv(GATEUP ? d.inter : d.rows, rpt));
  }
  // Slices of a dense source: its column chunks (down), each with every
  // position group.
  __device__ __forceinline__ int dense_slices(const DenseSrc& d) const {
    return GATEUP ? groups : groups * d.chunks;
  }

  // Sets nds and returns the launch's tiles.
  __device__ __forceinline__ int count() {
    int t = nms * tr;
    nds = 0;
    for (int s = 0; s < a.n_dense; ++s) {
      const DenseSrc d = dense_arg(arg, s);
      nds += dense_slices(d);
      t += dense_slices(d) * dense_tiles(d);
    }
    return t;
  }

  // The slice and row tile of tile t (t < count()).
  __device__ __forceinline__ void locate(int t, int& v, int& r) const {
    v = 0;
    for (int s = 0; s < a.n_dense; ++s) {
      const DenseSrc d = dense_arg(arg, s);
      const int dt = dense_tiles(d), ns = dense_slices(d);
      if (t < ns * dt) {
        const int i = uni(t / dt);
        v += i;
        r = t - i * dt;
        return;
      }
      t -= ns * dt;
      v += ns;
    }
    const int i = uni(t / tr);
    v = nds + i;
    r = t - i * tr;
  }

  __device__ __forceinline__ Slice slice(int v) const {
    Slice c;
    if (v < nds) {
      int s = 0, i = v;
      DenseSrc d = dense_arg(arg, 0);
      while (i >= dense_slices(d)) {  // v < nds: ends at a source
        i -= dense_slices(d);
        d = dense_arg(arg, ++s);
      }
      const int ch = uni(i / groups), g = i - ch * groups;
      c.w = static_cast<const char*>(d.w);
      c.p0 = g * kXP;
      c.nt = min(kXP, a.T - c.p0);
      c.listed = 0;
      c.goff = -1;
      if constexpr (GATEUP) {
        c.rows = d.inter;
        c.K = a.H;
        c.rb = (uint32_t)a.H * 2u;
        c.w2 = (int64_t)d.inter * c.rb;
        c.act = a.x;
        c.astride = a.H;
        c.out = d.out;
        c.ostride = d.inter;
        c.gscalar = 0.f;
      } else {
        c.w += (size_t)ch * d.cw * 2;
        c.rows = d.rows;
        c.K = min(d.cw, d.inter - ch * d.cw);
        c.rb = (uint32_t)(d.ld > 0 ? d.ld : d.inter) * 2u;
        c.w2 = 0;
        c.act = d.vin + (size_t)ch * d.cw;
        c.astride = d.vin_stride;
        c.out = d.out + (size_t)ch * d.chunk_out;
        c.ostride = d.out_stride;
        c.gscalar = d.gate;
      }
      c.tiles = uni(cdiv(c.rows, rpt));
    } else {
      const int e = uni(slc[v - nds]);
      const int j = e >> 8, m0 = (e & 255) * kXP;
      const Member mb = tb.mem[j];
      const char* blk = uni(mb.blk);
      c.p0 = uni(mb.off) + m0;
      c.nt = min(kXP, uni(mb.ntok) - m0);
      c.gscalar = 0.f;
      const int I = a.r.inter;
      if constexpr (GATEUP) {
        c.w = blk;
        c.rows = I;
        c.K = a.H;
        c.rb = (uint32_t)a.H * 2u;
        c.w2 = (int64_t)I * c.rb;
        c.act = a.x;
        c.astride = a.H;
        c.listed = 1;
        c.out = a.r.a;
        c.ostride = I;
        c.goff = -1;
      } else {
        c.w = blk + 2 * mat_bytes<uint16_t>(I, a.H);
        c.rows = a.H;
        c.K = I;
        c.rb = (uint32_t)I * 2u;
        c.w2 = 0;
        c.act = a.r.a;
        c.astride = I;
        c.listed = 0;
        c.out = a.r.p;
        c.ostride = a.H;
        c.goff = c.p0;
      }
      c.tiles = tr;
    }
    return c;
  }
};

// A wave's share of a slice.  The wave's columns are units u0 .. u0 + upw of
// 16 bytes in every row; its fragment (16 rows of them) is loaded as one list
// of units in row order, 64 per load, so that a load reads whole runs of a
// row (512 bytes of two rows for 2048 columns over 8 waves).
template <int KS>
struct Lanes {
  uint32_t w[KS];     // load j: byte offset from the fragment's first row
  uint32_t row;       // load j: the unit's row in bits 4 j .. 4 j + 3
  int upw;            // the wave's units per row
  uint32_t xo;        // activations: byte offset of the lane's position
  int u0, ulast;      // first unit, last unit of the row
  uint32_t ok;        // bit q: the lane's unit of step q exists
  int ragged;         // some lane's unit of some step does not (uniform)
};

__device__ __forceinline__ u32x4 ldw(const char* base, uint32_t off) {
  return __builtin_nontemporal_load((const DE_GLOBAL u32x4*)((const DE_GLOBAL char*)base + off));
}
__device__ __forceinline__ u32x4 ldx(const float* base, uint32_t off) {
  return *(const DE_GLOBAL u32x4*)((const DE_GLOBAL char*)base + off);
}

// Slice c for column slice ks of 2^lkw.  As matrix operands lane l holds row
// (position) l % 16 and columns 8 (l / 16) .. + 7 of each 32-column step; a
// unit that does not exist is read as the last one and zeroed.
template <int KS>
__device__ __forceinline__ Lanes<KS> lanes_of(const Slice& c, const Tables& tb, int ks, int lkw,
                                              int lane) {
  Lanes<KS> L;
  const int n = lane & 15, g = lane >> 4;
  const int S = (c.K + 31) >> 5, U = c.K >> 3;  // steps, units per row
  const int s0 = (ks * S) >> lkw, s1 = ((ks + 1) * S) >> lkw;
  L.ulast = U - 1;
  L.u0 = min(s0 * 4, L.ulast);
  const int upw = max(min(s1 * 4, U) - L.u0, 1);
  L.upw = upw;
  L.row = 0;
  const uint32_t inv = (65536u + upw - 1) / (uint32_t)upw;  // f / upw = f inv >> 16 for f < 512
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    const uint32_t f = (uint32_t)min(j * kWave + lane, 16 * upw - 1);
    const uint32_t row = (f * inv) >> 16, u = f - row * upw;
    L.w[j] = (uint32_t)min((int)row, c.rows - 1) * c.rb + (L.u0 + u) * 16u;
    L.row |= row << (4 * j);
  }
  L.ok = 0;
#pragma unroll
  for (int q = 0; q < KS; ++q) L.ok |= (s0 + q < s1 && (s0 + q) * 4 + g < U) ? 1u << q : 0u;
  const int m = min(n, c.nt - 1);
  const int pos = c.listed ? tb.tok[c.p0 + m] : c.p0 + m;
  L.xo = (uint32_t)pos * (uint32_t)c.astride * 4u;
  L.ragged = __builtin_amdgcn_ballot_w64(L.ok != (1u << KS) - 1u) != 0ull;
  return L;
}

// Where the unit of load j goes in the wave's LDS rows (bytes).
template <int KS>
__device__ __forceinline__ uint32_t stage_off(uint32_t rows, int upw, int j, int lane) {
  const uint32_t f = (uint32_t)min(j * kWave + lane, 16 * upw - 1);
  return (f + ((rows >> (4 * j)) & 15u) * (uint32_t)(kRowUnits<KS> - upw)) * 16u;
}

// Byte offset of the lane's 8 activations of step q.
template <int KS>
__device__ __forceinline__ uint32_t x_off(const Lanes<KS>& L, int q, int g) {
  return L.xo + (uint32_t)min(L.u0 + 4 * q + g, L.ulast) * 32u;
}

// f[0], f[1]: 8 fp32 values -> f[0], f[1], f[2]: their hi, mid and lo bf16
// parts.  A value that is not finite is carried by hi alone.
__device__ __forceinline__ void split8(u32x4 (&f)[3], bool ok) {
  uint32_t v[8], r[8], l[8];
  float chk = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[i] = ok ? f[i >> 2][i & 3] : 0u;
    const float rr = __uint_as_float(v[i]) - __uint_as_float(v[i] & 0xffff0000u);
    r[i] = __float_as_uint(rr);
    chk += rr;
  }
  if (__builtin_amdgcn_ballot_w64(!(chk == chk)) != 0ull) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if ((v[i] & 0x7f800000u) == 0x7f800000u) {
        r[i] = 0u;
        v[i] |= (v[i] & 0x007fffffu) ? 0x00400000u : 0u;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i)
    l[i] = __float_as_uint(__uint_as_float(r[i]) - __uint_as_float(r[i] & 0xffff0000u));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[0][i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], 0x07060302u);
    f[1][i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x07060302u);
    f[2][i] = __builtin_amdgcn_perm(l[2 * i + 1], l[2 * i], 0x07060302u);
  }
}

// One fragment of the wave: 16 weight rows against the activations, sums to
// acc.  The fragment goes from the load registers through the wave's LDS rows
// (st; loads in memory order, reads in operand order) and each load register
// is refilled at once from the next fragment (first row nw, lane offsets of
// nl; LOADS).  conv: the activations are fp32 values to be split first.
// fresh: each step's activation registers are refilled with nl's (of nx).
// The wave's LDS accesses execute in order, so only the compiler has to be
// kept from moving them.
template <int KS, bool LOADS>
__device__ __forceinline__ void fragment(u32x4 (&act)[KS][3], u32x4 (&w)[KS], f32x4& acc, char* st,
                                         uint32_t rows, int upw, bool conv, uint32_t ok,
                                         int ragged, const char* nw, const Lanes<KS>& nl,
                                         bool fresh, const float* nx, int lane) {
  // Opaque to the compiler: the offsets below are computed again for every
  // fragment instead of being kept in registers across them.
  asm volatile("" : "+v"(lane));
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    *reinterpret_cast<u32x4*>(st + stage_off<KS>(rows, upw, j, lane)) = w[j];
    if constexpr (LOADS) w[j] = ldw(nw, nl.w[j]);
  }
  asm volatile("" ::: "memory");
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4* rd = reinterpret_cast<const u32x4*>(st) + n * kRowUnits<KS> + g;
#pragma unroll
  for (int q = 0; q < KS; ++q) {
    const bool okq = !ragged || ((ok >> q) & 1u);
    if (conv) split8(act[q], okq);
    u32x4 b = rd[4 * q];
    if (ragged) {
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = okq ? b[i] : 0u;
    }
    // The step's three products are summed from zero, smallest part first, and
    // added to the fragment's sums: a chain through all steps would round
    // every part at the full sum's magnitude.
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 2; p >= 0; --p)
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, act[q][p]),
                                                  __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    acc += c;
    if constexpr (LOADS) {
      if (fresh) {
        const uint32_t o = x_off(nl, q, g);
        act[q][0] = ldx(nx, o);
        act[q][1] = ldx(nx, o + 16u);
      }
    }
    if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the operands read ahead
  }
  asm volatile("" ::: "memory");
}

// Waits for the wave's LDS accesses and the block's other waves; loads in
// flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// First row of row group rw's 16-row fragment i of tile r (the last one is
// moved up to end with the matrix; rows computed twice get the same value).
template <bool GATEUP>
__device__ __forceinline__ int frag_row(const Slice& c, int rpt, int r, int rw, int i) {
  const int lim = max(c.rows - 16, 0);
  return min(r * rpt + (GATEUP ? rw * 16 : rw * 32 + i * 16), lim);
}

// The block's tiles.
template <int KS, bool GATEUP>
__device__ __forceinline__ void stream(const GroupedArgs& a, Tiles<GATEUP>& tl, int lkw,
                                       float* red, int lane, int wave) {
  const int total = tl.count();
  const int lo = (int)((int64_t)total * blockIdx.x / gridDim.x);
  const int hi = (int)((int64_t)total * (blockIdx.x + 1) / gridDim.x);
  if (lo >= hi) return;
  const int kw = 1 << lkw, nrw = kWavesPB >> lkw;
  const int ks = wave & (kw - 1), rw = wave >> lkw;
  const int g = lane >> 4, n = lane & 15;
  int v, r;
  tl.locate(lo, v, r);
  Slice c = tl.slice(v);
  Lanes<KS> L = lanes_of<KS>(c, tl.tb, ks, lkw, lane);
  u32x4 act[KS][3], w[KS];
  f32x4 acc[2];
  char* st = reinterpret_cast<char*>(red + kRedFloats) + wave * 16 * kRowUnits<KS> * 16;
  const auto base = [&](const Slice& s, int tr, int i) {
    if (GATEUP) return uni(s.w + (size_t)frag_row<true>(s, tl.rpt, tr, rw, 0) * s.rb + i * s.w2);
    return uni(s.w + (size_t)frag_row<false>(s, tl.rpt, tr, rw, i) * s.rb);
  };
  {
    const char* p0 = base(c, r, 0);
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      act[q][0] = ldx(c.act, x_off(L, q, g));
      act[q][1] = ldx(c.act, x_off(L, q, g) + 16u);
    }
#pragma unroll
    for (int j = 0; j < KS; ++j) w[j] = ldw(p0, L.w[j]);
  }
  // The tile's output rows from the waves' partials.
  float* buf = red;
  const auto finish = [&]() {
    // Partials of the wave: position 4 g + i, row n of both fragments.
    float* p = buf + wave * 2 * kRedTile + 4 * g * kRedLd + n;
    if (4 * g < c.nt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[i * kRedLd] = acc[0][i];
        p[kRedTile + i * kRedLd] = acc[1][i];
      }
    }
    lds_barrier();
    constexpr int kOut = GATEUP ? 256 : 512;  // outputs of a row group
    for (int o = threadIdx.x; o < kOut * nrw; o += kBlock) {
      const int rg = o / kOut, pos = (o / (kOut / 16)) & 15, rr = o & 15;
      const int i = GATEUP ? 0 : (o >> 4) & 1;
      const int row = frag_row<GATEUP>(c, tl.rpt, r, rg, i) + rr;
      if (pos < c.nt && row < c.rows) {
        const float* q = buf + ((rg << lkw) * 2 + i) * kRedTile + pos * kRedLd + rr;
        float s = 0.f, u = 0.f;
        for (int k = 0; k < kw; ++k) {
          s += q[k * 2 * kRedTile];
          if constexpr (GATEUP) u += q[k * 2 * kRedTile + kRedTile];
        }
        float val;
        if constexpr (GATEUP)
          val = silu_f(s) * u;
        else
          val = (c.goff >= 0 ? tl.tb.gate[c.goff + pos] : c.gscalar) * s;
        *(DE_GLOBAL float*)(c.out + (size_t)(c.p0 + pos) * c.ostride + row) = val;
      }
    }
    buf = buf == red ? red + kRedBuf : red;
  };
  bool conv = true;
#pragma unroll 1
  for (int left = hi - lo; left > 1; --left) {
    const bool same = r + 1 < c.tiles;
    fragment<KS, true>(act, w, acc[0], st, L.row, L.upw, conv, L.ok, L.ragged, base(c, r, 1), L, false,
                       nullptr, lane);
    const uint32_t ok = L.ok;
    const int ragged = L.ragged;
    const float* nx = nullptr;
    const char* np;
    const uint32_t rows = L.row;
    const int upw = L.upw;
    if (same) {
      np = base(c, r + 1, 0);
    } else {
      const Slice ns = tl.slice(v + 1);
      L = lanes_of<KS>(ns, tl.tb, ks, lkw, lane);
      np = base(ns, 0, 0);
      nx = ns.act;
    }
    fragment<KS, true>(act, w, acc[1], st, rows, upw, false, ok, ragged, np, L, !same, nx, lane);
    finish();
    conv = !same;
    if (same) {
      ++r;
    } else {
      ++v;
      r = 0;
      c = tl.slice(v);
    }
  }
  fragment<KS, true>(act, w, acc[0], st, L.row, L.upw, conv, L.ok, L.ragged, base(c, r, 1), L, false,
                     nullptr, lane);
  fragment<KS, false>(act, w, acc[1], st, L.row, L.upw, false, L.ok, L.ragged, nullptr, L, false, nullptr,
                      lane);
  finish();
}

// The member slices: every resident member's positions in groups of 16, in
// member order.  One wave; returns their number.
__device__ __forceinline__ int member_slices(const Tables& tb, int nu, int32_t* slc, int lane) {
  int base = 0;
  for (int j0 = 0; j0 < nu; j0 += kWave) {
    const int j = j0 + lane;
    int ng = 0;
    if (j < nu && tb.mem[j].blk != nullptr) ng = (tb.mem[j].ntok + kXP - 1) / kXP;
    int inc = ng;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(inc, o, kWave);
      if (lane >= o) inc += up;
    }
    const int at = base + inc - ng;
    for (int i = 0; i < ng; ++i) slc[at + i] = (j << 8) | i;
    base += __builtin_amdgcn_readlane(inc, 63);
  }
  return base;
}

// LDS: [partials][staged weights][tables][selection state (gate/up)][member slices]
__device__ __forceinline__ int32_t* slices_at(const GroupedArgs& a, const Tables& tb) {
  char* p = reinterpret_cast<char*>(tb.gate + (a.has_routed ? a.r.pairs_max : 0));
  if (a.fuse_route) p += sel_view_bytes(a.T, a.sel.k, a.sel.N);
  return reinterpret_cast<int32_t*>(p);
}


// What a block knows of the routed part.
struct MfmaTables {
  Tables tb;
  const int32_t* slc;
  int nu, nms;        // members, member slices
};

// The block's tables: the lists (selected and united here in a gate/up launch
// with fused routing, else read), the members and their slices.  absent and
// nms are shared words.  Ends with a barrier.
template <int KS, bool GATEUP>
__device__ __forceinline__ MfmaTables mfma_tables(const GroupedArgs& a, int lane, int wave,
                                                  int* absent, int* nms) {
  MfmaTables mt;
  mt.tb = tables_at(a, kRedFloats + kStageFloats<KS>);
  if (threadIdx.x == 0) {
    *absent = 0;
    *nms = 0;
  }
  mt.nu = 0;
  if (GATEUP && a.fuse_route) {
    float z0[2][4];
    first_logits(a, wave, z0);
    __syncthreads();  // absent is initialised
    mt.nu = route_lists(a, mt.tb, z0, lane, wave, absent);
  } else {
    mt.nu = routed_count(a);
    __syncthreads();
    if (a.has_routed) fill_tables(a, mt.tb, mt.nu, absent);
    __syncthreads();
  }
  int32_t* slc = slices_at(a, mt.tb);
  mt.slc = slc;
  if (a.has_routed) {
    if (wave == 0) {
      const int c = member_slices(mt.tb, mt.nu, slc, lane);
      if (lane == 0) *nms = c;
    }
    __syncthreads();
  }
  mt.nms = uni(*nms);
  // A needed member without a slot: reported once per layer.
  if (GATEUP && *absent && !a.r.absent_ok && blockIdx.x == 0 && threadIdx.x == 0 &&
      a.r.status != nullptr)
    *(DE_GLOBAL int32_t*)a.r.status |= kStatusNotResident;
  return mt;
}

// One pass over the tables of a block: the slices are known (slc, nms).
template <int KS, bool GATEUP>
__device__ __forceinline__ void mfma_pass(const GroupedArgs& a, int arg, const Tables& tb,
                                          const int32_t* slc, int nms, int lane, int wave) {
  Tiles<GATEUP> tl{a, arg, tb, slc, cdiv(a.T, kXP), 0, nms, 0, 0};
  tl.rpt = (kWavesPB >> a.lkw) * (GATEUP ? 16 : 32);
  tl.tr = a.has_routed ? uni(cdiv(GATEUP ? a.r.inter : a.H, tl.rpt)) : 1;
  stream<KS, GATEUP>(a, tl, a.lkw, s_dyn, lane, wave);
}

template <int KS>
size_t mfma_lds(const GroupedArgs& a) {
  size_t b = (size_t)(kRedFloats + kStageFloats<KS>)*4 + tables_bytes(a);
  if (a.has_routed) b += ((size_t)a.r.max_union + a.r.pairs_max / kXP + 1) * 4;
  return b;
}

}  // namespace
}  // namespace de
