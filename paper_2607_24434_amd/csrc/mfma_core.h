// The grouped gate/up and down passes of a block of positions on the matrix
// cores, for bf16 and Q4_0 weights (the LM head's row-dot is a down pass of
// one source): the device functions of the separate launches and of the
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
// and meets one or two experts.  The bf16 gate/up launch of a V2-Lite layer at
// T = 9 streams 460 MB in 79 us, 5.8 TB/s with its prologue and its tail (a linear
// read of 4 GiB on the same card: 6.0).
//
// Q4_0: a fragment is a quarter of the bytes, so a tile is four fragments and
// all four are in flight.  The codes become bf16 operands with one conversion
// per two (the vector ALU needed one conversion and one FMA per weight and
// position); V2-Lite layer at T = 9: gate/up 42 us (vector ALU 63), down 30
// (51), bound by the latency of a fragment's way through LDS, conversion and
// matrix cores.
//
// Measured (rocprofv3): V2-Lite layer T = 9 gate/up 79 us (vector ALU 88), down
// 44 (47); T = 64 142 (554) and 82 (248); Moonlight layer T = 17 87 and 51; dense
// layer of 10944 at T = 9 19 and 13 (78 us with the combine before, 39 now); LM head
// of 102400 at T = 9 72 (101).
//
// More than 16 positions are several slices of 16 over the same rows.  Where
// a launch has one dense source (a dense layer, the LM head) the blocks that
// read the same rows for two groups sit on one XCD and run side by side, so the
// second reading comes from its L2, us before and now (loads that pass the L2
// by, blocks that drift apart when their groups' sizes differ): LM head of
// 102400 T = 17 134 and 98, T = 32 103 and 107, T = 64 165 and 160; dense layer
// of 10944 T = 17 62 and 57, T = 32 64 and 56, T = 64 100 and 72.
#pragma once

#include "grouped_core.h"
#include "grouped_mfma.h"
#include "topk_union.h"

namespace de {
namespace {

constexpr int kRedLd = 20;                    // LDS partials: row stride (4 extra: no bank conflicts)
constexpr int kRedTile = kXP * kRedLd;        // one 16 x 16 tile of partials
template <typename WT>
constexpr int kFrags = kQ4<WT> ? 4 : 2;       // 16-row fragments of a wave's tile
template <typename WT>
constexpr int kRedBuf = kWavesPB * kFrags<WT> * kRedTile;
template <typename WT>
constexpr int kRedFloats = 2 * kRedBuf<WT>;   // double buffered: one barrier per tile

// 16-byte units of a row per step of 32 columns (Q4_0: one unit is one block).
template <typename WT>
constexpr int kStepUnits = kQ4<WT> ? 1 : 4;
constexpr int pow2_ceil(int v) {
  int p = 1;
  while (p < v) p *= 2;
  return p;
}
// Lanes that load a row's units (a power of two), and the rows and number of a
// fragment's load instructions.
template <typename WT, int KS>
constexpr int kRowLanes = pow2_ceil(KS * kStepUnits<WT>);
template <typename WT, int KS>
constexpr int kLoadRows = kWave / kRowLanes<WT, KS> < 16 ? kWave / kRowLanes<WT, KS> : 16;
template <typename WT, int KS>
constexpr int kLoads = 16 / kLoadRows<WT, KS>;
// LDS of a wave's staged fragment: 16 rows of units with one unit of padding
// per row (no bank conflicts in the fragment reads), then (Q4_0) 16 rows of 8
// scales.
template <typename WT, int KS>
constexpr int kRowUnits = kStepUnits<WT> * KS + 1;
template <typename WT, int KS>
constexpr int kWaveStage = 16 * kRowUnits<WT, KS> * 16 + (kQ4<WT> ? 16 * 16 : 0);
template <typename WT, int KS>
constexpr int kStageFloats = kWavesPB * kWaveStage<WT, KS> / 4;

// Rows (gate/up: pairs) of a row group of waves in a tile.
template <typename WT, bool GATEUP>
__host__ __device__ constexpr int group_rows() {
  return GATEUP ? 8 * kFrags<WT> : 16 * kFrags<WT>;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A slice: up to 16 positions against the rows of one source (the same in
// every lane).
struct Slice {
  const char* w;      // gate/up: G; down: the matrix
  const char* sc;     // Q4_0: the scales of the first row
  int64_t w2;         // gate/up: bytes from a G row (and its scales) to its U row
  int rows, K;        // rows (gate/up: pairs), columns
  uint32_t rb, srb;   // bytes per row of weights (codes) and of scales
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
  DE_KARG(ws);
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
template <typename WT, bool GATEUP>
struct Tiles {
  const GroupedArgs& a;
  int arg;              // where the kernel arguments hold a
  Tables tb;
  const int32_t* slc;   // member slices: (member << 8) | position group
  int nms;              // member slices

  __device__ __forceinline__ int total() const { return a.geo.ndt + nms * a.geo.tr; }

  // The slice and row tile of tile t (t < total()).
  __device__ __forceinline__ void locate(int t, int& v, int& r) const {
    const MfmaGeom& g = a.geo;
    int base = g.ndt, first = g.nds, tiles = g.tr;
    if (t < g.ndt) {
      const int s = (a.n_dense > 2 && t >= g.t0[2]) ? 2 : ((a.n_dense > 1 && t >= g.t0[1]) ? 1 : 0);
      base = s == 0 ? 0 : (s == 1 ? g.t0[1] : g.t0[2]);
      first = s == 0 ? 0 : (s == 1 ? g.v0[1] : g.v0[2]);
      tiles = s == 0 ? g.tiles[0] : (s == 1 ? g.tiles[1] : g.tiles[2]);
    }
    const int i = uni((int)((uint32_t)(t - base) / (uint32_t)tiles));
    v = first + i;
    r = t - base - i * tiles;
  }

  __device__ __forceinline__ Slice slice(int v) const {
    Slice c;
    const MfmaGeom& geo = a.geo;
    if (v < geo.nds) {
      const int s = (a.n_dense > 2 && v >= geo.v0[2]) ? 2 : ((a.n_dense > 1 && v >= geo.v0[1]) ? 1 : 0);
      const int i = v - (s == 0 ? 0 : (s == 1 ? geo.v0[1] : geo.v0[2]));
      const DenseSrc d = dense_arg(arg, s);
      // One group (up to 16 positions) is the common case.
      const int ch = geo.groups == 1 ? i : uni(i / geo.groups), g = i - ch * geo.groups;
      c.w = static_cast<const char*>(d.w);
      c.p0 = g * kXP;
      c.nt = min(kXP, a.T - c.p0);
      c.listed = 0;
      c.goff = -1;
      if constexpr (GATEUP) {
        c.rows = d.inter;
        c.K = a.H;
        c.rb = (uint32_t)qrow_bytes<WT>(a.H);
        c.w2 = (int64_t)mat_bytes<WT>(d.inter, a.H);
        c.act = a.x;
        c.astride = a.H;
        c.out = d.out;
        c.ostride = d.inter;
        c.gscalar = 0.f;
      } else {
        c.w += qrow_bytes<WT>(ch * d.cw);
        c.rows = d.rows;
        c.K = min(d.cw, d.inter - ch * d.cw);
        c.rb = (uint32_t)qrow_bytes<WT>(d.ld > 0 ? d.ld : d.inter);
        c.w2 = 0;
        c.act = d.vin + (size_t)ch * d.cw;
        c.astride = d.vin_stride;
        c.out = d.out + (size_t)ch * d.chunk_out;
        c.ostride = d.out_stride;
        c.gscalar = d.gate;
      }
      // Q4_0: a matrix's scales follow its codes (a column chunk's are given).
      c.srb = c.rb >> 3;
      c.sc = GATEUP ? c.w + (size_t)c.rows * c.rb
                    : static_cast<const char*>(d.ws) + (size_t)ch * (d.cw >> 4);
      c.tiles = s == 0 ? geo.tiles[0] : (s == 1 ? geo.tiles[1] : geo.tiles[2]);
    } else {
      const int e = uni(slc[v - geo.nds]);
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
        c.rb = (uint32_t)qrow_bytes<WT>(a.H);
        c.w2 = (int64_t)mat_bytes<WT>(I, a.H);
        c.act = a.x;
        c.astride = a.H;
        c.listed = 1;
        c.out = a.r.a;
        c.ostride = I;
        c.goff = -1;
      } else {
        c.w = blk + 2 * mat_bytes<WT>(I, a.H);
        c.rows = a.H;
        c.K = I;
        c.rb = (uint32_t)qrow_bytes<WT>(I);
        c.w2 = 0;
        c.act = a.r.a;
        c.astride = I;
        c.listed = 0;
        c.out = a.r.p;
        c.ostride = a.H;
        c.goff = c.p0;
      }
      c.srb = c.rb >> 3;
      c.sc = c.w + (size_t)c.rows * c.rb;
      c.tiles = geo.tr;
    }
    return c;
  }
};

// A wave's share of a slice.  The wave's columns are units u0 .. u0 + upw of
// 16 bytes in every row; a load instruction reads them of kLoadRows consecutive
// rows of its fragment (whole runs: 512 bytes of two rows for 2048 columns over
// 8 waves), kRowLanes lanes a row.  So the loads' offsets, in memory and in LDS,
// differ by one constant and take two vector instructions; packed as one list of
// units (no idle lanes where the columns are no power of two) they took two
// products and a dozen (verify layers 1 to 3% slower).
template <typename WT, int KS>
struct Lanes {
  uint32_t lo, lim;   // the lane's unit of load 0, and of the last row (byte offsets)
  uint32_t so;        // the unit of load 0 in the wave's LDS rows (bytes)
  uint32_t ss;        // Q4_0: its scale there
  uint32_t rb;        // bytes per row of weights
  uint32_t xo;        // activations: byte offset of the lane's position
  int u0, ulast;      // first unit, last unit of the row
  uint32_t ok;        // bit q: the lane's columns of step q exist
};

// Weights: past the L2 where they are read once (through it the passes are 4 to
// 11% slower), kept there for the other position group's block of the XCD with
// REREAD.
template <bool REREAD>
__device__ __forceinline__ u32x4 ldw(const char* base, uint32_t off) {
  const DE_GLOBAL u32x4* p = (const DE_GLOBAL u32x4*)((const DE_GLOBAL char*)base + off);
  if constexpr (REREAD)
    return *p;
  else
    return __builtin_nontemporal_load(p);
}
// Activations.  SHARED: written by other blocks of this launch, so read at agent
// scope, past the XCDs' own L2 caches.
template <bool SHARED>
__device__ __forceinline__ u32x4 ldx(const float* base, uint32_t off) {
  const DE_GLOBAL char* p = (const DE_GLOBAL char*)base + off;
  if constexpr (SHARED) {
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint64_t w = __hip_atomic_load((const DE_GLOBAL uint64_t*)p + i, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
      v[2 * i] = (uint32_t)w;
      v[2 * i + 1] = (uint32_t)(w >> 32);
    }
    return v;
  } else {
    return *(const DE_GLOBAL u32x4*)p;
  }
}

// The lane's byte offset of load j from the fragment's first row (rows past the
// source's last one re-read that; with mask 0 every lane reads the first word).
// Q4_0: the scale's offset is an eighth of it, as the rows' bytes are.
template <typename WT, int KS>
__device__ __forceinline__ uint32_t load_off(const Lanes<WT, KS>& L, int j, uint32_t mask) {
  return min(L.lo + (uint32_t)(j * kLoadRows<WT, KS>) * L.rb, L.lim & mask);
}

// Slice c for column slice ks of 2^lkw.  As matrix operands lane l holds row
// (position) l % 16 and 8 columns of each 32-column step: bf16 weights 8 g ..
// 8 g + 7 with g = l / 16; Q4_0 4 g .. 4 g + 3 and 16 + 4 g .. (the low and
// high nibbles of 4 bytes of the block).  A unit that does not exist is never
// staged: its LDS words and its activations are zero.
template <typename WT, int KS>
__device__ __forceinline__ Lanes<WT, KS> lanes_of(const Slice& c, const Tables& tb, int ks, int lkw,
                                                  int lane) {
  Lanes<WT, KS> L;
  constexpr int SU = kStepUnits<WT>;
  const int n = lane & 15, g = lane >> 4;
  const int S = (c.K + 31) >> 5, U = (int)(qrow_bytes<WT>(c.K) >> 4);  // steps, units per row
  const int s0 = (ks * S) >> lkw, s1 = ((ks + 1) * S) >> lkw;
  L.ulast = U - 1;
  L.u0 = min(s0 * SU, L.ulast);
  const int upw = max(min(s1 * SU, U) - L.u0, 1);
  const int row = min(lane / kRowLanes<WT, KS>, kLoadRows<WT, KS> - 1);
  const int u = min(lane % kRowLanes<WT, KS>, upw - 1);  // (a lane without a unit: the last one)
  L.rb = c.rb;
  L.lo = (uint32_t)row * c.rb + (uint32_t)(L.u0 + u) * 16u;
  L.lim = (uint32_t)(min(c.rows, 16) - 1) * c.rb + (uint32_t)(L.u0 + u) * 16u;
  L.so = (uint32_t)(row * kRowUnits<WT, KS> + u) * 16u;
  L.ss = (uint32_t)(row * 8 + u) * 2u;
  L.ok = 0;
#pragma unroll
  for (int q = 0; q < KS; ++q)
    L.ok |= (s0 + q < s1 && (kQ4<WT> || (s0 + q) * SU + g < U)) ? 1u << q : 0u;
  const int m = min(n, c.nt - 1);
  const int pos = c.listed ? tb.tok[c.p0 + m] : c.p0 + m;
  L.xo = (uint32_t)pos * (uint32_t)c.astride * 4u;
  return L;
}

// The lane's 8 activations of step q (fp32).
template <typename WT, int KS, bool SHARED>
__device__ __forceinline__ void load_x(u32x4 (&f)[3], const float* x, const Lanes<WT, KS>& L, int q,
                                       int g) {
  if constexpr (kQ4<WT>) {
    const uint32_t o = L.xo + (uint32_t)min(L.u0 + q, L.ulast) * 128u + g * 16u;
    f[0] = ldx<SHARED>(x, o);
    f[1] = ldx<SHARED>(x, o + 64u);
  } else {
    const uint32_t o = L.xo + (uint32_t)min(L.u0 + 4 * q + g, L.ulast) * 32u;
    f[0] = ldx<SHARED>(x, o);
    f[1] = ldx<SHARED>(x, o + 16u);
  }
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

// Steps whose products are in flight together: independent chains of three
// matrix instructions.
template <int KS>
constexpr int kStepGroup = KS < 4 ? KS : (KS % 4 == 0 ? 4 : 3);

// c += the steps' products with the activations' hi, then mid, then lo parts.
template <int N>
__device__ __forceinline__ void add_products(const u32x4 (*act)[3], const u32x4 (&b)[N],
                                             f32x4 (&c)[N]) {
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int i = 0; i < N; ++i)
      c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, act[i][p]),
                                                     __builtin_bit_cast(bf16x8, b[i]), c[i], 0, 0,
                                                     0);
}

// acc of the steps' three products each, summed from zero, smallest part
// first: a chain through all steps would round every part at the full sum's
// magnitude.
template <int N>
__device__ __forceinline__ void products(const u32x4 (*act)[3], const u32x4 (&b)[N],
                                         f32x4 (&c)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 2; p >= 0; --p)
#pragma unroll
    for (int i = 0; i < N; ++i)
      c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, act[i][p]),
                                                     __builtin_bit_cast(bf16x8, b[i]), c[i], 0, 0,
                                                     0);
}

// Puts a bf16 fragment's load registers into the wave's LDS rows (loads in
// memory order, reads in operand order) and refills each at once from the next
// fragment (first row nw, lane offsets of nl; with mask 0 every lane re-reads
// nw).  The wave's LDS accesses execute in order, so only the compiler has to
// be kept from moving them.
template <typename WT, int KS, bool REREAD>
__device__ __forceinline__ void stage(u32x4* w, char* st,
                                      const Lanes<WT, KS>& L, const char* nw,
                                      const Lanes<WT, KS>& nl, uint32_t mask) {
#pragma unroll
  for (int j = 0; j < kLoads<WT, KS>; ++j) {
    *reinterpret_cast<u32x4*>(st + L.so + j * kLoadRows<WT, KS> * kRowUnits<WT, KS> * 16) = w[j];
    w[j] = ldw<REREAD>(nw, load_off(nl, j, mask));
  }
}

// The sums of the staged bf16 fragment: 16 weight rows against the
// activations.  Nothing branches between the matrix instructions.
template <int KS>
__device__ __forceinline__ f32x4 fragment_sums(const u32x4 (&act)[KS][3], const char* st,
                                               int lane) {
  constexpr int N = kStepGroup<KS>;
  const u32x4* rd = reinterpret_cast<const u32x4*>(st) +
                    (lane & 15) * kRowUnits<uint16_t, KS> + (lane >> 4);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q0 = 0; q0 < KS; q0 += N) {
    u32x4 b[N];
    f32x4 c[N];
#pragma unroll
    for (int i = 0; i < N; ++i) b[i] = rd[4 * (q0 + i)];
    products<N>(act + q0, b, c);
#pragma unroll
    for (int i = 0; i < N; ++i) acc += c[i];
    __builtin_amdgcn_sched_barrier(0);  // bounds the operands read ahead
  }
  return acc;
}

// The sums of the staged Q4_0 fragment.  A step is one block of 32 weights per
// row, d (q - 8): the codes q become bf16 operands (a byte 0 .. 15 read as
// e4m3 is q / 512, denormal or not, so one conversion with scale 512 makes two
// of them), the products q x are summed by the matrix cores on top of -8 times
// the block's activation sum (xm; hi parts first, so that what follows rounds
// at the small sum of (q - 8) x), and the scale, which lane l holds for its own
// row l % 16, is applied to the block's sums.
template <int KS>
__device__ __forceinline__ f32x4 fragment_sums_q4(const u32x4 (&act)[KS][3], const f32x4 (&xm)[KS],
                                                  const char* st, int lane) {
  constexpr int N = kStepGroup<KS>, RU = kRowUnits<q4_t, KS>;
  const uint32_t* rd = reinterpret_cast<const uint32_t*>(st) + (lane & 15) * RU * 4 + (lane >> 4);
  const u32x4 dv = reinterpret_cast<const u32x4*>(st + 16 * RU * 16)[lane & 15];
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q0 = 0; q0 < KS; q0 += N) {
    u32x4 b[N];
    f32x4 c[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t v = rd[4 * (q0 + i)];
      const uint32_t lo = v & 0x0f0f0f0fu, hi = (v >> 4) & 0x0f0f0f0fu;
#define DE_CODES(x, h) \
  __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x, 512.f, h))
      b[i] = u32x4{DE_CODES(lo, false), DE_CODES(lo, true), DE_CODES(hi, false),
                   DE_CODES(hi, true)};
#undef DE_CODES
    }
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = xm[q0 + i];
    add_products<N>(act + q0, b, c);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int q = q0 + i;
      const float d = half_bits_to_float((dv[q >> 1] >> (16 * (q & 1))) & 0xffffu);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = fmaf(d, c[i][j], acc[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// Waits for the wave's LDS accesses and the block's other waves; loads in
// flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// First row of 16-row group i of row group rw of tile r (the last one is moved
// up to end with the matrix; rows computed twice get the same value).
template <typename WT, bool GATEUP>
__device__ __forceinline__ int frag_row(const Slice& c, int rpt, int r, int rw, int i) {
  return min(r * rpt + rw * group_rows<WT, GATEUP>() + i * 16, max(c.rows - 16, 0));
}

// Fragment f of tile r: gate/up G and U of row group f / 2, down row group f.
template <typename WT, bool GATEUP>
__device__ __forceinline__ const char* frag_base(const Slice& c, int rpt, int r, int rw, int f) {
  const size_t row = (size_t)frag_row<WT, GATEUP>(c, rpt, r, rw, GATEUP ? f >> 1 : f);
  return uni(c.w + row * c.rb + (GATEUP && (f & 1) ? c.w2 : 0));
}
template <typename WT, bool GATEUP>
__device__ __forceinline__ const char* scale_base(const Slice& c, int rpt, int r, int rw, int f) {
  const size_t row = (size_t)frag_row<WT, GATEUP>(c, rpt, r, rw, GATEUP ? f >> 1 : f);
  return uni(c.sc + row * c.srb + (GATEUP && (f & 1) ? c.w2 : 0));
}

// A wave's sums of fragment f: position 4 g + i, row n.
template <typename WT>
__device__ __forceinline__ void put_partial(float* buf, const f32x4& acc, int f, int nt, int wave,
                                            int lane) {
  const int g = lane >> 4, n = lane & 15;
  float* p = buf + (wave * kFrags<WT> + f) * kRedTile + 4 * g * kRedLd + n;
  if (4 * g < nt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i * kRedLd] = acc[i];
  }
}

// Output o of a tile (a thread's are threadIdx.x, + kBlock, ...: whole waves): its
// position in the slice and its row.
template <typename WT, bool GATEUP>
__device__ __forceinline__ bool output_at(const Slice& c, int rpt, int r, int o, int& rr, int& i,
                                          int& rg, int& pos, int& row) {
  constexpr int kG = GATEUP ? kFrags<WT> / 2 : kFrags<WT>;  // 16-row groups of a row group
  // Row within 16, 16-row group, position, row group.
  rr = o & 15;
  i = (o >> 4) & (kG - 1);
  pos = (o / (16 * kG)) & 15;
  rg = o / (256 * kG);
  row = frag_row<WT, GATEUP>(c, rpt, r, rg, i) + rr;
  return pos < c.nt && row < c.rows;
}
template <typename WT, bool GATEUP>
__device__ __forceinline__ int tile_outs(int lkw) {
  return 256 * (GATEUP ? kFrags<WT> / 2 : kFrags<WT>) * (kWavesPB >> lkw);
}

template <bool GATEUP>
__device__ __forceinline__ float output_value(const Slice& c, const Tables& tb, int pos, float s,
                                              float u) {
  if constexpr (GATEUP) return silu_f(s) * u;
  return (c.goff >= 0 ? tb.gate[c.goff + pos] : c.gscalar) * s;
}

// The tile's outputs from the waves' sums (after the barrier).  SHARED: other
// blocks of this launch read them.  nan is set where one is NaN.
template <typename WT, bool GATEUP, bool SHARED>
__device__ __forceinline__ void tile_outputs(const Slice& c, const Tables& tb, int rpt, int r,
                                             int lkw, const float* buf, int& nan) {
  const int kw = 1 << lkw;
  constexpr int kWaveRed = kFrags<WT> * kRedTile;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // addresses are computed again for every tile
#pragma unroll 1
  for (int o = tid; o < tile_outs<WT, GATEUP>(lkw); o += kBlock) {
    int rr, i, rg, pos, row;
    if (output_at<WT, GATEUP>(c, rpt, r, o, rr, i, rg, pos, row)) {
      const float* q = buf + (rg << lkw) * kWaveRed + (GATEUP ? 2 * i : i) * kRedTile +
                       pos * kRedLd + rr;
      float s = 0.f, u = 0.f;
      for (int k = 0; k < kw; ++k) {
        s += q[k * kWaveRed];
        if constexpr (GATEUP) u += q[k * kWaveRed + kRedTile];
      }
      const float val = output_value<GATEUP>(c, tb, pos, s, u);
      st_out<SHARED>(c.out + (size_t)(c.p0 + pos) * c.ostride + row, val);
      nan |= val == val ? 0 : 1;
    }
  }
}

// A bf16 row's product with one position in fp32, by one wave, in the vector ALU
// path's order.  Every lane gets the sum, and whether the position itself holds a
// NaN.
template <bool SHARED>
__device__ __forceinline__ float plain_dot(const Slice& c, const Tables& tb, int pos, int row,
                                           int64_t to, int lane, bool& xnan) {
  const int p = c.listed ? tb.tok[c.p0 + pos] : c.p0 + pos;
  const float* x = c.act + (size_t)p * c.astride;
  const char* w = c.w + (size_t)row * c.rb + to;
  float s = 0.f;
  bool nan = false;
#pragma unroll 1
  for (int u = lane; u < c.K / 8; u += kWave) {
    float v[8];
    unpack(ldw<true>(w, (uint32_t)u * 16u), v);
    const u32x4 x0 = ldx<SHARED>(x, u * 32u), x1 = ldx<SHARED>(x, u * 32u + 16u);
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(v[i], __uint_as_float(x0[i]), s);
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(v[4 + i], __uint_as_float(x1[i]), s);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      nan = nan || (x0[i] & 0x7fffffffu) > 0x7f800000u || (x1[i] & 0x7fffffffu) > 0x7f800000u;
  }
  xnan = __builtin_amdgcn_ballot_w64(nan) != 0ull;
  return row_total(s);
}

// Takes the wave's outputs that are NaN among the block's tiles (as in stream)
// from plain products: an infinite weight meets a zero mid or lo part of nearly
// every finite activation, and that product is NaN on the matrix cores.  After the
// tiles, so that the loop over them only notes a NaN (0.2%; with the products in
// the loop 1%).
template <typename WT, bool GATEUP, bool SHARED, class TL>
__device__ __forceinline__ void plain_outputs(const TL& tl, int v, int r, int step, int count,
                                              int lkw, int lane) {
  const int rpt = tl.a.geo.rpt;
  Slice c = tl.slice(v);
#pragma unroll 1
  for (; count > 0; --count) {
#pragma unroll 1
    for (int o = threadIdx.x; o < tile_outs<WT, GATEUP>(lkw); o += kBlock) {
      int rr, i, rg, pos, row;
      const bool mine = output_at<WT, GATEUP>(c, rpt, r, o, rr, i, rg, pos, row);
      float* const p = c.out + (size_t)(c.p0 + pos) * c.ostride + row;
      float val = 0.f;
      if (mine) {  // (its own store)
        if constexpr (SHARED)
          val = __hip_atomic_load((DE_GLOBAL float*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          val = *(DE_GLOBAL float*)p;
      }
      unsigned long long bad = __builtin_amdgcn_ballot_w64(!(val == val));
      while (bad != 0ull) {
        const int l = (int)__builtin_ctzll(bad);
        const int lp = __builtin_amdgcn_readlane(pos, l), lr = __builtin_amdgcn_readlane(row, l);
        bad &= bad - 1;
        bool xnan;
        const float s = plain_dot<SHARED && !GATEUP>(c, tl.tb, lp, lr, 0, lane, xnan);
        if (xnan) {  // all outputs of the position are NaN, whatever the weights
          bad &= ~__builtin_amdgcn_ballot_w64(pos == lp);
          continue;
        }
        float u = 0.f;
        if constexpr (GATEUP) u = plain_dot<false>(c, tl.tb, lp, lr, c.w2, lane, xnan);
        if (lane == l) st_out<SHARED>(p, output_value<GATEUP>(c, tl.tb, pos, s, u));
      }
    }
    if (++r >= c.tiles && count > 1) {
      r = 0;
      c = tl.slice(v += step);
    }
  }
}

// What a wave holds: the activation fragments of its slice and the weights in
// flight.  bf16: one fragment, refilled from the next one.  Q4_0 (a fragment
// is a quarter of the bytes): the tile's four fragments with their units'
// scales, each refilled from the same fragment of the next tile, and -8 times
// the activation sum of every block.
template <typename WT, int KS>
struct Regs {
  static constexpr int kDepth = kQ4<WT> ? kFrags<WT> : 1;
  u32x4 act[KS][3];
  u32x4 w[kDepth][kLoads<WT, KS>];
  uint32_t sc[kQ4<WT> ? kDepth : 1][kQ4<WT> ? kLoads<WT, KS> : 1];
  f32x4 xm[kQ4<WT> ? KS : 1];
};

__device__ __forceinline__ uint32_t ldh(const char* base, uint32_t off) {
  return *(const DE_GLOBAL uint16_t*)((const DE_GLOBAL char*)base + off);
}

// The loads of the wave's fragment f of tile r into ring slot d.
template <typename WT, int KS, bool GATEUP, bool REREAD>
__device__ __forceinline__ void issue_fragment(Regs<WT, KS>& R, const Slice& c,
                                               const Lanes<WT, KS>& L, int rpt, int r, int rw,
                                               int f, int d, uint32_t mask) {
  const char* p = frag_base<WT, GATEUP>(c, rpt, r, rw, f);
#pragma unroll
  for (int j = 0; j < kLoads<WT, KS>; ++j) R.w[d][j] = ldw<REREAD>(p, load_off(L, j, mask));
  if constexpr (kQ4<WT>) {
    const char* ps = scale_base<WT, GATEUP>(c, rpt, r, rw, f);
#pragma unroll
    for (int j = 0; j < kLoads<WT, KS>; ++j) R.sc[d][j] = ldh(ps, load_off(L, j, mask) >> 3);
  }
}

// The loads of a slice's activations (as fp32 values).
template <typename WT, int KS, bool SHARED>
__device__ __forceinline__ void load_slice(Regs<WT, KS>& R, const Slice& c, const Lanes<WT, KS>& L,
                                           int lane) {
#pragma unroll
  for (int q = 0; q < KS; ++q) load_x<WT, KS, SHARED>(R.act[q], c.act, L, q, lane >> 4);
}

// Makes operands of them; the wave's LDS rows are cleared (units past the
// wave's columns stay zero).
template <typename WT, int KS>
__device__ __forceinline__ void enter_slice(Regs<WT, KS>& R, const Lanes<WT, KS>& L, char* st,
                                            int lane) {
  const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < kWaveStage<WT, KS>; i += kWave * 16)
    if (i + lane * 16 < kWaveStage<WT, KS>) *reinterpret_cast<u32x4*>(st + i + lane * 16) = z;
#pragma unroll
  for (int q = 0; q < KS; ++q) {
    split8(R.act[q], (L.ok >> q) & 1u);
    if constexpr (kQ4<WT>) {
      const uint32_t m8 = 0xc100c100u;  // two bf16 -8
      const u32x4 m[1] = {u32x4{m8, m8, m8, m8}};
      f32x4 c[1];
      products<1>(&R.act[q], m, c);
      R.xm[q] = c[0];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("" ::: "memory");
}

// One tile of the wave: its fragments' sums to buf.  The registers are
// refilled from tile nr of slice nc (lanes N; mask 0: nothing follows, the
// loads all read one word).
template <typename WT, int KS, bool GATEUP, bool REREAD>
__device__ __forceinline__ void tile(Regs<WT, KS>& R, const Slice& c, const Lanes<WT, KS>& L, int r,
                                     const Slice& nc, const Lanes<WT, KS>& N, int nr, uint32_t mask,
                                     int rpt, int rw, char* st, float* buf, int wave,
                                     int lane_in) {
  constexpr int NF = kFrags<WT>, D = Regs<WT, KS>::kDepth;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    // Opaque to the compiler: the LDS offsets are computed again for every
    // fragment instead of being kept in registers across them.
    int lane = lane_in;
    asm volatile("" : "+v"(lane));
    f32x4 acc;
    if constexpr (kQ4<WT>) {
      char* sst = st + 16 * kRowUnits<WT, KS> * 16;
      constexpr int LR = kLoadRows<WT, KS>;
#pragma unroll
      for (int j = 0; j < kLoads<WT, KS>; ++j) {
        *reinterpret_cast<u32x4*>(st + L.so + j * LR * kRowUnits<WT, KS> * 16) = R.w[f][j];
        *reinterpret_cast<uint16_t*>(sst + L.ss + j * LR * 16) = (uint16_t)R.sc[f][j];
      }
      issue_fragment<WT, KS, GATEUP, REREAD>(R, nc, N, rpt, nr, rw, f, f, mask);
      asm volatile("" ::: "memory");
      acc = fragment_sums_q4<KS>(R.act, R.xm, st, lane);
    } else {
      if (f + D < NF)
        stage<WT, KS, REREAD>(R.w[0], st, L, frag_base<WT, GATEUP>(c, rpt, r, rw, f + D), L, ~0u);
      else
        stage<WT, KS, REREAD>(R.w[0], st, L, frag_base<WT, GATEUP>(nc, rpt, nr, rw, f + D - NF), N,
                              mask);
      asm volatile("" ::: "memory");
      acc = fragment_sums<KS>(R.act, st, lane);
    }
    asm volatile("" ::: "memory");
    put_partial<WT>(buf, acc, f, c.nt, wave, lane);
  }
}

// The block's `count` > 0 tiles from tile r of slice v (then of every step-th
// slice after it).  True where the thread wrote a NaN.
template <typename WT, int KS, bool GATEUP, bool REREAD, bool SHARED>
__device__ __forceinline__ bool stream(const Tiles<WT, GATEUP>& tl, int v, int r, int step,
                                       int count, int lkw, float* red, int lane, int wave) {
  int nan = 0;
  const int ks = wave & ((1 << lkw) - 1), rw = wave >> lkw, rpt = tl.a.geo.rpt;
  Slice c = tl.slice(v);
  Lanes<WT, KS> L = lanes_of<WT, KS>(c, tl.tb, ks, lkw, lane);
  Regs<WT, KS> R;
  char* st = reinterpret_cast<char*>(red + kRedFloats<WT>) + wave * kWaveStage<WT, KS>;
  // The first activations go out before the weights: they arrive first and
  // are split while the weights are on their way.
  load_slice<WT, KS, SHARED && !GATEUP>(R, c, L, lane);
#pragma unroll
  for (int f = 0; f < Regs<WT, KS>::kDepth; ++f)
    issue_fragment<WT, KS, GATEUP, REREAD>(R, c, L, rpt, r, rw, f, f, ~0u);
  enter_slice<WT, KS>(R, L, st, lane);
  float* buf = red;
#pragma unroll 1
  for (int left = count; left > 0; --left) {
    // The tile after this one.
    Slice nc = c;
    Lanes<WT, KS> N = L;
    int nr = r + 1;
    const bool more = left > 1, fresh = more && nr >= c.tiles;
    if (fresh) {
      nc = tl.slice(v += step);
      N = lanes_of<WT, KS>(nc, tl.tb, ks, lkw, lane);
    }
    if (!more || fresh) nr = more ? 0 : r;
    tile<WT, KS, GATEUP, REREAD>(R, c, L, r, nc, N, nr, more ? ~0u : 0u, rpt, rw, st, buf, wave, lane);
    lds_barrier();
    tile_outputs<WT, GATEUP, SHARED>(c, tl.tb, rpt, r, lkw, buf, nan);
    buf = buf == red ? red + kRedBuf<WT> : red;
    // A later slice's are used at once: left in flight into the next tile,
    // where they may or may not be, they would make every tile wait for all
    // loads but its newest.
    if (fresh) {
      // (Offsets computed again, not kept in registers across the tile.)
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const Lanes<WT, KS> M = lanes_of<WT, KS>(nc, tl.tb, ks, lkw, ln);
      load_slice<WT, KS, SHARED && !GATEUP>(R, nc, M, ln);
      enter_slice<WT, KS>(R, M, st, ln);
    }
    c = nc;
    L = N;
    r = nr;
  }
  return nan != 0;
}

// Room for the member slices: lists that share no entry need no more.
__host__ __device__ __forceinline__ int slice_room(const RoutedSrc& r) {
  return r.max_union + r.pairs_max / kXP + 1;
}

// The member slices: every resident member's positions in groups of 16, in
// member order.  Each member's list has been checked by itself (fill_tables);
// lists that overlap could make more slices than there is room for, and those are
// dropped.  One wave; returns their number.
__device__ __forceinline__ int member_slices(const Tables& tb, int nu, int32_t* slc, int room,
                                             int lane) {
  int base = 0;
  for (int j0 = 0; j0 < nu; j0 += kWave) {
    const int j = j0 + lane;
    int ng = 0;
    if (j < nu && tb.mem[j].blk != nullptr) ng = (tb.mem[j].ntok + kXP - 1) / kXP;
    const int inc = wave_scan_i32(ng);
    const int first = base + inc - ng;
    for (int i = 0; i < ng && first + i < room; ++i) slc[first + i] = (j << 8) | i;
    base += __builtin_amdgcn_readlane(inc, 63);
  }
  return min(base, room);
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
template <typename WT, int KS, bool GATEUP, bool SHARED = false>
__device__ __forceinline__ MfmaTables mfma_tables(const GroupedArgs& a, int lane, int wave,
                                                  int* absent, int* nms) {
  MfmaTables mt;
  mt.tb = tables_at(a, kRedFloats<WT> + kStageFloats<WT, KS>);
  if (threadIdx.x == 0) {
    *absent = 0;
    *nms = 0;
  }
  int32_t* slc = slices_at(a, mt.tb);
  mt.slc = slc;
  if (GATEUP && a.fuse_route) {
    float z0[2][4];
    first_logits(a, wave, z0);
    // (route_lists starts with a barrier: absent is initialised.)
    mt.nu = uni(route_lists<SHARED>(a, mt.tb, z0, lane, wave, absent, slc, nms));
  } else if (a.has_routed) {
    __syncthreads();
    mt.nu = uni(fill_tables(a, mt.tb, absent));
    __syncthreads();
    if (wave == 0) {
      const int c = member_slices(mt.tb, mt.nu, slc, slice_room(a.r), lane);
      if (lane == 0) *nms = c;
    }
    __syncthreads();
  } else {
    mt.nu = mt.nms = 0;
    return mt;
  }
  mt.nms = uni(*nms);
  // A needed member without a slot: reported once per layer.
  if (GATEUP && *absent && !a.r.absent_ok && blockIdx.x == 0 && threadIdx.x == 0 &&
      a.r.status != nullptr)
    *(DE_GLOBAL int32_t*)a.r.status |= kStatusNotResident;
  return mt;
}

// Member `part` of `parts` equal shares of `total` tiles: first tile, and their
// number to `count`.
__device__ __forceinline__ int share(uint32_t total, uint32_t part, uint32_t parts, int& count) {
  const uint32_t each = uni((int)(total / parts)), rest = total - each * parts;
  count = (int)(each + (part < rest ? 1u : 0u));
  return (int)(part * each + min(part, rest));
}

// One pass over the tables of a block: the slices are known (slc, nms).  The
// block's share of the tiles is contiguous.  REREAD: one dense source and G
// position groups; the blocks are cut into G runs, and block i of every run
// takes the same rows for its group.  SHARED: blocks of this launch read what
// others wrote.
template <typename WT, int KS, bool GATEUP, bool REREAD = false, bool SHARED = false>
__device__ __forceinline__ void mfma_pass(const GroupedArgs& a, int arg, const Tables& tb,
                                          const int32_t* slc, int nms, int lane, int wave) {
  const Tiles<WT, GATEUP> tl{a, arg, tb, slc, nms};
  const auto start = [&](int block, int& v, int& r, int& step, int& count) {
    step = 1;
    if constexpr (REREAD) {
      const int G = a.geo.groups, run = gridDim.x / G, g = uni(block / run);
      const int lo = share(a.geo.ndt / G, block - g * run, run, count);
      const int chunk = uni(lo / a.geo.tiles[0]);
      v = chunk * G + g;
      r = lo - chunk * a.geo.tiles[0];
      step = G;
    } else {
      const int lo = share(tl.total(), block, gridDim.x, count);
      if (count > 0) tl.locate(lo, v, r);
    }
  };
  int v, r, step, count, block = blockIdx.x;
  start(block, v, r, step, count);
  if (count <= 0) return;
  const bool nan =
      stream<WT, KS, GATEUP, REREAD, SHARED>(tl, v, r, step, count, a.lkw, s_dyn, lane, wave);
  if constexpr (!kQ4<WT>) {
    if (__builtin_amdgcn_ballot_w64(nan) == 0ull) return;
    asm volatile("" : "+s"(block));  // computed again, not kept through the tiles
    start(block, v, r, step, count);
    plain_outputs<WT, GATEUP, SHARED>(tl, v, r, step, count, a.lkw, lane);
  }
}

// Host side: a with the geometry of its pass.
template <typename WT, bool GATEUP>
GroupedArgs with_geometry(GroupedArgs a) {
  MfmaGeom& g = a.geo;
  g.rpt = (kWavesPB >> a.lkw) * group_rows<WT, GATEUP>();
  g.groups = cdiv(a.T, kXP);
  g.tr = a.has_routed ? cdiv(GATEUP ? a.r.inter : a.H, g.rpt) : 1;
  g.nds = g.ndt = 0;
  for (int i = 0; i < a.n_dense; ++i) {
    const DenseSrc& d = a.dense[i];
    g.v0[i] = g.nds;
    g.t0[i] = g.ndt;
    g.tiles[i] = cdiv(GATEUP ? d.inter : d.rows, g.rpt);
    const int ns = g.groups * (GATEUP ? 1 : d.chunks);
    g.nds += ns;
    g.ndt += ns * g.tiles[i];
  }
  return a;
}

template <typename WT, int KS>
size_t mfma_lds(const GroupedArgs& a) {
  size_t b = (size_t)(kRedFloats<WT> + kStageFloats<WT, KS>)*4 + tables_bytes(a);
  if (a.has_routed) b += (size_t)slice_room(a.r) * 4;
  return b;
}

}  // namespace
}  // namespace de
