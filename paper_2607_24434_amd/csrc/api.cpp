// C ABI of the draft/verify hot path: argument checks (host only, before any
// HIP call), scratch layout, and the launch sequence of each layer call.
#include "../../include/draftexpert.h"
#include "de_common.h"
#include "draft_persistent.h"
#include "grouped_mfma.h"
#include "verify_fused.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <cstring>

namespace de {

const DevInfo& dev_info() {
  static DevInfo info[64];
  static bool ready[64] = {false};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!ready[dev]) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
      cus = 256;
    info[dev].device = dev;
    info[dev].num_cus = cus;
    ready[dev] = true;
  }
  return info[dev];
}

int draft_layer_chain(const de_moe_desc* d, int T, const float* x, const float* w_router,
                      const float* bias, const de_expert_table* routed, const void* shared_w,
                      const void* draft_w, float gamma, int r, float* y, int32_t* pred_idx,
                      float* pred_gate, const de_epilogue* epi, void* ws, size_t ws_bytes,
                      hipStream_t stream, bool logits_ready, const float* next_router);
int verify_layer_chain(const de_moe_desc* d, int T, const float* x, const float* w_router,
                       const float* bias, const de_expert_table* routed, const void* shared_w,
                       float* y, int32_t* topk_idx, float* topk_gate, int32_t* n_union,
                       int32_t* union_ids, int32_t* offsets, int32_t* tok_list, float* gate_list,
                       int32_t* pair_pos, const de_epilogue* epi, void* ws, size_t ws_bytes,
                       hipStream_t stream, bool logits_ready, const float* next_router);
int dense_swiglu_chain(int T, int H, int I, int wdtype, const float* x, const void* w, float* y,
                       const de_epilogue* epi, void* ws, size_t ws_bytes, hipStream_t stream,
                       const de_moe_desc* next_desc, void* next_ws, const float* next_router);

// Bytes of a [rows, cols] weight matrix and of a [G|U|D] expert block.
size_t mat_bytes(int wdtype, int rows, int cols) {
  if (wdtype == DE_Q4_0) return (size_t)rows * cols * 9 / 16;
  return (size_t)rows * cols * (wdtype == DE_BF16 ? 2 : 4);
}

size_t expert_bytes(int wdtype, int inter, int hidden) {
  return 2 * mat_bytes(wdtype, inter, hidden) + mat_bytes(wdtype, hidden, inter);
}

// Host checks of an expert table against a layer shape (also used by the
// model calls before they enqueue anything).
int check_table(const de_moe_desc& d, const de_expert_table* t) {
  if (t == nullptr || t->base == nullptr || (reinterpret_cast<uintptr_t>(t->base) & 15u) != 0)
    return DE_ERR_INVALID;
  const int64_t need = (int64_t)expert_bytes(d.wdtype, d.inter, d.hidden);
  if (t->slot_stride_bytes < need || (t->slot_stride_bytes & 15) != 0) return DE_ERR_INVALID;
  if (t->n_slots < 1) return DE_ERR_INVALID;
  if (t->slot_of_expert == nullptr && t->n_slots < d.n_experts) return DE_ERR_INVALID;
  return DE_OK;
}

thread_local hipError_t t_last_hip = hipSuccess;

hipError_t note_hip(hipError_t e) {
  if (e != hipSuccess) t_last_hip = e;
  return e;
}

}  // namespace de

namespace {

constexpr int kMaxT = 64;
constexpr int kMaxK = 32;
constexpr int kMaxN = 256;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
size_t up256(size_t v) { return (v + 255) & ~size_t(255); }
int elem_bytes(int wdtype) { return wdtype == DE_BF16 ? 2 : 4; }
// Element alignment of every row length (16-byte rows; Q4_0: whole blocks).
int elem_align(int wdtype) { return wdtype == DE_Q4_0 ? 32 : (wdtype == DE_BF16 ? 8 : 4); }

// The shared path's down projection runs as up to this many dense sources
// (intermediate chunks), each with its own [T, H] partial.
constexpr int kMaxSharedChunks = 3;
// A dense layer's, on the matrix cores (on the vector ALU kMaxSharedChunks).
constexpr int kMaxDenseChunks = 3 + de::kMaxMore;

// Chunks of the shared intermediate for the down pass: the fewest (up to
// max_chunks) whose T input rows fit 64 KB and that are no wider than
// `width` (the routed experts' intermediate, so that every down tile of the
// launch streams rows of about the same length), each a whole number of
// 16-byte weight units; when none qualifies, the valid split with the
// smallest chunk.
int shared_chunks(int inter, int T, int max_chunks, int align, int width) {
  int best = 1;
  for (int c = 1; c <= max_chunks; ++c) {
    if (inter % c != 0 || (inter / c) % align != 0) continue;
    if ((size_t)T * (inter / c) * 4 <= 64 * 1024 && inter / c <= width) return c;
    best = c;
  }
  return best;
}

// The grouped passes of a MoE layer on the matrix cores (on = false: on the
// vector ALU).
struct MfmaPlan {
  bool on;
  int chunks, cw;      // the shared down projection's column chunks and their width
  int lkw_gu, lkw_dn;  // log2 of the column slices of a block
};

// Width of n column chunks of a K-column reduction (the last may be narrower),
// and the number of chunks that have columns.
int chunk_width(int K, int n, int align) { return (K / align + n - 1) / n * align; }
int chunk_count(int K, int n, int align) {
  return (K + chunk_width(K, n, align) - 1) / chunk_width(K, n, align);
}

// Blocks of two positions or more whose sources' columns fit the waves'
// registers.  V2-Lite layer, gate/up + down, us on the matrix cores against
// the vector ALU: bf16 T = 2 54 against 57, T = 9 120 against 136, T = 64 234
// against 802; Q4_0 T = 9 76 against 113.  (One bf16 position is the same within
// the runs' spread, and the persistent draft pass computes it in the vector ALU's
// order.)  Two Q4_0 positions of few experts stay on the vector ALU where a row of
// codes fills its waves: there the layer is bound by a fragment's way to the matrix
// cores.  Whole layer of 2048 columns (I = 1408, no shared block), us there and on
// the vector ALU: one expert a position 30 and 23, three 35 and 30, six 42 and 37,
// eight 45 and 45; 1024 columns: two experts 25 and 26, six 26 and 32.  The plan
// follows from the layer's shape and the block alone, so that calls over parts of a
// layer (an expert cache's chunks) sum in the same order.
MfmaPlan mfma_plan(const de_moe_desc& d, int T, int kk, bool has_shared, bool has_draft) {
  MfmaPlan p{};
  const int Is = has_shared ? d.shared_inter : 0, Id = has_draft ? d.draft_inter : 0;
  if (d.wdtype == DE_F32 || T < 2 || d.hidden > de::kMfmaMaxK || d.inter > de::kMfmaMaxK ||
      Id > de::kMfmaMaxK || !de::mfma_fits(d.wdtype, T, d.n_experts, d.top_k) ||
      (d.wdtype == DE_Q4_0 && T == 2 && kk <= 6 && d.hidden > 1024))
    return p;
  if (Is > 0) {
    // No wider than the routed experts' rows where possible, so that every
    // down tile of the launch streams about the same.
    const int most = kMaxSharedChunks - (Id > 0 ? 1 : 0);
    const int al = elem_align(d.wdtype);
    int n = 1;
    while (n < most && chunk_width(Is, n, al) > std::max(d.inter, 256)) ++n;
    p.cw = chunk_width(Is, n, al);
    p.chunks = chunk_count(Is, n, al);
    if (p.cw > de::kMfmaMaxK) return p;
  }
  const int mu = std::min(T * kk, d.n_experts);
  p.lkw_gu = de::mfma_lkw(d.wdtype, true, d.hidden, mu * d.inter + Is + Id);
  p.lkw_dn = de::mfma_lkw(d.wdtype, false, std::max(std::max(d.inter, p.cw), Id),
                          (mu + p.chunks + (Id > 0 ? 1 : 0)) * d.hidden);
  p.on = true;
  return p;
}

// True when the verify layer of this shape can run as one launch.
bool fused_shape(const de_moe_desc& d, int T) {
  return d.wdtype == DE_BF16 && T >= de::kVerifyFusedMinT && T <= de::kVerifyFusedMaxT &&
         mfma_plan(d, T, d.top_k, d.shared_inter > 0, false).on;
}

constexpr size_t kCtlBytes = 4096;
constexpr size_t kStatusOff = 256;
// The single-launch verify layer's arrival flags: at an offset that does not
// depend on the block length, which no other call writes (a call with
// another block length lays its buffers out differently).
constexpr size_t kFusedFlagsOff = 1024;
static_assert(kFusedFlagsOff + (de::kPDMaxGrid + 32) * 8 <= kCtlBytes, "control area");


struct Layout {
  size_t ctl, z, idx, gate, nu, uids, offs, tok, glist, ppos;
  size_t a_r, a_s, a_d, p_r, p_s, p_d;
  size_t total;
};

Layout layout(const de_moe_desc& d, int T) {
  Layout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t r = o;
    o += up256(bytes);
    return r;
  };
  const size_t tk = (size_t)T * d.top_k;
  // Control area: the routing launch's arrival counters [T] (zero after
  // de_workspace_init and after every call), the status word at byte 256
  // (sticky until de_layer_status reads it), the single-launch verify layer's
  // flags from byte 1024.
  L.ctl = take(kCtlBytes);
  L.z = take((size_t)T * d.n_experts * 4);
  L.idx = take(tk * 4);
  L.gate = take(tk * 4);
  L.nu = take(4);
  L.uids = take((size_t)d.n_experts * 4);
  L.offs = take(((size_t)d.n_experts + 1) * 4);
  L.tok = take(tk * 4);
  L.glist = take(tk * 4);
  L.ppos = take(tk * 4);
  // (The persistent draft pass keeps all its gate/up outputs, Is + Id + I of them,
  // from a_r on: a_r holds at least I.)
  L.a_r = take(tk * d.inter * 4);
  L.a_s = take((size_t)T * d.shared_inter * 4);
  L.a_d = take((size_t)T * d.draft_inter * 4);
  L.p_r = take(tk * d.hidden * 4);
  L.p_s = take((size_t)kMaxSharedChunks * T * d.hidden * 4);
  L.p_d = take((size_t)T * d.hidden * 4);
  L.total = o;
  return L;
}

// What de_workspace_bytes reports beyond what the calls use: room for a (value,
// epoch) word for every value of a single-launch verify layer, which its blocks once
// handed on in that form.  The size reported for these shapes stays what programs
// have sized their memory by; no call asks for the room.
size_t spare_bytes(const de_moe_desc& d, int T) {
  if (!fused_shape(d, T)) return 0;
  const size_t tk = (size_t)T * d.top_k;
  return up256((tk * (d.inter + d.hidden) + (size_t)T * d.shared_inter +
                (size_t)kMaxSharedChunks * T * d.hidden) * 8);
}

// Every launch that waits at device-wide points gets its own epoch (its arrival
// words are larger than those of earlier launches); 0 never occurs, so a zeroed
// word is always behind.
uint32_t next_epoch() {
  static std::atomic<uint32_t> epoch{1};
  const uint32_t e = epoch.fetch_add(1);
  return e != 0 ? e : epoch.fetch_add(1);
}

int check_T(int T) { return (T >= 1 && T <= kMaxT) ? DE_OK : DE_ERR_INVALID; }

int check_ws(const de_moe_desc& d, int T, const void* ws, size_t ws_bytes) {
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0) return DE_ERR_WORKSPACE;
  if (ws_bytes < layout(d, T).total) return DE_ERR_WORKSPACE;
  return DE_OK;
}

int check_epi(const de_epilogue* epi) {
  if (epi == nullptr) return DE_OK;
  if (epi->normed != nullptr && !(epi->eps >= 0.f)) return DE_ERR_INVALID;
  return DE_OK;
}

int hip_status(hipError_t e) { return de::note_hip(e) == hipSuccess ? DE_OK : DE_ERR_HIP; }

// Router logits (into the workspace) and the ordered top-k lists of every
// position; the layer calls build the union in their gate/up kernel.
hipError_t route(const de_moe_desc& d, int T, const float* x, const float* w_router,
                 const Layout& L, void* ws, const de::TopkUnionArgs& sel, hipStream_t s,
                 bool select = true) {
  de::RouteArgs r{};
  r.sel = sel;
  r.select = select ? 1 : 0;
  r.x = x;
  r.w = w_router;
  r.H = d.hidden;
  r.z = reinterpret_cast<float*>(static_cast<char*>(ws) + L.z);
  r.sel.z = r.z;
  r.counter = reinterpret_cast<unsigned*>(static_cast<char*>(ws) + L.ctl);
  return de::launch_route(r, s);
}

// One-shot phase timers armed by de_time_next_phase (per host thread).
thread_local hipEvent_t t_start[4] = {nullptr, nullptr, nullptr, nullptr};
thread_local hipEvent_t t_stop[4] = {nullptr, nullptr, nullptr, nullptr};

// Launches one phase with its armed events (if any) around it.
template <typename F>
hipError_t timed_phase(int phase, hipStream_t s, F launch) {
  hipEvent_t a = t_start[phase], b = t_stop[phase];
  t_start[phase] = t_stop[phase] = nullptr;
  if (a != nullptr && hipEventRecord(a, s) != hipSuccess) return hipErrorInvalidValue;
  const hipError_t e = launch();
  if (e != hipSuccess) return e;
  if (b != nullptr && hipEventRecord(b, s) != hipSuccess) return hipErrorInvalidValue;
  return hipSuccess;
}

// The single-launch verify layer: every armed phase timer brackets it (the
// gate/up and down phases both run inside it).
template <typename F>
hipError_t timed_layer(hipStream_t s, F launch) {
  hipEvent_t a[3], b[3];
  for (int i = 0; i < 3; ++i) {
    a[i] = t_start[i];
    b[i] = t_stop[i];
    t_start[i] = t_stop[i] = nullptr;
  }
  for (int i = 0; i < 3; ++i)
    if (a[i] != nullptr && hipEventRecord(a[i], s) != hipSuccess) return hipErrorInvalidValue;
  const hipError_t e = launch();
  if (e != hipSuccess) return e;
  for (int i = 0; i < 3; ++i)
    if (b[i] != nullptr && hipEventRecord(b[i], s) != hipSuccess) return hipErrorInvalidValue;
  return hipSuccess;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// kk: list entries per position that can enter the union (k, or 1 for the
// drafter's top-1), which bounds the union by T * kk.
de::RoutedSrc routed_src(const de_moe_desc& d, int T, int kk, const de_expert_table* tab,
                         const int32_t* nu, const int32_t* uids, const int32_t* offs,
                         const int32_t* tok, const float* glist, float* a_r, float* p_r,
                         int32_t* status) {
  de::RoutedSrc r{};
  r.status = status;
  r.absent_ok = 0;
  r.base = static_cast<const char*>(tab->base);
  r.stride = tab->slot_stride_bytes;
  r.slot_of_expert = tab->slot_of_expert;
  r.n_slots = tab->n_slots;
  r.n_union = nu;
  r.union_ids = uids;
  r.offsets = offs;
  r.tok_list = tok;
  r.gate_list = glist;
  r.max_union = T * kk < d.n_experts ? T * kk : d.n_experts;
  r.n_experts = d.n_experts;
  r.pairs_max = T * d.top_k;  // capacity of the lists, A_r and P_r
  r.inter = d.inter;
  r.a = a_r;
  r.p = p_r;
  return r;
}

// Chunks of a dense reduction of K columns for a matrix-core down pass of
// `rows` rows: 0 when even `most` chunks are too wide.
int mfma_chunks(int K, int rows, int T, int most) {
  int best = 0;
  long cost = 0;
  const int cus = de::dev_info().num_cus;
  for (int n = 1; n <= most; ++n) {
    const int cw = chunk_width(K, n, 8);
    if (cw > de::kMfmaMaxK || chunk_count(K, n, 8) != n) continue;
    const long tiles = (long)n * ((rows + 31) / 32) * ((T + 15) / 16);
    const long c = (tiles + cus - 1) / cus * ((cw + 255) / 256);
    if (best == 0 || c < cost) {
      best = n;
      cost = c;
    }
  }
  return best;
}

// What the launches of a device whose blocks wait for each other (drafted
// positions, the single-launch verify layer) know of each other.  All blocks of
// one have to be resident: two launches on two streams could each hold a part of
// the chip.  A launch therefore joins only its own stream's, or goes out once the
// last one's blocks need nothing more of the chip (its epoch is then in *done,
// which it writes); else the caller's separate launches run, with the same bits.
struct PDDevice {
  std::mutex mu;
  uint32_t* done = nullptr;  // pinned host word; NULL: not allocated yet
  hipStream_t stream = nullptr;
  uint32_t epoch = 0;        // the last launch's; 0: none yet
};
constexpr int kPDDevices = 64;

PDDevice* pd_device() {
  static PDDevice devs[kPDDevices];
  const int i = de::dev_info().device;
  return i >= 0 && i < kPDDevices ? &devs[i] : nullptr;
}

// True when such a launch may go to stream s now (p.mu is held).
bool pd_may_launch(PDDevice& p, hipStream_t s) {
  // Under capture a replay would find its own epoch in the flags.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return false;
  }
  if (p.done == nullptr) {
    // (Another stream may be under capture, which forbids allocations and would be
    // spoilt by one, except in the thread's relaxed mode.)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    void* w = nullptr;
    const hipError_t e = hipHostMalloc(&w, sizeof(uint32_t), hipHostMallocMapped);
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) {  // the next call tries again
      (void)hipGetLastError();
      return false;
    }
    p.done = static_cast<uint32_t*>(w);
    __atomic_store_n(p.done, 0u, __ATOMIC_RELAXED);
  }
  if (p.epoch == 0 || __atomic_load_n(p.done, __ATOMIC_ACQUIRE) == p.epoch) return true;
  // (One handle stands for every thread's own stream.)
  return s == p.stream && s != hipStreamPerThread;
}

// gate/up + down + combine over the union (kk entries per position) and the
// dense sources (shared path with gate 1, optionally the draft expert).
// With dense_on false the dense sources are left out of the two grouped
// launches (their partials from an earlier call stay in the workspace); with
// combine_on false the combine is not launched.  Both true for a whole layer.
int run_grouped(const de_moe_desc& d, int T, const float* x, const de::RoutedSrc& r,
                const int32_t* pair_pos, int kk, const void* shared_w, const void* draft_w,
                float gamma, float* y, const de_epilogue* epi, const Layout& L, void* ws,
                const de::TopkUnionArgs* fused_sel, hipStream_t s, bool dense_on = true,
                bool combine_on = true, bool fuse_select = false,
                const float* next_router = nullptr) {
  bool fused = fused_sel != nullptr && fuse_select && dense_on && combine_on &&
               next_router == nullptr && draft_w == nullptr && !r.absent_ok &&
               fused_shape(d, T) && de::verify_fused_enabled() &&
               de::dev_info().num_cus <= de::kPDMaxGrid;
  PDDevice* const dev = fused ? pd_device() : nullptr;
  std::unique_lock<std::mutex> lock;
  if (fused) {
    if (dev != nullptr) lock = std::unique_lock<std::mutex>(dev->mu);
    fused = dev != nullptr && pd_may_launch(*dev, s);
    if (!fused && lock.owns_lock()) lock.unlock();
  }
  const bool q4 = d.wdtype == DE_Q4_0;
  const size_t esz = q4 ? 0 : elem_bytes(d.wdtype);
  de::GroupedArgs g{};
  if (fused_sel != nullptr) {
    g.fuse_route = 1;
    g.fuse_select = fuse_select ? 1 : 0;
    g.sel = *fused_sel;
  }
  g.T = T;
  g.H = d.hidden;
  g.x = x;
  g.has_routed = 1;
  g.r = r;
  g.n_dense = 0;
  de::CombineArgs c{};
  c.T = T;
  c.H = d.hidden;
  c.n_dense = 0;
  if (dense_on && shared_w != nullptr && d.shared_inter > 0) {
    de::DenseSrc& ds = g.dense[g.n_dense++];
    ds.w = shared_w;
    ds.inter = d.shared_inter;
    ds.out = at<float>(ws, L.a_s);
  }
  if (dense_on && draft_w != nullptr && d.draft_inter > 0) {
    de::DenseSrc& ds = g.dense[g.n_dense++];
    ds.w = draft_w;
    ds.inter = d.draft_inter;
    ds.out = at<float>(ws, L.a_d);
  }
  const bool has_draft = draft_w != nullptr && d.draft_inter > 0;
  const MfmaPlan mx = mfma_plan(d, T, kk, shared_w != nullptr && d.shared_inter > 0, has_draft);
  g.mfma = mx.on ? 1 : 0;
  g.lkw = mx.lkw_gu;
  hipError_t e = hipSuccess;
  de::FusedArgs f{};
  if (fused) {
    f.gu = g;
  } else {
    e = timed_phase(DE_PHASE_GATEUP, s, [&] { return de::launch_gateup(g, d.wdtype, s); });
    if (e != hipSuccess) return DE_ERR_HIP;
  }
  g.lkw = mx.lkw_dn;
  // The down pass reads the gate/up activations of each dense source.  The
  // shared path's down projection is split along its intermediate dimension
  // into chunks whose block of input rows fits a down block's LDS staging
  // (two chunks for two 1408-wide shared experts at T = 9); each chunk writes
  // its own partial, and the combine sums them.
  int nd = 0;
  if (shared_w != nullptr && d.shared_inter > 0) {
    const int max_chunks = kMaxSharedChunks - (has_draft ? 1 : 0);
    const int chunks = mx.on ? mx.chunks
                             : shared_chunks(d.shared_inter, T, max_chunks, elem_align(d.wdtype),
                                             d.inter);
    const int cl = mx.on ? mx.cw : d.shared_inter / chunks;
    const char* D = static_cast<const char*>(shared_w) +
                    2 * de::mat_bytes(d.wdtype, d.shared_inter, d.hidden);
    c.n_dense = 0;
    if (mx.on) {
      de::DenseSrc& ds = g.dense[nd++];
      ds = de::DenseSrc{};
      ds.w = D;
      ds.ws = q4 ? D + (size_t)d.hidden * d.shared_inter / 2 : nullptr;
      ds.inter = d.shared_inter;
      ds.rows = d.hidden;
      ds.gate = 1.0f;
      ds.vin = at<float>(ws, L.a_s);
      ds.vin_stride = d.shared_inter;
      ds.out = at<float>(ws, L.p_s);
      ds.out_stride = d.hidden;
      ds.chunks = chunks;
      ds.cw = cl;
      ds.chunk_out = T * d.hidden;
    }
    for (int i = 0; i < chunks; ++i) {
      c.dense_p[c.n_dense++] = at<float>(ws, L.p_s) + (size_t)i * T * d.hidden;
      if (mx.on) continue;
      de::DenseSrc& ds = g.dense[nd++];
      // Columns [i cl, (i+1) cl) of D; Q4_0: their codes, and their scales
      // after the matrix's codes.
      ds.w = D + (q4 ? (size_t)i * cl / 2 : (size_t)i * cl * esz);
      ds.ws = q4 ? D + (size_t)d.hidden * d.shared_inter / 2 + (size_t)i * cl / 16 : nullptr;
      ds.inter = cl;
      ds.ld = d.shared_inter;
      ds.rows = d.hidden;
      ds.gate = 1.0f;
      ds.vin = at<float>(ws, L.a_s) + (size_t)i * cl;
      ds.vin_stride = d.shared_inter;
      ds.out = at<float>(ws, L.p_s) + (size_t)i * T * d.hidden;
      ds.out_stride = d.hidden;
    }
  }
  if (has_draft) {
    de::DenseSrc& ds = g.dense[nd++];
    ds.w = static_cast<const char*>(draft_w) + 2 * de::mat_bytes(d.wdtype, d.draft_inter, d.hidden);
    ds.ws = q4 ? static_cast<const char*>(ds.w) + (size_t)d.hidden * d.draft_inter / 2 : nullptr;
    ds.inter = d.draft_inter;
    ds.ld = d.draft_inter;
    ds.rows = d.hidden;
    ds.gate = gamma;
    ds.vin = at<float>(ws, L.a_d);
    ds.vin_stride = d.draft_inter;
    ds.out = at<float>(ws, L.p_d);
    ds.out_stride = d.hidden;
    ds.chunks = 1;
    ds.cw = d.draft_inter;
    c.dense_p[c.n_dense++] = ds.out;
  }
  g.n_dense = dense_on ? nd : 0;  // the combine reads the dense partials either way
  g.fuse_route = 0;
  c.p_r = r.p;
  c.pair_pos = pair_pos;
  c.kk = kk;
  c.pairs_max = r.pairs_max;
  c.y = y;
  c.residual = epi ? epi->residual : nullptr;
  c.normed = epi ? epi->normed : nullptr;
  c.eps = epi ? epi->eps : 0.f;
  if (fused) {
    f.dn = g;
    f.c = c;
    f.flags = at<uint64_t>(ws, kFusedFlagsOff);
    f.epoch = next_epoch();
    f.status = r.status;
    f.done = dev->done;
    e = timed_layer(s, [&] { return de::launch_verify_fused(f, s); });
    if (e == hipSuccess) {
      dev->stream = s;
      dev->epoch = f.epoch;
    }
    return hip_status(e);
  }
  e = timed_phase(DE_PHASE_DOWN, s, [&] { return de::launch_down(g, d.wdtype, s); });
  if (e != hipSuccess) return DE_ERR_HIP;
  if (!combine_on) return DE_OK;
  if (next_router != nullptr) {
    // The next layer's router logits go to this workspace's logit rows, where
    // the next layer call (same shape, T and workspace) reads them.
    de::RouteArgs nr{};
    nr.sel.T = T;
    nr.sel.N = d.n_experts;
    nr.w = next_router;
    nr.H = d.hidden;
    nr.z = at<float>(ws, L.z);
    return hip_status(de::launch_combine_route(c, nr, s));
  }
  return hip_status(de::launch_combine(c, s));
}

}  // namespace

namespace de {

int32_t* layer_status_word(void* ws) { return at<int32_t>(ws, kStatusOff); }

size_t layer_scratch_bytes(const de_moe_desc& d, int T) { return layout(d, T).total; }
size_t layer_values_offset(const de_moe_desc& d, int T) { return layout(d, T).a_r; }

// The LM head of a block of positions runs on the matrix cores unless
// DE_LMHEAD_MFMA is "0" (the vector-ALU row-dot then runs; the two differ only
// in the fp32 summation order).
bool lmhead_mfma_enabled() {
  const char* e = std::getenv("DE_LMHEAD_MFMA");
  return e == nullptr || e[0] != '0';
}

// The verify layer runs as one launch, where its shape allows, only when
// DE_VERIFY_FUSED is "1": every block waits at its two device-wide points for the
// slowest one, and it is slower than the separate launches (both give the same
// bits).
bool verify_fused_enabled() {
  const char* e = std::getenv("DE_VERIFY_FUSED");
  return e != nullptr && e[0] == '1';
}

// The persistent draft pass is used unless DE_DRAFT_PERSISTENT is "0" (the
// separate launches then run every draft layer; both give the same bits).
bool draft_persistent_enabled() {
  const char* e = std::getenv("DE_DRAFT_PERSISTENT");
  return e == nullptr || e[0] != '0';
}

// The single draft layer calls (T = 1, r = 1) through the persistent kernel
// as well; DE_PD_SINGLE=0 keeps them on the separate launches.
bool pd_single_enabled() {
  const char* e = std::getenv("DE_PD_SINGLE");
  return e == nullptr || e[0] != '0';
}

// Runs draft layers layers[0..n) (n >= 1) of one position (T = 1, the top-1
// drafter of Eq. 5) in persistent launches of at most kPDMaxLayers layers.  x_in is the
// first layer's input RMSNorm(h), h_in its residual (NULL: y = layer(x));
// z_ready: the first layer's router logits are already in the workspace's
// logit row.  Returns kPDNotApplicable, before enqueueing anything, when the
// shape or the layers do not fit the kernel, another stream's launch is under
// way or the stream is being captured.
int draft_persistent_run(const de_moe_desc& d, int n, const PDLayer* layers, const float* x_in,
                         const float* h_in, bool z_ready, float* y_out, float* normed_out,
                         int32_t* pred_idx, float* pred_gate, float eps, void* ws,
                         size_t ws_bytes, hipStream_t s) {
  if (!draft_persistent_enabled() || n < 1 || d.wdtype == DE_F32) return kPDNotApplicable;
  if (ws == nullptr || ws_bytes < layout(d, 1).total) return kPDNotApplicable;
  if (n > kPDMaxLayers && normed_out == nullptr) return kPDNotApplicable;
  // Every layer with a draft block, or none (then the term is dropped).
  const bool has_draft = d.draft_inter > 0 && layers[0].draft != nullptr;
  for (int l = 0; l < n; ++l)
    if ((d.draft_inter > 0 && (layers[l].draft != nullptr) != has_draft) ||
        (d.shared_inter > 0 && !layers[l].shared))
      return kPDNotApplicable;
  // The shared down projection in the chunks the separate launches use.
  const int max_chunks = kMaxSharedChunks - (has_draft ? 1 : 0);
  const int chunks =
      d.shared_inter > 0 ? shared_chunks(d.shared_inter, 1, max_chunks, elem_align(d.wdtype), d.inter)
                         : 0;
  const PDShape sh{d.wdtype, d.hidden, d.n_experts, d.top_k, d.inter, d.shared_inter,
                   has_draft ? d.draft_inter : 0, chunks, chunks > 0 ? d.shared_inter / chunks : 0};
  const int grid = dev_info().num_cus;
  if (!draft_persistent_fits(sh, grid, nullptr, nullptr)) return kPDNotApplicable;
  PDDevice* const dev = pd_device();
  if (dev == nullptr) return kPDNotApplicable;
  std::lock_guard<std::mutex> lock(dev->mu);
  if (!pd_may_launch(*dev, s)) return kPDNotApplicable;
  const Layout L = layout(d, 1);
  PDArgs a{};
  a.wdtype = d.wdtype;
  a.done = dev->done;
  a.H = d.hidden;
  a.N = d.n_experts;
  a.k = d.top_k;
  a.I = d.inter;
  a.Is = d.shared_inter;
  a.Id = sh.Id;
  a.n_chunks = sh.n_chunks;
  a.chunk = sh.chunk;
  a.has_draft = has_draft ? 1 : 0;
  a.score_func = d.score_func;
  a.norm_topk = d.norm_topk;
  a.routed_scale = d.routed_scale;
  a.eps = eps;
  a.grid = grid;
  a.spin_limit = 1u << 20;
  a.lds_bytes = draft_persistent_lds(sh);
  a.a_buf = at<float>(ws, L.a_r);
  a.z_plain = at<float>(ws, L.z);
  a.status = at<int32_t>(ws, kStatusOff);
  for (int l0 = 0; l0 < n; l0 += kPDMaxLayers) {
    const int cnt = n - l0 < kPDMaxLayers ? n - l0 : kPDMaxLayers;
    a.L = cnt;
    for (int i = 0; i < cnt; ++i) a.layers[i] = layers[l0 + i];
    // Later launches continue from the previous one's output (read by every
    // block before any block writes the output rows).
    a.x_in = l0 == 0 ? x_in : normed_out;
    a.h_in = l0 == 0 ? h_in : y_out;
    a.z_in = (l0 == 0 && z_ready) ? a.z_plain : nullptr;
    a.y_out = y_out;
    a.normed_out = normed_out;
    a.pred_idx = pred_idx ? pred_idx + (size_t)l0 * d.top_k : nullptr;
    a.pred_gate = pred_gate ? pred_gate + (size_t)l0 * d.top_k : nullptr;
    a.epoch = next_epoch();
    const hipError_t e =
        timed_phase(DE_PHASE_DRAFT_PASS, s, [&] { return launch_draft_persistent(a, s); });
    if (e != hipSuccess) {
      // A launch that never started (the device cannot hold the grid, for
      // instance) leaves the work to the separate launches.
      if (l0 == 0 && (e == hipErrorCooperativeLaunchTooLarge || e == hipErrorNotSupported))
        return kPDNotApplicable;
      return DE_ERR_HIP;
    }
    dev->stream = s;
    dev->epoch = a.epoch;
  }
  return DE_OK;
}

PDLayer pd_layer(const de_layer_weights& w) {
  PDLayer p{};
  p.w_router = w.w_router;
  p.bias = w.bias;
  p.routed = static_cast<const char*>(w.routed.base);
  p.stride = w.routed.slot_stride_bytes;
  p.slot_of_expert = w.routed.slot_of_expert;
  p.n_slots = w.routed.n_slots;
  p.shared = static_cast<const char*>(w.shared_w);
  p.draft = static_cast<const char*>(w.draft_w);
  p.gamma = w.gamma;
  return p;
}

// Reads the status word after the stream's work so far, clears it, and maps
// its bits to a return code (a missing expert first).
int take_status(int32_t* word, hipStream_t stream) {
  int32_t v = 0;
  if (hipMemcpyAsync(&v, word, sizeof(v), hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return DE_ERR_HIP;
  if (v == 0) return DE_OK;
  if (hipMemsetAsync(word, 0, sizeof(v), stream) != hipSuccess) return DE_ERR_HIP;
  return (v & kStatusNotResident) ? DE_ERR_NOT_RESIDENT : DE_ERR_INVALID;
}

// The grouped part of a layer whose routing already ran: the union of the
// first `ucols` entries of each position's lists idx / gate [T, k] (device),
// built in the gate/up prologue, then gate/up and down over the members the
// table marks resident, with the dense sources when dense_on, and the combine
// when combine_on.  Calls over the same lists with disjoint resident members
// (dense_on in exactly one, combine_on in the last) produce the same bits as
// one call with every member resident: each pair's partial is written once,
// and the combine sums them in list order.
int layer_after_route(const de_moe_desc& d, int T, const float* x, const de_expert_table* routed,
                      const int32_t* idx, const float* gate, int ucols, const void* shared_w,
                      const void* draft_w, float gamma, float* y, const de_epilogue* epi,
                      bool dense_on, bool combine_on, int32_t* n_union, void* ws,
                      size_t ws_bytes, hipStream_t stream) {
  int rc = de_check_desc(&d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (!x || !idx || !gate || !y || !aligned16(x) || ucols < 1 || ucols > d.top_k)
    return DE_ERR_INVALID;
  if (d.shared_inter > 0 && (shared_w == nullptr || !aligned16(shared_w))) return DE_ERR_INVALID;
  if (draft_w != nullptr && !aligned16(draft_w)) return DE_ERR_INVALID;
  if (!std::isfinite(gamma)) return DE_ERR_INVALID;
  if ((rc = check_table(d, routed)) != DE_OK) return rc;
  if ((rc = check_epi(epi)) != DE_OK) return rc;
  if ((rc = check_ws(d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(d, T);
  TopkUnionArgs a{};
  a.T = T;
  a.N = d.n_experts;
  a.k = d.top_k;
  a.score_func = d.score_func;
  a.norm_topk = d.norm_topk;
  a.routed_scale = d.routed_scale;
  a.idx_out = const_cast<int32_t*>(idx);  // read only: the prologue copies the lists
  a.gate_out = const_cast<float*>(gate);
  a.ucols = ucols;
  a.n_union = n_union ? n_union : at<int32_t>(ws, L.nu);
  a.union_ids = at<int32_t>(ws, L.uids);
  a.offsets = at<int32_t>(ws, L.offs);
  a.tok_list = at<int32_t>(ws, L.tok);
  a.gate_list = at<float>(ws, L.glist);
  a.pair_pos = at<int32_t>(ws, L.ppos);
  a.z = at<float>(ws, L.z);
  RoutedSrc r = routed_src(d, T, ucols, routed, a.n_union, a.union_ids, a.offsets, a.tok_list,
                           a.gate_list, at<float>(ws, L.a_r), at<float>(ws, L.p_r),
                           at<int32_t>(ws, L.ctl + kStatusOff));
  // The cache marks every member outside the requested chunk absent on
  // purpose: their work is skipped, not reported.
  r.absent_ok = 1;
  return run_grouped(d, T, x, r, a.pair_pos, ucols, shared_w, draft_w, gamma, y, epi, L, ws, &a,
                     stream, dense_on, combine_on);
}

}  // namespace de

extern "C" {

const char* de_hip_error_detail(void) {
  return de::t_last_hip == hipSuccess ? "" : hipGetErrorString(de::t_last_hip);
}

int de_check_desc(const de_moe_desc* d) {
  if (d == nullptr) return DE_ERR_INVALID;
  if (d->wdtype != DE_F32 && d->wdtype != DE_BF16 && d->wdtype != DE_Q4_0)
    return DE_ERR_UNSUPPORTED;
  if (d->score_func != DE_SOFTMAX && d->score_func != DE_SIGMOID) return DE_ERR_UNSUPPORTED;
  if (d->norm_topk != 0 && d->norm_topk != 1) return DE_ERR_INVALID;
  if (d->n_experts < 1 || d->n_experts > kMaxN) return DE_ERR_INVALID;
  if (d->top_k < 1 || d->top_k > kMaxK || d->top_k > d->n_experts) return DE_ERR_INVALID;
  const int al = elem_align(d->wdtype);
  if (d->hidden < al || d->hidden > (1 << 16) || d->hidden % al) return DE_ERR_INVALID;
  if (d->inter < al || d->inter > (1 << 17) || d->inter % al) return DE_ERR_INVALID;
  if (d->shared_inter < 0 || d->shared_inter > (1 << 17) || d->shared_inter % al) return DE_ERR_INVALID;
  if (d->draft_inter < 0 || d->draft_inter > (1 << 17) || d->draft_inter % al) return DE_ERR_INVALID;
  if (!std::isfinite(d->routed_scale)) return DE_ERR_INVALID;
  return DE_OK;
}

size_t de_workspace_bytes(const de_moe_desc* d, int T) {
  if (de_check_desc(d) != DE_OK || check_T(T) != DE_OK) return 0;
  return layout(*d, T).total + spare_bytes(*d, T);
}

int de_workspace_init(void* ws, size_t ws_bytes, hipStream_t stream) {
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || ws_bytes < 256)
    return DE_ERR_WORKSPACE;
  return hip_status(hipMemsetAsync(ws, 0, ws_bytes, stream));
}

int de_route_topk(const de_moe_desc* d, int T, const float* x, const float* w_router,
                  const float* bias, int32_t* topk_idx, float* topk_gate, void* ws,
                  size_t ws_bytes, hipStream_t stream) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (x == nullptr || w_router == nullptr || topk_idx == nullptr || topk_gate == nullptr)
    return DE_ERR_INVALID;
  if (!aligned16(x) || !aligned16(w_router) || d->hidden % 4) return DE_ERR_INVALID;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  de::TopkUnionArgs a{};
  a.T = T;
  a.N = d->n_experts;
  a.k = d->top_k;
  a.bias = bias;
  a.score_func = d->score_func;
  a.norm_topk = d->norm_topk;
  a.routed_scale = d->routed_scale;
  a.idx_out = topk_idx;
  a.gate_out = topk_gate;
  a.ucols = d->top_k;
  return hip_status(route(*d, T, x, w_router, L, ws, a, stream));
}

int de_expert_union(int T, int k, int N, const int32_t* topk_idx, const float* topk_gate,
                    int32_t* n_union, int32_t* union_ids, int32_t* offsets, int32_t* tok_list,
                    float* gate_list, int32_t* pair_pos, hipStream_t stream) {
  if (check_T(T) != DE_OK || N < 1 || N > kMaxN || k < 1 || k > kMaxK || k > N)
    return DE_ERR_INVALID;
  if (!topk_idx || !topk_gate || !n_union || !union_ids || !offsets || !tok_list || !gate_list ||
      !pair_pos)
    return DE_ERR_INVALID;
  de::TopkUnionArgs a{};
  a.T = T;
  a.N = N;
  a.k = k;
  a.z = nullptr;
  a.idx_in = topk_idx;
  a.gate_in = topk_gate;
  a.ucols = k;
  a.n_union = n_union;
  a.union_ids = union_ids;
  a.offsets = offsets;
  a.tok_list = tok_list;
  a.gate_list = gate_list;
  a.pair_pos = pair_pos;
  return hip_status(de::launch_union(a, stream));
}

int de_grouped_swiglu(const de_moe_desc* d, int T, const float* x, const de_expert_table* routed,
                      const int32_t* n_union, const int32_t* union_ids, const int32_t* offsets,
                      const int32_t* tok_list, const float* gate_list, const int32_t* pair_pos,
                      const void* shared_w, float* y, const de_epilogue* epi, void* ws,
                      size_t ws_bytes, hipStream_t stream) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (!x || !y || !n_union || !union_ids || !offsets || !tok_list || !gate_list || !pair_pos)
    return DE_ERR_INVALID;
  if (!aligned16(x)) return DE_ERR_INVALID;
  if (d->shared_inter > 0 && (shared_w == nullptr || !aligned16(shared_w))) return DE_ERR_INVALID;
  if ((rc = de::check_table(*d, routed)) != DE_OK) return rc;
  if ((rc = check_epi(epi)) != DE_OK) return rc;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  const de::RoutedSrc r = routed_src(*d, T, d->top_k, routed, n_union, union_ids, offsets,
                                     tok_list, gate_list, at<float>(ws, L.a_r),
                                     at<float>(ws, L.p_r), at<int32_t>(ws, L.ctl + kStatusOff));
  return run_grouped(*d, T, x, r, pair_pos, d->top_k, shared_w, nullptr, 0.f, y, epi, L, ws,
                     nullptr, stream);
}

int de_draft_layer_topr(const de_moe_desc* d, int T, const float* x, const float* w_router,
                        const float* bias, const de_expert_table* routed, const void* shared_w,
                        const void* draft_w, float gamma, int r, float* y, int32_t* pred_idx,
                        float* pred_gate, const de_epilogue* epi, void* ws, size_t ws_bytes,
                        hipStream_t stream) {
  return de::draft_layer_chain(d, T, x, w_router, bias, routed, shared_w, draft_w, gamma, r, y,
                               pred_idx, pred_gate, epi, ws, ws_bytes, stream, false, nullptr);
}

int de_draft_layer(const de_moe_desc* d, int T, const float* x, const float* w_router,
                   const float* bias, const de_expert_table* routed, const void* shared_w,
                   const void* draft_w, float gamma, float* y, int32_t* pred_idx,
                   float* pred_gate, const de_epilogue* epi, void* ws, size_t ws_bytes,
                   hipStream_t stream) {
  return de_draft_layer_topr(d, T, x, w_router, bias, routed, shared_w, draft_w, gamma, 1, y,
                             pred_idx, pred_gate, epi, ws, ws_bytes, stream);
}

int de_verify_layer(const de_moe_desc* d, int T, const float* x, const float* w_router,
                    const float* bias, const de_expert_table* routed, const void* shared_w,
                    float* y, int32_t* topk_idx, float* topk_gate, int32_t* n_union,
                    int32_t* union_ids, int32_t* offsets, int32_t* tok_list, float* gate_list,
                    int32_t* pair_pos, const de_epilogue* epi, void* ws, size_t ws_bytes,
                    hipStream_t stream) {
  return de::verify_layer_chain(d, T, x, w_router, bias, routed, shared_w, y, topk_idx,
                                topk_gate, n_union, union_ids, offsets, tok_list, gate_list,
                                pair_pos, epi, ws, ws_bytes, stream, false, nullptr);
}

}  // extern "C"

namespace de {

// The layer calls of a chain of MoE layers (the stacked model): with
// logits_ready the router logits were already written to the workspace by the
// previous layer's combine; with next_router this layer's combine also writes
// the next layer's logits (which needs epi->normed).
int draft_layer_chain(const de_moe_desc* d, int T, const float* x, const float* w_router,
                      const float* bias, const de_expert_table* routed, const void* shared_w,
                      const void* draft_w, float gamma, int r, float* y, int32_t* pred_idx,
                      float* pred_gate, const de_epilogue* epi, void* ws, size_t ws_bytes,
                      hipStream_t stream, bool logits_ready, const float* next_router) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (r < 1 || r > d->top_k) return DE_ERR_INVALID;
  if (!x || !w_router || !y || !aligned16(x) || !aligned16(w_router) || d->hidden % 4)
    return DE_ERR_INVALID;
  if (d->shared_inter > 0 && (shared_w == nullptr || !aligned16(shared_w))) return DE_ERR_INVALID;
  if (draft_w != nullptr && !aligned16(draft_w)) return DE_ERR_INVALID;
  if (!std::isfinite(gamma)) return DE_ERR_INVALID;
  if ((rc = de::check_table(*d, routed)) != DE_OK) return rc;
  if ((rc = check_epi(epi)) != DE_OK) return rc;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  de::TopkUnionArgs a{};
  a.T = T;
  a.N = d->n_experts;
  a.k = d->top_k;
  a.bias = bias;
  a.score_func = d->score_func;
  a.norm_topk = d->norm_topk;
  a.routed_scale = d->routed_scale;
  a.idx_out = pred_idx ? pred_idx : at<int32_t>(ws, L.idx);
  a.gate_out = pred_gate ? pred_gate : at<float>(ws, L.gate);
  a.ucols = r;  // the drafter reads only the r leading experts of each position
  // Without the predicted lists and the top-k renormalisation nothing reads
  // past the r leading entries: the prologue selects only those.
  a.rounds = (pred_idx == nullptr && pred_gate == nullptr && !d->norm_topk) ? r : 0;
  a.n_union = at<int32_t>(ws, L.nu);
  a.union_ids = at<int32_t>(ws, L.uids);
  a.offsets = at<int32_t>(ws, L.offs);
  a.tok_list = at<int32_t>(ws, L.tok);
  a.gate_list = at<float>(ws, L.glist);
  a.pair_pos = at<int32_t>(ws, L.ppos);
  a.z = at<float>(ws, L.z);
  // Logits only; the gate/up prologue selects the top-k in every block.
  if (next_router != nullptr && (epi == nullptr || epi->normed == nullptr)) return DE_ERR_INVALID;
  // One position with its leading expert: the persistent kernel runs the
  // whole layer (routing, gate/up, down, combine) in one launch, with the
  // same bits.
  if (T == 1 && r == 1 && !logits_ready && next_router == nullptr && pd_single_enabled()) {
    PDLayer pl{};
    pl.w_router = w_router;
    pl.bias = bias;
    pl.routed = static_cast<const char*>(routed->base);
    pl.stride = routed->slot_stride_bytes;
    pl.slot_of_expert = routed->slot_of_expert;
    pl.n_slots = routed->n_slots;
    pl.shared = static_cast<const char*>(shared_w);
    pl.draft = static_cast<const char*>(draft_w);
    pl.gamma = gamma;
    rc = draft_persistent_run(*d, 1, &pl, x, epi ? epi->residual : nullptr, false, y,
                              epi ? epi->normed : nullptr, pred_idx, pred_gate,
                              epi ? epi->eps : 0.f, ws, ws_bytes, stream);
    if (rc != kPDNotApplicable) return rc;
  }
  if (!logits_ready && route(*d, T, x, w_router, L, ws, a, stream, false) != hipSuccess)
    return DE_ERR_HIP;
  const de::RoutedSrc rs = routed_src(*d, T, r, routed, a.n_union, a.union_ids, a.offsets,
                                      a.tok_list, a.gate_list, at<float>(ws, L.a_r),
                                      at<float>(ws, L.p_r), at<int32_t>(ws, L.ctl + kStatusOff));
  return run_grouped(*d, T, x, rs, a.pair_pos, r, shared_w, draft_w, gamma, y, epi, L, ws, &a,
                     stream, true, true, true, next_router);
}

int verify_layer_chain(const de_moe_desc* d, int T, const float* x, const float* w_router,
                       const float* bias, const de_expert_table* routed, const void* shared_w,
                       float* y, int32_t* topk_idx, float* topk_gate, int32_t* n_union,
                       int32_t* union_ids, int32_t* offsets, int32_t* tok_list, float* gate_list,
                       int32_t* pair_pos, const de_epilogue* epi, void* ws, size_t ws_bytes,
                       hipStream_t stream, bool logits_ready, const float* next_router) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (!x || !w_router || !y || !aligned16(x) || !aligned16(w_router) || d->hidden % 4)
    return DE_ERR_INVALID;
  if (d->shared_inter > 0 && (shared_w == nullptr || !aligned16(shared_w))) return DE_ERR_INVALID;
  if ((rc = de::check_table(*d, routed)) != DE_OK) return rc;
  if ((rc = check_epi(epi)) != DE_OK) return rc;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  de::TopkUnionArgs a{};
  a.T = T;
  a.N = d->n_experts;
  a.k = d->top_k;
  a.bias = bias;
  a.score_func = d->score_func;
  a.norm_topk = d->norm_topk;
  a.routed_scale = d->routed_scale;
  a.idx_out = topk_idx ? topk_idx : at<int32_t>(ws, L.idx);
  a.gate_out = topk_gate ? topk_gate : at<float>(ws, L.gate);
  a.ucols = d->top_k;
  a.n_union = n_union ? n_union : at<int32_t>(ws, L.nu);
  a.union_ids = union_ids ? union_ids : at<int32_t>(ws, L.uids);
  a.offsets = offsets ? offsets : at<int32_t>(ws, L.offs);
  a.tok_list = tok_list ? tok_list : at<int32_t>(ws, L.tok);
  a.gate_list = gate_list ? gate_list : at<float>(ws, L.glist);
  a.pair_pos = pair_pos ? pair_pos : at<int32_t>(ws, L.ppos);
  a.z = at<float>(ws, L.z);
  // Logits only; the gate/up prologue selects the top-k in every block.
  if (next_router != nullptr && (epi == nullptr || epi->normed == nullptr)) return DE_ERR_INVALID;
  if (!logits_ready && route(*d, T, x, w_router, L, ws, a, stream, false) != hipSuccess)
    return DE_ERR_HIP;
  const de::RoutedSrc r = routed_src(*d, T, d->top_k, routed, a.n_union, a.union_ids,
                                     a.offsets, a.tok_list, a.gate_list, at<float>(ws, L.a_r),
                                     at<float>(ws, L.p_r), at<int32_t>(ws, L.ctl + kStatusOff));
  return run_grouped(*d, T, x, r, a.pair_pos, d->top_k, shared_w, nullptr, 0.f, y, epi, L, ws, &a,
                     stream, true, true, true, next_router);
}

int accept_len_embed(int K, int V, const float* target_logits, const int32_t* draft_tokens,
                     int32_t* target_argmax, int32_t* out, void* ws, size_t ws_bytes,
                     const void* emb, int H, float* h, float* normed, float eps,
                     hipStream_t stream);

}  // namespace de

extern "C" {

size_t de_accept_workspace_bytes(int K, int V) {
  if (K < 0 || K > 1024 || V < 1) return 0;
  const size_t rows = (size_t)K + 1, ch = (size_t)de::accept_chunks(V);
  return 256 + up256(rows * 4) + 2 * up256(rows * ch * 4);
}

int de_accept_len(int K, int V, const float* target_logits, const int32_t* draft_tokens,
                  int32_t* target_argmax, int32_t* out, void* ws, size_t ws_bytes,
                  hipStream_t stream) {
  return de::accept_len_embed(K, V, target_logits, draft_tokens, target_argmax, out, ws, ws_bytes,
                              nullptr, 0, nullptr, nullptr, 0.f, stream);
}

}  // extern "C"

namespace de {

// de_accept_len that also writes the bonus token's embedding row to h [H] and
// its RMSNorm to normed when emb (bf16 [V, H]) is not NULL.
int accept_len_embed(int K, int V, const float* target_logits, const int32_t* draft_tokens,
                     int32_t* target_argmax, int32_t* out, void* ws, size_t ws_bytes,
                     const void* emb, int H, float* h, float* normed, float eps,
                     hipStream_t stream) {
  if (K < 0 || K > 1024 || V < 1 || !target_logits || !target_argmax || !out) return DE_ERR_INVALID;
  if (K > 0 && draft_tokens == nullptr) return DE_ERR_INVALID;
  if (emb != nullptr && (H < 1 || h == nullptr || normed == nullptr)) return DE_ERR_INVALID;
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 ||
      ws_bytes < de_accept_workspace_bytes(K, V))
    return DE_ERR_WORKSPACE;
  const size_t rows = (size_t)K + 1;
  de::AcceptArgs a{};
  a.emb = static_cast<const uint16_t*>(emb);
  a.H = H;
  a.h = h;
  a.normed = normed;
  a.eps = eps;
  a.K = K;
  a.V = V;
  a.logits = target_logits;
  a.drafts = draft_tokens;
  a.amax = target_argmax;
  a.out = out;
  a.done_cnt = at<unsigned>(ws, 0);
  a.row_cnt = at<unsigned>(ws, 256);
  a.part = at<uint64_t>(ws, 256 + up256(rows * 4));
  return hip_status(de::launch_argmax_accept(a, stream));
}

}  // namespace de

extern "C" {

int de_lm_head(int T, int H, int V, const float* x, const void* w_lm, float* logits,
               hipStream_t stream) {
  if (check_T(T) != DE_OK || H < 8 || H % 8 || V < 1 || !x || !w_lm || !logits) return DE_ERR_INVALID;
  if (!aligned16(x) || !aligned16(w_lm)) return DE_ERR_INVALID;
  // On the matrix cores wherever a row's columns fit the waves' registers (102400
  // rows of 2048, us against the row-dot: T = 1 67 and 74, T = 4 69 and 77; 8192
  // rows 11 and 14).  Wider rows: 5 to 12 positions in a kernel that keeps their
  // parts in LDS, else the row-dot.
  const bool mx = H <= de::kMfmaMaxK && de::lmhead_mfma_enabled();
  if (!mx && de::rowdot_mfma_fits(T, H) && de::lmhead_mfma_enabled())
    return hip_status(de::launch_rowdot_mfma(T, H, V, x, w_lm, logits, stream));
  de::GroupedArgs g{};
  g.T = T;
  g.H = H;
  g.x = x;
  g.has_routed = 0;
  g.n_dense = 1;
  g.dense[0].w = w_lm;
  g.dense[0].inter = H;
  g.dense[0].rows = V;
  g.dense[0].gate = 1.0f;
  g.dense[0].vin = x;
  g.dense[0].vin_stride = H;
  g.dense[0].out = logits;
  g.dense[0].out_stride = V;
  if (mx) {
    g.mfma = 1;
    g.lkw = de::mfma_lkw(DE_BF16, false, H, V);
    g.dense[0].chunks = 1;
    g.dense[0].cw = H;
  }
  return hip_status(de::launch_down(g, DE_BF16, stream));
}

int de_rmsnorm(int T, int H, const float* x, float eps, float* out, hipStream_t stream) {
  if (T < 1 || T > 65536 || H < 1 || !x || !out || !(eps >= 0.f)) return DE_ERR_INVALID;
  return hip_status(de::launch_rmsnorm(T, H, x, eps, out, stream));
}

int de_embed_gather(int T, int H, int V, const int32_t* tokens, const void* emb, float* h,
                    float* normed, float eps, int32_t* status, hipStream_t stream) {
  if (T < 1 || T > 65536 || H < 1 || V < 1 || !tokens || !emb || !h || !(eps >= 0.f))
    return DE_ERR_INVALID;
  return hip_status(de::launch_embed(T, H, V, tokens, static_cast<const uint16_t*>(emb), h, normed,
                                     eps, status, stream));
}

int de_layer_status(void* ws, size_t ws_bytes, hipStream_t stream) {
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || ws_bytes < kCtlBytes)
    return DE_ERR_WORKSPACE;
  return de::take_status(de::layer_status_word(ws), stream);
}

size_t de_dense_workspace_bytes(int T, int H, int I) {
  if (check_T(T) != DE_OK || H < 1 || I < 1) return 0;
  return up256((size_t)T * I * 4) + (size_t)kMaxDenseChunks * up256((size_t)T * H * 4);
}

// Intermediate chunks of a dense layer's down pass: as many as there are
// dense sources (each a whole number of 16-byte units), so that its few
// output rows are streamed by three times the waves.
int dense_chunks(int I, int align) {
  for (int c = kMaxSharedChunks; c > 1; --c)
    if (I % c == 0 && (I / c) % align == 0) return c;
  return 1;
}

int de_dense_swiglu(int T, int H, int I, int wdtype, const float* x, const void* w, float* y,
                    const de_epilogue* epi, void* ws, size_t ws_bytes, hipStream_t stream) {
  return de::dense_swiglu_chain(T, H, I, wdtype, x, w, y, epi, ws, ws_bytes, stream, nullptr,
                                nullptr, nullptr);
}

}  // extern "C"

namespace de {

// The dense layer in a chain: with next_router, its combine also writes the
// following MoE layer's router logits (next_desc's shape) to that layer's
// workspace next_ws, where its call with the logits ready reads them.
int dense_swiglu_chain(int T, int H, int I, int wdtype, const float* x, const void* w, float* y,
                       const de_epilogue* epi, void* ws, size_t ws_bytes, hipStream_t stream,
                       const de_moe_desc* next_desc, void* next_ws, const float* next_router) {
  if (wdtype != DE_F32 && wdtype != DE_BF16) return DE_ERR_UNSUPPORTED;
  const int al = elem_align(wdtype);
  if (check_T(T) != DE_OK || H < al || H % al || I < al || I % al || I > (1 << 17))
    return DE_ERR_INVALID;
  if (!x || !w || !y || !aligned16(x) || !aligned16(w)) return DE_ERR_INVALID;
  if (check_epi(epi) != DE_OK) return DE_ERR_INVALID;
  if (next_router != nullptr &&
      (next_desc == nullptr || next_ws == nullptr || epi == nullptr || epi->normed == nullptr ||
       next_desc->hidden != H || !de::combine_route_fits(H) || !aligned16(next_router)))
    return DE_ERR_INVALID;
  if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 ||
      ws_bytes < up256((size_t)T * I * 4) + kMaxSharedChunks * up256((size_t)T * H * 4))
    return DE_ERR_WORKSPACE;
  float* A = static_cast<float*>(ws);
  float* P = at<float>(ws, up256((size_t)T * I * 4));
  const size_t pstride = up256((size_t)T * H * 4) / 4;
  de::GroupedArgs g{};
  g.T = T;
  g.H = H;
  g.x = x;
  g.has_routed = 0;
  g.n_dense = 1;
  g.dense[0].w = w;
  g.dense[0].inter = I;
  g.dense[0].out = A;
  // Down: D [H, I] in column chunks, each with its own partial.  (Their number
  // follows from the shape alone, whatever the scratch holds: the same sums.)
  int nc = 0;
  if (wdtype == DE_BF16 && H <= de::kMfmaMaxK) nc = mfma_chunks(I, H, T, kMaxDenseChunks);
  const bool mx = nc > 0;
  if (!mx) nc = dense_chunks(I, al);
  const int cw = (I / al + nc - 1) / nc * al;
  if (mx) {
    g.mfma = 1;
    g.lkw = de::mfma_lkw(wdtype, true, H, I);
  }
  if (timed_phase(DE_PHASE_GATEUP, stream, [&] { return de::launch_gateup(g, wdtype, stream); }) !=
      hipSuccess)
    return DE_ERR_HIP;
  if (mx) g.lkw = de::mfma_lkw(wdtype, false, cw, nc * H);
  const char* D = static_cast<const char*>(w) + 2 * (size_t)I * H * elem_bytes(wdtype);
  // The `n` chunks from chunk c0 on, to the partials from `slot` on.
  const auto down = [&](int c0, int n, int slot) {
    g.n_dense = mx ? 1 : n;
    for (int i = 0; i < g.n_dense; ++i) {
      const int col = (c0 + i) * cw;
      g.dense[i] = de::DenseSrc{};
      g.dense[i].w = D + (size_t)col * elem_bytes(wdtype);
      g.dense[i].inter = mx ? I - col : cw;
      g.dense[i].ld = I;
      g.dense[i].rows = H;
      g.dense[i].gate = 1.0f;
      g.dense[i].vin = A + (size_t)col;
      g.dense[i].vin_stride = I;
      g.dense[i].out = P + (size_t)(slot + i) * pstride;
      g.dense[i].out_stride = H;
      g.dense[i].chunks = n;
      g.dense[i].cw = cw;
      g.dense[i].chunk_out = (int)pstride;
    }
    return de::launch_down(g, wdtype, stream);
  };
  de::CombineArgs c{};
  c.T = T;
  c.H = H;
  c.more_stride = (int)pstride;
  const auto partials = [&](int n) {
    c.n_dense = std::min(n, 3);
    for (int i = 0; i < c.n_dense; ++i) c.dense_p[i] = P + (size_t)i * pstride;
    c.n_more = n - c.n_dense;
  };
  // A scratch of three partials or more that does not hold all of them: the sum of
  // the chunks so far is the first partial of the next group (the combine sums in
  // chunk order, from zero, so the bits are those of one group).
  const int fit = (int)std::min<size_t>(
      (ws_bytes - up256((size_t)T * I * 4)) / up256((size_t)T * H * 4), (size_t)nc);
  const hipError_t e = timed_phase(DE_PHASE_DOWN, stream, [&] {
    hipError_t r = down(0, fit, 0);
    partials(fit);
    for (int c0 = fit; c0 < nc && r == hipSuccess;) {
      c.y = P;
      if ((r = de::launch_combine(c, stream)) != hipSuccess) break;
      const int n = std::min(fit - 1, nc - c0);
      r = down(c0, n, 1);
      partials(n + 1);
      c0 += n;
    }
    return r;
  });
  if (e != hipSuccess) return DE_ERR_HIP;
  c.y = y;
  c.residual = epi ? epi->residual : nullptr;
  c.normed = epi ? epi->normed : nullptr;
  c.eps = epi ? epi->eps : 0.f;
  if (next_router != nullptr) {
    de::RouteArgs nr{};
    nr.sel.T = T;
    nr.sel.N = next_desc->n_experts;
    nr.w = next_router;
    nr.H = H;
    nr.z = at<float>(next_ws, layout(*next_desc, T).z);
    return hip_status(de::launch_combine_route(c, nr, stream));
  }
  return hip_status(de::launch_combine(c, stream));
}

}  // namespace de

extern "C" {

int de_verify_single_launch(const de_moe_desc* d, int T) {
  if (de_check_desc(d) != DE_OK || check_T(T) != DE_OK || !de::verify_fused_enabled()) return 0;
  return fused_shape(*d, T) ? 1 : 0;
}

int de_time_next_phase(int phase, hipEvent_t start, hipEvent_t stop) {
  if (phase != DE_PHASE_GATEUP && phase != DE_PHASE_DOWN && phase != DE_PHASE_LAYER &&
      phase != DE_PHASE_DRAFT_PASS)
    return DE_ERR_INVALID;
  t_start[phase] = start;
  t_stop[phase] = stop;
  return DE_OK;
}

int de_confidence(int T, int V, const float* logits, float* q, hipStream_t stream) {
  if (T < 1 || T > 65536 || V < 1 || !logits || !q) return DE_ERR_INVALID;
  return hip_status(de::launch_confidence(T, V, logits, q, stream));
}

int de_expansion(int L, int k, int N, const int32_t* pred_idx, uint64_t* uhat, int first,
                 const float* q, float tau, int budget, int slots, int32_t* out,
                 hipStream_t stream) {
  if (L < 1 || L > 65536 || N < 1 || N > 256 || k < 1 || k > N) return DE_ERR_INVALID;
  if (!pred_idx || !uhat || !q || !out || budget < DE_BUDGET_CACHE || slots < 0 ||
      tau != tau)
    return DE_ERR_INVALID;
  if ((reinterpret_cast<uintptr_t>(uhat) & 7u) != 0) return DE_ERR_INVALID;
  de::ExpansionArgs a{};
  a.L = L;
  a.k = k;
  a.N = N;
  a.pred = pred_idx;
  a.uhat = reinterpret_cast<unsigned long long*>(uhat);
  a.first = first != 0;
  a.q = q;
  a.tau = tau;
  a.budget = budget;
  a.slots = slots;
  a.out = out;
  return hip_status(de::launch_expansion(a, stream));
}

int de_residual_target(const de_moe_desc* d, int T, const void* ws, size_t ws_bytes,
                       float* m_star, hipStream_t stream) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (m_star == nullptr) return DE_ERR_INVALID;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  de::ResidualArgs a{};
  a.T = T;
  a.H = d->hidden;
  a.kk = d->top_k;
  a.pairs_max = T * d->top_k;
  a.p_r = at<float>(const_cast<void*>(ws), L.p_r);
  a.pair_pos = at<int32_t>(const_cast<void*>(ws), L.ppos);
  a.out = m_star;
  return hip_status(de::launch_residual(a, stream));
}

int de_layer_router_logits(const de_moe_desc* d, int T, const void* ws, size_t ws_bytes,
                           float* z, hipStream_t stream) {
  int rc = de_check_desc(d);
  if (rc != DE_OK) return rc;
  if ((rc = check_T(T)) != DE_OK) return rc;
  if (z == nullptr) return DE_ERR_INVALID;
  if ((rc = check_ws(*d, T, ws, ws_bytes)) != DE_OK) return rc;
  const Layout L = layout(*d, T);
  return hip_status(hipMemcpyAsync(z, static_cast<const char*>(ws) + L.z,
                                   (size_t)T * d->n_experts * 4, hipMemcpyDeviceToDevice,
                                   stream));
}

int de_row_kl(int rows, int n, const float* a, int lda, const float* b, int ldb,
              const float* bias, int sigmoid, float tau, float* kl, float* ce,
              hipStream_t stream) {
  if (rows < 1 || rows > (1 << 20) || n < 1 || lda < n || ldb < n) return DE_ERR_INVALID;
  if (!a || !b || !kl || !(tau > 0.f) || !std::isfinite(tau)) return DE_ERR_INVALID;
  if (sigmoid != 0 && (bias != nullptr || ce != nullptr || tau != 1.f)) return DE_ERR_INVALID;
  de::RowKlArgs r{};
  r.rows = rows;
  r.n = n;
  r.a = a;
  r.lda = lda;
  r.b = b;
  r.ldb = ldb;
  r.bias = bias;
  r.sigmoid = sigmoid != 0;
  r.tau = tau;
  r.kl = kl;
  r.ce = ce;
  return hip_status(de::launch_rowkl(r, stream));
}

int de_stream_probe(const void* buf, size_t bytes, float* sink, hipStream_t stream) {
  if (!buf || !sink || bytes == 0 || bytes % 16 || !aligned16(buf)) return DE_ERR_INVALID;
  return hip_status(de::launch_stream_probe(buf, bytes, sink, stream));
}

}  // extern "C"
