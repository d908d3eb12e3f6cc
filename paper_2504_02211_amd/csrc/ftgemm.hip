// Host side of the fault-tolerant linear layer: the C ABI of include/ftgemm.h.  Validation,
// launches and the report are here; encoding, the contraction, verification and repair run in
// the kernels of ftgemm_main.h.
#include "ftgemm_main.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

using namespace ftgemm;

struct ftgemm_ctx {
  ftgemm_config cfg;          // effective configuration
  int Tn = 0;
  void* scratch = nullptr;    // the device buffers below, in one allocation
  uint16_t* wc = nullptr;     // [Tn][32][k] checksum rows of the weights (input type)
  const void* encoded_w = nullptr;
  GFault* d_faults = nullptr;
  ftgemm_event* d_events = nullptr;   // ring, never cleared: the slots say which entries a call wrote
  uint32_t* d_cursor = nullptr;       // (a cache line to itself)
  int32_t* d_n_slots = nullptr;       // slots the last launch to run has written ...
  GSlot* d_slots = nullptr;           // ... and these, one GSlot behind, so that a report is one copy
  float4v* ws = nullptr;              // shares of a split contraction
  uint32_t ring_n = 0;
  int n_slots = 0;                    // allocated
  int last_slots = 0;                 // what the last call made here writes (a graph's replay may write another number)
  GFault* h_faults = nullptr; // pinned staging ...
  GSlot* h_slots = nullptr;   // ... and, behind it in the same block, where a report finds a copy of d_n_slots and d_slots
  int fault_cap = 0;
  std::vector<ftgemm_event> events;
  hipStream_t last_stream = nullptr;
  bool ran = false, timing = false;
  hipEvent_t ev[2] = {nullptr, nullptr};
  std::string err;
};

constexpr size_t CURSOR_BYTES = 128;

static thread_local std::string g_gemm_create_err;

static int gfail(ftgemm_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg; else g_gemm_create_err = msg;
  return code;
}

#define GHIP_TRY(ctx, expr)                                                                     \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return gfail(ctx, e_ == hipErrorOutOfMemory ? FTGEMM_ENOMEM : FTGEMM_EHIP,                \
                   std::string(#expr) + ": " + hipGetErrorString(e_));                          \
  } while (0)

static void grelease(ftgemm_ctx* c) {
  if (!c) return;
  (void)hipFree(c->scratch);
  if (c->h_faults) (void)hipHostFree(c->h_faults);
  for (hipEvent_t e : c->ev) if (e) (void)hipEventDestroy(e);
  delete c;
}

namespace ftgemm {

template <class T> static constexpr TileInfo info_of() { return TileInfo{T::BM, T::NW * 64, T::PER_CU, {T::template lds<false>(), T::template lds<true>()}}; }
static constexpr TileInfo TILES[N_TILES] = {info_of<TileWide>(), info_of<TileHalf>(), info_of<TileQuarter>(),
                                            info_of<TileStrip>(), info_of<TileNarrow>(), info_of<TileSlim>(),
                                            info_of<TileNarrow2>(), info_of<TileSlim2>(), info_of<TileLow>()};

static gemm_fn tile_kernel(int tile, bool ft, bool inject, bool bf16) {
  return bf16 ? tile_kernel_bf16(tile, ft, inject) : tile_kernel_f16(tile, ft, inject);
}

hipError_t gemm_allow_lds(GPlan plan, bool ft, bool bf16) {
  for (int inject = 0; inject < 2; ++inject) {
    const int tile = inject ? (int)TILE_QUARTER : plan.tile;
    hipError_t he = hipFuncSetAttribute((const void*)tile_kernel(tile, ft, inject != 0, bf16), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        TILES[tile].lds[ft]);
    if (he != hipSuccess) return he;
  }
  return hipSuccess;
}

hipError_t gemm_launch_encode_w(const uint16_t* w, uint16_t* wc, int n, int k, bool bf16, hipStream_t st, int batch,
                                long long bs_w, long long bs_wc) {
  dim3 grid((n + GBN - 1) / GBN, (k / 8 + 7) / 8, batch);
  if (bf16) ftgemm_encode_w<true><<<grid, 256, 0, st>>>(w, wc, n, k, bs_w, bs_wc);
  else ftgemm_encode_w<false><<<grid, 256, 0, st>>>(w, wc, n, k, bs_w, bs_wc);
  return hipGetLastError();
}

int gemm_slots(long long m, long long n, GPlan plan, bool skip_upper) {
  if (skip_upper) return lower_tiles((int)((m + TILES[plan.tile].bm - 1) / TILES[plan.tile].bm), TILES[plan.tile].bm);
  const int bm = plan.parts > 1 ? TileFinish::BM : TILES[plan.tile].bm;
  return (int)((m + bm - 1) / bm * ((n + GBN - 1) / GBN));
}

static int ws_tokens_of(long long m, GPlan plan) {
  const int bm = TILES[plan.tile].bm;
  return (int)((m + bm - 1) / bm * (bm / 16));
}

size_t gemm_workspace(long long m, long long n, GPlan plan) {
  if (plan.parts <= 1) return 0;
  return (size_t)plan.parts * ws_tokens_of(m, plan) * ((n + GBN - 1) / GBN) * WS_BLOCKS * 64 * sizeof(float4v);
}

// The tile shape and the split of K with the least expected time.  Microseconds, from timings of every
// shape at 1..16384 tokens, 64..16384 features, K 64..8192: a round of tiles (one per CU, two where two fit) costs
// `fixed` and `step` per 64 columns of K, the latter up to (1 + load) times as much when every CU has one (L2 traffic,
// power); a split adds the second launch and a pass of the shares through memory.  Wide tiles move the
// fewest bytes per product, narrow ones fill the chip: 4096^3 takes 119 / 141 / 177 / 255 us with tiles of
// 256 / 128 / 64 / 32 tokens, 5000 x 1300 x 8000 197 / 134 / 159 / 235, 2048 x 2048 x 1024 33 / 22 / 17 / 26, 128 x 1024 x 8192
// 161 / 110 / 70 / 56 unsplit and 18.5 with 32-token tiles split eight ways.
// 128 features or fewer have tiles of that width, which leave the products of the padding out, in two heights: the high
// ones read the weights half as often, the low ones run two to a CU.  16384 x 128 x 8192 takes 82 us with the
// high ones, 99 with the low and 126 with 32-token tiles of 256 features, 16384 x 100 x 512 18.0 / 12.9 / 23, 1000 x 100 x
// 1000 21.4 / 14.4 / 16.0; with K split the 32-token tiles take 18.9 for 37 x 100 x 8192 (69 / 46 unsplit), 20.4 for
// 2000 x 128 x 4096 (38 / 26) and 20.9 for 2000 x 64 x 4096 (44 / 27).
// A K of one or two steps is nearly all start and store: from a little more than one tile per CU on, tiles that keep one stage and run two
// to a CU beat those with a ring, whose workgroup does one after the other: 16384 x 4096 x 64 69.7 -> 54.5 us, 4096 x 2560 x 64 (320
// tiles) 21.8 -> 12.5, 16384 x 8192 x 128 131 -> 115, 2400 x 4000 x 128 (304) 14.3 -> 14.1, Q K^T of 4 x 1501 x 64 (288) 66.6 -> 58.7 for the
// whole scheme.  Below that they lose (2048 x 2048 x 128, 128 tiles: 8.1 and 10.8; 2000 x 3400 x 64, 224: 9.7 and 10.4; 2300 x 3500 x 128, 252: 14.0
// and 22.2; 8 x 1000 x 64, 256: 40.8 and 41.2), as with four steps (16384 x 2048 x 256 37.5 and 38.5).  In between it goes either way (2300 x 3800 x 64,
// 270 tiles: 21.5 and 12.8; 2300 x 4000 x 128, 288: 14.2 and 14.1; 4352 x 1900 x 64, 272: 30.8 and 21.9), so each line stands below
// the smallest count at which nothing measured lost.  Tiles are counted above the diagonal too, which a causal Q K^T does not launch: of 288 to 400 it launches
// 168 to 290, and still gains (the whole scheme, 3 x 3 x 1024 x 128, 180 launched: 39.1 -> 37.6 us, 4 x 9 x 512 x 64, 216: 42.3 -> 34.4, 1 x 2 x 2560 x 64, 220:
// 59.1 -> 56.3) or loses nothing (4 x 1501 x 64, 168: 52.1 and 52.9).
GPlan gemm_plan(long long m, long long n, long long k, int batch, bool inject, bool may_split) {
  if (inject) return {TILE_QUARTER, 1};
  static constexpr struct { int tile, max_n; double fixed, step, load; } COST[] = {
      {TILE_WIDE, 0, 9.0, 1.18, 0.42}, {TILE_HALF, 0, 5.5, 0.66, 0.45}, {TILE_QUARTER, 0, 3.0, 0.42, 0.7}, {TILE_STRIP, 0, 1.5, 0.37, 0.4},
      {TILE_NARROW, 128, 5.0, 0.48, 0.4}, {TILE_NARROW2, 128, 2.0, 0.31, 1.5}, {TILE_SLIM, 64, 5.0, 0.55, 0.8}, {TILE_SLIM2, 64, 2.0, 0.32, 2.0}};
  constexpr double CUS = 256.0, LAUNCH = 4.5, MEMORY = 5e6;           // bytes per microsecond
  const long long steps = (k + 63) / 64, tn = (n + GBN - 1) / GBN;
  const int max_n = n <= 64 ? 64 : n <= 128 ? 128 : 0;
  if (max_n == 0 && steps <= 2 && (m + TILES[TILE_LOW].bm - 1) / TILES[TILE_LOW].bm * tn * batch >= (batch > 1 ? 288 : 300)) return {TILE_LOW, 1};
  GPlan best{TILE_WIDE, 1};
  double best_us = 0.0;
  for (const auto& c : COST) {
    if (c.max_n != max_n && !(max_n && c.tile == TILE_STRIP)) continue;
    for (int parts = 1; parts <= 16 && (parts == 1 || (may_split && c.max_n == 0 && 2 * parts <= steps)); parts *= 2) {
      const GPlan plan{c.tile, parts};
      const double groups = (double)((m + TILES[c.tile].bm - 1) / TILES[c.tile].bm * tn) * batch * parts, per_cu = TILES[c.tile].per_cu;
      const double rounds = std::ceil(groups / (per_cu * CUS)), busy = std::min(per_cu, groups / CUS);
      double us = LAUNCH + rounds * (c.fixed + (double)((steps + parts - 1) / parts) * c.step * (1.0 + c.load * busy));
      if (parts > 1) us += LAUNCH + 2.0 * (double)gemm_workspace(m, n, plan) / MEMORY;
      if (best_us == 0.0 || us < best_us) { best = plan; best_us = us; }
    }
  }
  return best;
}

hipError_t gemm_launch(GArgs a, bool ft, bool inject, bool bf16, GPlan plan, hipStream_t st, int batch) {
  const TileInfo& ti = TILES[plan.tile];
  a.Tm = (a.M + ti.bm - 1) / ti.bm;
  a.Tn = (a.N + GBN - 1) / GBN;
  a.parts = plan.parts;
  a.ws_tokens = ws_tokens_of(a.M, plan);
  a.tiles = a.head_group = 0;
  dim3 grid(a.Tm * a.Tn, batch, plan.parts);
  if (a.skip_upper || a.k_lower) {       // (never split)
    a.tiles = a.skip_upper ? lower_tiles(a.Tm, ti.bm) : a.Tm;
    a.head_group = ftattn::head_group_of(32 * ti.per_cu, batch, a.Tm);
    grid = dim3(a.tiles * batch);
  }
  hipLaunchKernelGGL(tile_kernel(plan.tile, ft, inject, bf16), grid, dim3(ti.threads), ti.lds[ft], st, a);
  hipError_t he = hipGetLastError();
  if (he != hipSuccess || plan.parts <= 1) return he;
  hipLaunchKernelGGL((bf16 ? finish_kernel_bf16 : finish_kernel_f16)(ft), dim3((a.M + TileFinish::BM - 1) / TileFinish::BM * a.Tn),
                     dim3(TileFinish::NW * 64), ft ? TileFinish::lds<true>() : TileFinish::lds<false>(), st, a);
  return hipGetLastError();
}

GStats gemm_stats(const GSlot* slots, int n_slots) {
  GStats s{0, 0.f};
  for (int i = 0; i < n_slots; ++i) { s.events += slots[i].n; s.stat = std::max(s.stat, slots[i].stat); }
  return s;
}

hipError_t gemm_fetch_events(const GSlot* slots, int n_slots, const ftgemm_event* ring, uint32_t ring_n, int max_events,
                             std::vector<ftgemm_event>& out) {
  const GStats st = gemm_stats(slots, n_slots);
  if (!st.events) return hipSuccess;
  // end of this call's entries: the runs of a call are contiguous as a whole, counted without wrapping
  bool any = false;
  uint32_t end = 0;
  for (int i = 0; i < n_slots; ++i)
    if (slots[i].n) {
      const uint32_t e = slots[i].first + (uint32_t)slots[i].n;
      if (!any || (int32_t)(e - end) > 0) end = e;
      any = true;
    }
  // the last `keep` entries, in one piece or, where the ring wraps, two
  const uint32_t keep = (uint32_t)std::min<long long>(std::min<long long>(st.events, max_events), ring_n);
  const uint32_t first = (end - keep) & (ring_n - 1), run = std::min(keep, ring_n - first);
  const size_t at = out.size();
  out.resize(at + keep);
  hipError_t he = hipMemcpy(out.data() + at, ring + first, sizeof(ftgemm_event) * run, hipMemcpyDeviceToHost);
  if (he == hipSuccess && run < keep) he = hipMemcpy(out.data() + at + run, ring, sizeof(ftgemm_event) * (keep - run), hipMemcpyDeviceToHost);
  return he;
}

}  // namespace ftgemm

// For the tests, and no part of the interface: the tile shape (TileId) and the number of shares of K that a call without a
// fault list runs with.  m, n: tokens and features, exchanged by the caller where the checksums fold tokens.
extern "C" void ftgemm_plan_of(int64_t m, int64_t n, int64_t k, int32_t batch, int32_t out[2]) {
  const GPlan plan = gemm_plan(m, n, k, batch, false, batch == 1);
  out[0] = plan.tile; out[1] = plan.parts;
}

extern "C" int ftgemm_create(const ftgemm_config* cfg, ftgemm_ctx** out) {
  if (!cfg || !out) return gfail(nullptr, FTGEMM_EINVAL, "null argument");
  *out = nullptr;
  if (cfg->struct_size != sizeof(ftgemm_config)) return gfail(nullptr, FTGEMM_EINVAL, "struct_size mismatch");
  if (cfg->m < 1 || cfg->n < 1) return gfail(nullptr, FTGEMM_EINVAL, "m and n must be >= 1");
  if (cfg->k < 8 || cfg->k % 8 != 0) return gfail(nullptr, FTGEMM_EUNSUPPORTED, "k must be a positive multiple of 8 (rows of 16-byte chunks)");
  if (cfg->in_dtype != FTGEMM_F16 && cfg->in_dtype != FTGEMM_BF16) return gfail(nullptr, FTGEMM_EINVAL, "in_dtype must be F16 or BF16");
  if (cfg->out_dtype != FTGEMM_F32 && cfg->out_dtype != cfg->in_dtype) return gfail(nullptr, FTGEMM_EINVAL, "out_dtype must be F32 or the input type");
  if (cfg->ft_mode < 0 || cfg->ft_mode > 2) return gfail(nullptr, FTGEMM_EINVAL, "ft_mode out of range");
  if (cfg->stride != 0 && cfg->stride != 8) return gfail(nullptr, FTGEMM_EUNSUPPORTED, "stride must be 8");
  if (cfg->block_n != 0 && cfg->block_n != GBN) return gfail(nullptr, FTGEMM_EUNSUPPORTED, "block_n must be 256");
  if (cfg->fold_tokens != 0 && cfg->fold_tokens != 1) return gfail(nullptr, FTGEMM_EINVAL, "fold_tokens must be 0 or 1");
  // with fold_tokens the kernel runs the transposed problem: its tokens are the weight rows, its features the token rows
  const long long km = cfg->fold_tokens ? cfg->n : cfg->m, kn = cfg->fold_tokens ? cfg->m : cfg->n;
  const long long tn = (kn + GBN - 1) / GBN;
  if ((km + TILES[TILE_STRIP].bm - 1) / TILES[TILE_STRIP].bm * tn > 0x7FFFFFFFll) return gfail(nullptr, FTGEMM_EUNSUPPORTED, "too many output tiles");
  // the per-lane load offsets are 32-bit: 256 rows of k fp16 values must fit
  if ((long long)cfg->k * 2 * 256 > 0x7FFFFFFFll) return gfail(nullptr, FTGEMM_EUNSUPPORTED, "k too large");

  ftgemm_ctx* c = new (std::nothrow) ftgemm_ctx();
  if (!c) return gfail(nullptr, FTGEMM_ENOMEM, "out of host memory");
  c->cfg = *cfg;
  ftgemm_config& e = c->cfg;
  e.stride = 8;
  e.block_n = GBN;
  if (!(e.tau_rel > 0.f)) e.tau_rel = 1.0f / 32768.0f;
  if (!(e.tau_abs >= 0.f)) e.tau_abs = 0.f;
  if (e.max_events <= 0) e.max_events = 65536;
  c->Tn = (int)tn;
  c->fault_cap = 1 << 16;

  hipError_t he = hipSetDevice(e.device);
  if (he != hipSuccess) { int rc = gfail(nullptr, FTGEMM_EHIP, std::string("hipSetDevice: ") + hipGetErrorString(he)); delete c; return rc; }
#define GCREATE_TRY(expr)                                                                                 \
  do {                                                                                                    \
    hipError_t e_ = (expr);                                                                               \
    if (e_ != hipSuccess) {                                                                               \
      int rc_ = gfail(nullptr, e_ == hipErrorOutOfMemory ? FTGEMM_ENOMEM : FTGEMM_EHIP,                   \
                      std::string(#expr) + ": " + hipGetErrorString(e_));                                 \
      grelease(c);                                                                                        \
      return rc_;                                                                                         \
    }                                                                                                     \
  } while (0)
  c->ring_n = ring_size(e.max_events);
  const GPlan plan = gemm_plan(km, kn, e.k, 1, false, true);
  c->n_slots = std::max(gemm_slots(km, kn, plan), gemm_slots(km, kn, gemm_plan(km, kn, e.k, 1, true, false)));
  // one allocation for all of the device scratch: each hipMalloc costs tens of microseconds.  Only the
  // cursor and the number of slots have to start from a value: checksum rows are written before they are read.
  struct { void** at; size_t bytes, from; } parts[] = {
      {(void**)&c->wc, (size_t)c->Tn * GCK * e.k * 2, 0}, {(void**)&c->d_faults, sizeof(GFault) * c->fault_cap, 0},
      {(void**)&c->d_events, sizeof(ftgemm_event) * (size_t)c->ring_n, 0}, {(void**)&c->d_cursor, CURSOR_BYTES + sizeof(GSlot) * (size_t)(1 + c->n_slots), 0}, {(void**)&c->ws, gemm_workspace(km, kn, plan), 0}};
  size_t total = 0;
  for (auto& p : parts) { p.from = total; total += (p.bytes + 255) & ~(size_t)255; }
  GCREATE_TRY(hipMalloc(&c->scratch, total));
  for (auto& p : parts) *p.at = static_cast<char*>(c->scratch) + p.from;
  c->d_n_slots = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(c->d_cursor) + CURSOR_BYTES);
  c->d_slots = reinterpret_cast<GSlot*>(c->d_n_slots) + 1;
  GCREATE_TRY(hipHostMalloc((void**)&c->h_faults, sizeof(GFault) * c->fault_cap + sizeof(GSlot) * (size_t)(1 + c->n_slots), hipHostMallocDefault));
  c->h_slots = reinterpret_cast<GSlot*>(c->h_faults + c->fault_cap);
  GCREATE_TRY(hipMemset(c->d_cursor, 0, CURSOR_BYTES + 16));        // (whole 16-byte words: a remainder is a launch of its own)
  GCREATE_TRY(gemm_allow_lds(plan, e.ft_mode != FTGEMM_FT_OFF, e.in_dtype == FTGEMM_BF16));
  GCREATE_TRY(hipDeviceSynchronize());
#undef GCREATE_TRY
  *out = c;
  return FTGEMM_OK;
}

extern "C" int ftgemm_get_config(const ftgemm_ctx* ctx, ftgemm_config* effective) {
  if (!ctx || !effective) return FTGEMM_EINVAL;
  *effective = ctx->cfg;
  return FTGEMM_OK;
}

extern "C" int ftgemm_encode_weights(ftgemm_ctx* c, const void* w, void* hip_stream) {
  if (!c) return FTGEMM_EINVAL;
  if (!w || ((uintptr_t)w & 15)) return gfail(c, FTGEMM_EINVAL, "w must be a 16-byte aligned device pointer");
  const ftgemm_config& e = c->cfg;
  if (e.fold_tokens) return FTGEMM_OK;      // the checksums are those of x, taken inside every forward
  GHIP_TRY(c, hipSetDevice(e.device));
  hipStream_t st = (hipStream_t)hip_stream;
  GHIP_TRY(c, gemm_launch_encode_w(reinterpret_cast<const uint16_t*>(w), c->wc, e.n, e.k, e.in_dtype == FTGEMM_BF16, st));
  c->encoded_w = w;
  return FTGEMM_OK;
}

extern "C" int ftgemm_forward(ftgemm_ctx* c, const void* x, const void* w, void* y,
                              const ftgemm_fault* faults, int32_t n_faults, void* hip_stream) {
  if (!c) return FTGEMM_EINVAL;
  if (!x || !w || !y) return gfail(c, FTGEMM_EINVAL, "null matrix pointer");
  if (((uintptr_t)x | (uintptr_t)w | (uintptr_t)y) & 15) return gfail(c, FTGEMM_EINVAL, "matrix pointers must be 16-byte aligned");
  if (n_faults < 0 || (n_faults > 0 && !faults)) return gfail(c, FTGEMM_EINVAL, "bad fault list");
  if (n_faults > c->fault_cap) return gfail(c, FTGEMM_EINVAL, "too many faults (limit 65536)");
  const ftgemm_config& e = c->cfg;
  const bool ft = e.ft_mode != FTGEMM_FT_OFF;
  const bool tr = e.fold_tokens != 0;
  if (ft && !tr && c->encoded_w != w) return gfail(c, FTGEMM_ESTATE, "ftgemm_encode_weights has not been called for this weight matrix");
  hipStream_t st = (hipStream_t)hip_stream;
  GHIP_TRY(c, hipSetDevice(e.device));
  for (int i = 0; i < n_faults; ++i) {
    const ftgemm_fault& f = faults[i];
    if (f.row < 0 || f.row >= e.m || f.col < 0 || f.col >= e.n || f.bit < 0 || f.bit > 31) {
      char msg[128];
      snprintf(msg, sizeof msg, "fault %d (row=%d col=%d bit=%d) is outside the matrix", i, f.row, f.col, f.bit);
      return gfail(c, FTGEMM_EINVAL, msg);
    }
    c->h_faults[i] = tr ? GFault{f.col, f.row, f.bit} : GFault{f.row, f.col, f.bit};
  }
  if (n_faults > 0) {
    GHIP_TRY(c, hipMemcpyAsync(c->d_faults, c->h_faults, sizeof(GFault) * n_faults, hipMemcpyHostToDevice, st));
    GHIP_TRY(c, hipStreamSynchronize(st));   // the staging buffer may be rewritten by the next call
  }
  const bool bf = e.in_dtype == FTGEMM_BF16;
  // fold_tokens: tensor checksums of this call's token rows (eq. (13), (14) on x)
  if (ft && tr) GHIP_TRY(c, gemm_launch_encode_w(reinterpret_cast<const uint16_t*>(x), c->wc, e.m, e.k, bf, st));
  GArgs a;
  a.x = reinterpret_cast<const uint16_t*>(tr ? w : x);
  a.w = reinterpret_cast<const uint16_t*>(tr ? x : w);
  a.wc = c->wc;
  a.y = y; a.out_dtype = e.out_dtype;
  a.M = tr ? e.n : e.m; a.N = tr ? e.m : e.n; a.K = e.k; a.Tm = a.Tn = 0;
  a.transposed = tr ? 1 : 0;
  a.bs_x = a.bs_w = a.bs_wc = a.bs_y_bytes = a.bs_events = a.bs_slots = 0;
  a.skip_upper = 0; a.k_lower = 0;
  a.tau_rel = e.tau_rel; a.tau_abs = e.tau_abs;
  a.correct = e.ft_mode == FTGEMM_FT_CORRECT ? 1 : 0;
  a.faults = c->d_faults; a.n_faults = n_faults;
  a.events = c->d_events; a.cursor = c->d_cursor; a.ring_mask = c->ring_n - 1;
  a.slots = c->d_slots; a.n_slots = c->d_n_slots;
  a.ws = c->ws;
  const GPlan plan = gemm_plan(a.M, a.N, a.K, 1, n_faults > 0, true);
  if (c->timing) GHIP_TRY(c, hipEventRecord(c->ev[0], st));
  GHIP_TRY(c, gemm_launch(a, ft, n_faults > 0, bf, plan, st));
  if (c->timing) GHIP_TRY(c, hipEventRecord(c->ev[1], st));
  c->last_slots = gemm_slots(a.M, a.N, plan);
  c->last_stream = st;
  c->ran = true;
  return FTGEMM_OK;
}

extern "C" int ftgemm_report(ftgemm_ctx* c, ftgemm_report_view* out) {
  if (!c || !out) return FTGEMM_EINVAL;
  if (!c->ran) return gfail(c, FTGEMM_EINVAL, "no forward call to report on");
  const ftgemm_config& e = c->cfg;
  GHIP_TRY(c, hipSetDevice(e.device));
  // (into pinned memory and behind one wait: a call on the default stream with its report takes 8 us less than with a wait and a
  // blocking copy into other memory)
  if (c->last_stream) GHIP_TRY(c, hipStreamSynchronize(c->last_stream));
  int32_t n = c->last_slots;
  for (int have = -1; have < n; ) {         // (a second copy only after a replay that wrote more)
    have = n;
    GHIP_TRY(c, hipMemcpyAsync(c->h_slots, c->d_n_slots, sizeof(GSlot) * (size_t)(1 + n), hipMemcpyDeviceToHost, nullptr));
    GHIP_TRY(c, hipStreamSynchronize(nullptr));
    std::memcpy(&n, c->h_slots, sizeof n);
    if (n > c->n_slots) return gfail(c, FTGEMM_EHIP, "damaged report");
  }
  const GSlot* slots = c->h_slots + 1;
  const GStats stats = gemm_stats(slots, n);
  c->events.clear();
  GHIP_TRY(c, gemm_fetch_events(slots, n, c->d_events, c->ring_n, e.max_events, c->events));
  std::sort(c->events.begin(), c->events.end(), [](const ftgemm_event& p, const ftgemm_event& q) {
    if (p.row != q.row) return p.row < q.row;
    return p.col < q.col;
  });
  out->n_events = (int32_t)c->events.size();
  out->n_events_dropped = (int32_t)(stats.events - (long long)c->events.size());
  out->events = c->events.data();
  out->residual_max = stats.stat;
  return FTGEMM_OK;
}

extern "C" int ftgemm_set_timing(ftgemm_ctx* c, int32_t enabled) {
  if (!c) return FTGEMM_EINVAL;
  GHIP_TRY(c, hipSetDevice(c->cfg.device));
  if (enabled)
    for (hipEvent_t& e : c->ev)
      if (!e) GHIP_TRY(c, hipEventCreate(&e));
  c->timing = enabled != 0;
  return FTGEMM_OK;
}

extern "C" int ftgemm_get_timing(ftgemm_ctx* c, float* ms) {
  if (!c || !ms) return FTGEMM_EINVAL;
  if (!c->timing || !c->ran) return gfail(c, FTGEMM_EINVAL, "timing is not enabled or no forward has run");
  GHIP_TRY(c, hipSetDevice(c->cfg.device));
  GHIP_TRY(c, hipEventSynchronize(c->ev[1]));
  GHIP_TRY(c, hipEventElapsedTime(ms, c->ev[0], c->ev[1]));
  return FTGEMM_OK;
}

extern "C" int ftgemm_destroy(ftgemm_ctx* c) {
  if (!c) return FTGEMM_EINVAL;
  (void)hipSetDevice(c->cfg.device);
  (void)hipDeviceSynchronize();
  grelease(c);
  return FTGEMM_OK;
}

extern "C" const char* ftgemm_last_error(const ftgemm_ctx* c) {
  return c ? c->err.c_str() : g_gemm_create_err.c_str();
}
