// Host side of the fault-tolerant fused attention library: the C ABI of include/ftattn.h.
// Validation, fault bucketing, launches and the report are here; every arithmetic step of
// the attention pass runs in the kernels of ftattn_device.h.
#include "ftattn_main.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace ftattn;

// Shape-derived sizes of one configuration: tiles per head and the element counts of the encoded
// key / value tiles.
struct Geometry {
  int BH = 0, Ti = 0, Tj = 0, BM = 0;
  size_t n_kc = 0, n_vt = 0;
  size_t beyond = 0;      // bytes behind the encoded tiles that may be read (TILES_BEYOND)
  // Row tiles split by their keys (see share_of): those launched from number first_split on, in shares of up to `piece`
  // key tiles, `shares` in all; n_ws floats hold their state.
  int first_split = 0, piece = 1, shares = 0;
  size_t n_ws = 0;
};

// Device buffers one pass works on (owned by a context, or carved out of the static scratch array).
struct Buffers {
  _Float16* kc = nullptr;
  _Float16* vt = nullptr;
  const DevFault* faults = nullptr;
  const int32_t* fault_off = nullptr;
  ftattn_event* events = nullptr;
  int32_t* ev_count = nullptr;
  unsigned long long* recheck = nullptr;
  uint32_t* resmax = nullptr;
  float* ws = nullptr;                // state of split row tiles (null: no row tile is split)
  unsigned char* work = nullptr;      // STAT_WORK
  uint32_t* ended = nullptr;          // where workgroups of calls in one launch count that they have ended
  uint32_t* range = nullptr;          // the word this call sets
  uint32_t* range_next = nullptr;     // the word the next call sets: cleared by this call
};

// Offsets in the block a report reads: event count, recheck count, two range words used in turn by
// consecutive calls, residual maxima.  One block, so that a report is one copy behind one wait:
// a pass over 2 x 3 x 333 x 128 with its report takes 53 us, and took 98 with a blocking copy for each.
// STAT_WORK: what calls in one launch count in, zero between them: event count, range word, recheck count, workgroups that have ended.
// Nothing clears these first, so they must come back to zero by themselves also where calls overlapped (which spoils the reports of
// those calls): the last word is counted by calls of one number of heads only, each of which adds that number and takes it off again,
// and the workgroup that ends last of all is the last one of its own call and finds everything that was counted.
constexpr size_t STAT_EVENTS = 0, STAT_RECHECK = 8, STAT_RANGE = 16, STAT_WORK = 64, STAT_RESMAX = 256;

struct ftattn_ctx {
  ftattn_config cfg;          // effective configuration
  Geometry geo;
  // device scratch
  _Float16* kc = nullptr;
  _Float16* vt = nullptr;
  float* ws = nullptr;
  void* vt_alloc = nullptr;      // the allocations of vt and ws where they have one of their own
  void* ws_alloc = nullptr;
  DevFault* d_faults = nullptr;
  int32_t* d_fault_off = nullptr;
  ftattn_event* d_events = nullptr;
  unsigned char* d_stat = nullptr;    // counters and residual maxima of the report, one block (STAT_*)
  unsigned calls = 0;
  int fault_cap = 0;
  // pinned host staging
  DevFault* h_faults = nullptr;
  unsigned char* h_stat = nullptr;    // where a report finds a copy of d_stat
  int32_t* h_fault_off = nullptr;     // behind it, in the same block
  size_t stat_bytes = 0;
  // report storage
  std::vector<ftattn_event> events;
  std::vector<uint8_t> tile_flags, rowtile_flags;
  std::vector<float> resmax;
  hipStream_t last_stream = nullptr;
  bool ran = false;
  bool timing = false;
  bool masked_faults = false;
  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};   // before encode, before fused kernel, after
  std::string err;
};

static thread_local std::string g_create_err;

static int fail(ftattn_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg; else g_create_err = msg;
  return code;
}

#define HIP_TRY(ctx, expr)                                                                      \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return fail(ctx, e_ == hipErrorOutOfMemory ? FTATTN_ENOMEM : FTATTN_EHIP,                 \
                  std::string(#expr) + ": " + hipGetErrorString(e_));                           \
  } while (0)

static void release(ftattn_ctx* c) {
  if (!c) return;
  (void)hipFree(c->kc); (void)hipFree(c->vt_alloc); (void)hipFree(c->ws_alloc); (void)hipFree(c->d_faults);
  (void)hipFree(c->d_fault_off); (void)hipFree(c->d_events); (void)hipFree(c->d_stat);
  if (c->h_faults) (void)hipHostFree(c->h_faults);
  if (c->h_stat) (void)hipHostFree(c->h_stat);
  for (hipEvent_t e : c->ev) if (e) (void)hipEventDestroy(e);
  delete c;
}

typedef kernel_fn main_fn;

template <int D, bool INJ>
static main_fn pick(bool ft, bool causal) {
  if (ft) return causal ? ftattn_main<D, true, true, INJ> : ftattn_main<D, true, false, INJ>;
  return causal ? ftattn_main<D, false, true, INJ> : ftattn_main<D, false, false, INJ>;
}

// inject: the variant that carries the fault-injection code; calls without a fault list run the
// variant that has none of it
// the ablation modes are instantiated in translation units of their own (ftattn_perstep.hip,
// ftattn_elementwide.hip), so that all of them compile side by side
namespace ftattn {
void (*select_perstep(int D, bool causal, bool inject, int mode))(const KArgs);
void (*select_elementwide(int D, bool causal, bool inject))(const KArgs);
void (*select_lazy(int D, bool ft, bool causal, bool inject))(const KArgs);
kernel_fn select_split(int D, bool ft, bool causal);
kernel_fn select_self(int D, bool ft, bool causal);
kernel_fn select_finish(int D, bool ft, bool causal);
}

static main_fn select_kernel(int D, bool ft, bool causal, bool inject) {
  if (D == 128) return inject ? pick<128, true>(ft, causal) : pick<128, false>(ft, causal);
  if (D == 64) return inject ? pick<64, true>(ft, causal) : pick<64, false>(ft, causal);
  return nullptr;
}

static size_t lds_bytes(int D, bool ft) {
  if (D == 128) return ft ? Unit<128, true>::LDS_TOTAL : Unit<128, false>::LDS_TOTAL;
  return ft ? Unit<64, true>::LDS_TOTAL : Unit<64, false>::LDS_TOTAL;
}

// Which row tiles are split by their keys, and into shares of how many: the plan with the least expected time.
// Microseconds, from timings of both head sizes with 1..512 row tiles of 2..256 key tiles: a workgroup costs `fixed`
// and `tile` per key tile, one at a time per CU (two that share a CU at head_dim 64 take about twice as long each); a
// split adds the launch that puts the shares together, and their state passes through memory twice.  Measured, unsplit and
// as planned here: 1 x 1 x 16384 x 128 causal 496 and 128 us, 2 x 3 x 5001 x 128 178 and 134, 1 x 5 x 3001 x 64 causal
// 74 and 45, 1 x 20 x 2048 x 128 causal 92 and 74.  Row tiles of equal length that fill the CUs a whole number of
// times and a little more: only those left over are split (3 x 16 x 1531 x 128, 288 row tiles: 154 and 131 us; all
// split in two 191).  Beyond twice the CUs (causal: light row tiles fill up the last round; else four times) a split
// gains nothing, and neither do short rows, where starting and finishing a workgroup is most of it (6 key tiles, 2 x 3 x
// 333 x 128: 28.8 and 27.9 us; 8, 1 x 2 x 512 x 64: 22.1 and 20.8; 11, 1 x 7 x 700 x 128: 41 and 37; 16, 1 x 1 x 1000 x 128:
// 48 and 32).  A call with a fault list is never split: faults name values of Algorithm 1's one pass over the keys.
static void plan_split(const ftattn_config& e, Geometry& g) {
  constexpr long long CUS = 256;
  const long long tiles = (long long)g.BH * g.Ti;
  g.first_split = (int)tiles;
  if (e.per_step != 0 || e.stride != 8 || e.rescale_margin > 0.f || g.Tj < 12 || tiles >= (e.causal ? 2 : 4) * CUS) return;
  // (the same plan for every ft_mode, so that the unprotected variant computes the same numbers; its key tiles are about
  // 0.7 times as long)
  const bool d128 = e.head_dim == 128;
  const double fixed = d128 ? 9.0 : 4.5, tile = d128 ? 2.6 : 1.2;
  constexpr double FINISH = 5.0, PER_PART = 1.0, MEMORY = 4e6;       // bytes per microsecond
  constexpr size_t WS_BYTES = (size_t)96 << 20;
  const size_t state = (size_t)nwave_of(e.head_dim) * 64 * sizeof(float) * (d128 ? part_values<128, true>() : part_values<64, true>());
  const int per_row = g.BM / BN;
  const double keys = g.BH * (e.causal ? 0.5 * per_row * g.Ti * (g.Ti + 1.0) - (per_row * g.Ti - g.Tj) : (double)g.Ti * g.Tj);
  auto count = [&](long long whole, int piece) {      // shares of all row tiles but the first `whole`
    long long n = 0;
    for (int p = 0; p * piece < g.Tj; ++p) n += row_tiles_with(p, e.causal != 0, (int)(tiles - whole), g.BH, g.Ti, piece, per_row);
    return n;
  };
  auto cost = [&](long long whole, int piece, long long n) {
    const int parts = (g.Tj + piece - 1) / piece;
    const double longest = piece * tile + fixed;
    double us = (double)(whole / CUS) * (g.Tj * tile + fixed);
    if (n <= CUS || !e.causal) us += std::ceil((double)n / CUS) * longest;
    else us += std::max(longest, (keys * tile + n * fixed) / CUS + 0.5 * longest);
    if (parts > 1) us += FINISH + PER_PART * parts + 2.0 * n * (double)state / MEMORY;
    return us;
  };
  double best = cost(0, g.Tj, tiles);
  for (int some = 0; some < 2; ++some) {
    const long long whole = some ? tiles / CUS * CUS : 0;
    if (some ? e.causal || whole == 0 || whole == tiles : tiles >= 2 * CUS) continue;
    for (int parts = 2; parts <= MAX_PARTS && parts <= g.Tj; ++parts) {
      const int piece = (g.Tj + parts - 1) / parts;
      const long long n = count(whole, piece);
      if (n * state > WS_BYTES) break;
      const double us = cost(whole, piece, n);
      if (us < 0.97 * best) {
        best = us;
        g.first_split = (int)whole; g.piece = piece; g.shares = (int)n; g.n_ws = n * state / sizeof(float);
      }
    }
  }
}

constexpr size_t tiles_beyond(int D) { return (size_t)TILES_BEYOND * (BN + CKR) * D * 2; }      // (value tiles are no larger)

// Checks cfg and resolves its defaults into e (tile sizes, thresholds, scale) and g.  Touches no
// device.  On failure returns the error code and points `why` at a constant message.
static int resolve_config(const ftattn_config* cfg, ftattn_config& e, Geometry& g, const char*& why) {
  why = "";
  if (cfg->struct_size != sizeof(ftattn_config)) { why = "struct_size mismatch"; return FTATTN_EINVAL; }
  if (cfg->batch < 1 || cfg->heads < 1 || cfg->seq < 1) { why = "batch, heads, seq must be >= 1"; return FTATTN_EINVAL; }
  if ((long long)cfg->batch * cfg->heads > 65535) { why = "batch*heads > 65535"; return FTATTN_EUNSUPPORTED; }
  if (cfg->head_dim != 64 && cfg->head_dim != 128) { why = "head_dim must be 64 or 128"; return FTATTN_EUNSUPPORTED; }
  if (cfg->in_dtype != FTATTN_F16 && cfg->in_dtype != FTATTN_BF16) { why = "in_dtype must be F16 or BF16"; return FTATTN_EINVAL; }
  if (cfg->out_dtype != FTATTN_F32 && cfg->out_dtype != cfg->in_dtype) { why = "out_dtype must be F32 or the input type"; return FTATTN_EINVAL; }
  if (cfg->ft_mode < 0 || cfg->ft_mode > 2) { why = "ft_mode out of range"; return FTATTN_EINVAL; }
  if (cfg->stride != 0 && cfg->stride != 8 && cfg->stride != 1) { why = "stride must be 8 (or 1: the traditional checksum)"; return FTATTN_EUNSUPPORTED; }
  if (cfg->block_n != 0 && cfg->block_n != BN) { why = "block_n must be 64"; return FTATTN_EUNSUPPORTED; }
  if (cfg->block_m != 0 && cfg->block_m != bm_of(cfg->head_dim)) {
    why = "block_m must be 0 or the library's row tile (256 for head_dim 128, 128 for head_dim 64)";
    return FTATTN_EUNSUPPORTED;
  }
  if (cfg->causal != 0 && cfg->causal != 1) { why = "causal must be 0 or 1"; return FTATTN_EINVAL; }
  if (cfg->rowsum_fold != 0 && cfg->rowsum_fold != 1) { why = "rowsum_fold must be 0 or 1"; return FTATTN_EINVAL; }
  if (cfg->per_step < 0 || cfg->per_step > 2) { why = "per_step must be 0, 1 or 2"; return FTATTN_EINVAL; }
  if (cfg->per_step != 0 && (cfg->ft_mode != FTATTN_FT_CORRECT || cfg->rowsum_fold != 0)) {
    why = "per_step needs ft_mode FTATTN_FT_CORRECT and rowsum_fold 0";
    return FTATTN_EINVAL;
  }
  if (cfg->stride == 1 && (cfg->ft_mode == FTATTN_FT_OFF || cfg->rowsum_fold != 0 || cfg->per_step != 0)) {
    why = "stride 1 needs a protected ft_mode, rowsum_fold 0 and per_step 0";
    return FTATTN_EINVAL;
  }
  if (cfg->rescale_margin > 0.f && (cfg->per_step != 0 || cfg->stride == 1 || cfg->rowsum_fold != 0)) {
    why = "rescale_margin needs per_step 0, stride 8 and rowsum_fold 0";
    return FTATTN_EINVAL;
  }
  if (cfg->rescale_margin > 8.f) { why = "rescale_margin must be at most 8 (the exponentials are held in fp16)"; return FTATTN_EINVAL; }
  e = *cfg;
  if (!(e.rescale_margin > 0.f)) e.rescale_margin = 0.f;
  e.stride = cfg->stride == 1 ? 1 : 8;
  e.block_n = BN;
  if (!(e.softmax_scale > 0.f)) e.softmax_scale = 1.0f / std::sqrt((float)e.head_dim);
  if (!(e.eps1 > 0.f)) e.eps1 = 0.03f;
  if (!(e.tau_o > 0.f)) e.tau_o = 0.75f / 512.0f;
  if (!(e.delta_l > 0.f)) e.delta_l = 1.0f / 1024.0f;
  if (e.max_events <= 0) e.max_events = 65536;
  e.block_m = bm_of(e.head_dim);
  g.BH = e.batch * e.heads;
  g.Tj = (e.seq + BN - 1) / BN;
  g.BM = e.block_m;
  g.Ti = (e.seq + g.BM - 1) / g.BM;
  g.n_kc = (size_t)g.BH * g.Tj * (BN + CKR) * e.head_dim;
  g.n_vt = (size_t)g.BH * g.Tj * (e.head_dim + CKR) * BN;
  g.beyond = tiles_beyond(e.head_dim);
  plan_split(e, g);
  return FTATTN_OK;
}

// Whether a call without a fault list is one launch.
static bool in_one_launch(const ftattn_config& e, const Geometry& g) {
  return self_encodes(e.head_dim, g.Ti, g.Tj) && e.per_step == 0 && e.stride == 8 && !(e.rescale_margin > 0.f);
}

// For the tests, and no part of the interface: how a call without a fault list is split.  out: number of the first row
// tile that is split (all row tiles: none is), key tiles of a share at most, shares, bytes of their state.
extern "C" int ftattn_split_of(const ftattn_config* cfg, int64_t out[4]) {
  ftattn_config e;
  Geometry g;
  const char* why;
  if (int rc = resolve_config(cfg, e, g, why)) return rc;
  out[0] = g.first_split; out[1] = g.piece; out[2] = g.shares; out[3] = (int64_t)(g.n_ws * sizeof(float));
  return FTATTN_OK;
}

// For the tests, and no part of the interface: 1 where a call without a fault list is one launch.
extern "C" int ftattn_in_one_launch(const ftattn_config* cfg) {
  ftattn_config e;
  Geometry g;
  const char* why;
  if (int rc = resolve_config(cfg, e, g, why)) return rc;
  return in_one_launch(e, g);
}

// Lets the kernels that a configuration runs, with a fault list or without one, use their dynamic LDS.  Needs the
// device current.  (Only those: a call to the runtime for each takes about 10 us of the 110 to 300 that creating a
// context takes.)
static hipError_t allow_lds(const ftattn_config& e, bool split, bool self, const char*& why) {
  const int D = e.head_dim;
  const bool ft = e.ft_mode != FTATTN_FT_OFF, causal = e.causal != 0, lazy = e.rescale_margin > 0.f;
  const int bytes = (int)lds_bytes(D, ft);
  why = "no kernel for this tile shape";
  for (int v = 0; v < 4; ++v) {
    const bool inject = v == 1;
    if (v == 2 ? !split : v == 3 ? !self : false) continue;
    main_fn f = v == 2 ? select_split(D, ft, causal)
                : v == 3 ? select_self(D, ft, causal)
                : e.per_step ? select_perstep(D, causal, inject, e.per_step)
                : e.stride == 1 ? select_elementwide(D, causal, inject)
                : lazy ? select_lazy(D, ft, causal, inject)
                       : select_kernel(D, ft, causal, inject);
    if (!f) return hipErrorInvalidValue;
    hipError_t he = hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (he != hipSuccess) { why = "hipFuncSetAttribute"; return he; }
  }
  return hipSuccess;
}

extern "C" int ftattn_create(const ftattn_config* cfg, ftattn_ctx** out) {
  if (!cfg || !out) return fail(nullptr, FTATTN_EINVAL, "null argument");
  *out = nullptr;
  ftattn_config e;
  Geometry g;
  const char* why;
  if (int rc = resolve_config(cfg, e, g, why)) return fail(nullptr, rc, why);

  ftattn_ctx* c = new (std::nothrow) ftattn_ctx();
  if (!c) return fail(nullptr, FTATTN_ENOMEM, "out of host memory");
  c->cfg = e;
  c->geo = g;

  hipError_t he = hipSetDevice(e.device);
  if (he != hipSuccess) { int rc = fail(nullptr, FTATTN_EHIP, std::string("hipSetDevice: ") + hipGetErrorString(he)); delete c; return rc; }

  c->fault_cap = 1 << 16;
  const size_t n_rt = (size_t)g.BH * g.Ti;
#define CREATE_TRY(expr)                                                                                  \
  do {                                                                                                    \
    hipError_t e_ = (expr);                                                                               \
    if (e_ != hipSuccess) {                                                                               \
      int rc_ = fail(nullptr, e_ == hipErrorOutOfMemory ? FTATTN_ENOMEM : FTATTN_EHIP,                    \
                     std::string(#expr) + ": " + hipGetErrorString(e_));                                  \
      release(c);                                                                                         \
      return rc_;                                                                                         \
    }                                                                                                     \
  } while (0)
  // The encoded tiles and the state of split row tiles share an allocation (each one, with its memset, costs about 30 us to
  // make and 15 to 20 to free) unless only that takes it beyond 64 MiB, where the runtime needs 35 us to make one and 270 to free it.
  constexpr size_t CHEAP = (size_t)64 << 20;
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  auto together = [](size_t x, size_t y) { return x + y <= CHEAP || x > CHEAP || y > CHEAP; };
  const size_t kc_bytes = up(g.n_kc * 2), vt_bytes = up(g.n_vt * 2), ws_bytes = g.n_ws * sizeof(float);
  const bool vt_joined = together(kc_bytes, vt_bytes + g.beyond);
  const size_t tiles_bytes = kc_bytes + (vt_joined ? vt_bytes : 0);
  const bool ws_joined = ws_bytes && together(tiles_bytes + g.beyond, ws_bytes);
  CREATE_TRY(hipMalloc((void**)&c->kc, tiles_bytes + g.beyond + (ws_joined ? ws_bytes : 0)));
  if (vt_joined) {
    c->vt = c->kc + kc_bytes / 2;
  } else {
    CREATE_TRY(hipMalloc(&c->vt_alloc, vt_bytes + g.beyond));
    c->vt = static_cast<_Float16*>(c->vt_alloc);
  }
  if (ws_joined) {
    c->ws = reinterpret_cast<float*>(reinterpret_cast<char*>(c->kc) + tiles_bytes + g.beyond);
  } else if (ws_bytes) {
    CREATE_TRY(hipMalloc(&c->ws_alloc, ws_bytes));
    c->ws = static_cast<float*>(c->ws_alloc);
  }
  CREATE_TRY(hipMalloc((void**)&c->d_faults, sizeof(DevFault) * c->fault_cap));
  CREATE_TRY(hipMalloc((void**)&c->d_fault_off, sizeof(int32_t) * (n_rt + 1)));
  CREATE_TRY(hipMalloc((void**)&c->d_events, sizeof(ftattn_event) * (size_t)e.max_events));
  c->stat_bytes = STAT_RESMAX + sizeof(uint32_t) * n_rt * 4;
  CREATE_TRY(hipMalloc((void**)&c->d_stat, c->stat_bytes));
  CREATE_TRY(hipMemset(c->d_stat, 0, c->stat_bytes));
  // (one pinned block for both: an allocation of its own for the copy of d_stat made this call 5 us longer)
  CREATE_TRY(hipHostMalloc((void**)&c->h_stat, c->stat_bytes + sizeof(int32_t) * (n_rt + 1), hipHostMallocDefault));
  c->h_fault_off = reinterpret_cast<int32_t*>(c->h_stat + c->stat_bytes);
  CREATE_TRY(hipHostMalloc((void**)&c->h_faults, sizeof(DevFault) * c->fault_cap, hipHostMallocDefault));
  // the checksum rows of the encoded tiles are never written when ft_mode is OFF; keep them defined
  CREATE_TRY(hipMemset(c->kc, 0, tiles_bytes));
  if (!vt_joined) CREATE_TRY(hipMemset(c->vt, 0, vt_bytes));
  {
    hipError_t le = allow_lds(e, g.n_ws != 0, in_one_launch(e, g), why);
    if (le != hipSuccess) {
      int rc = fail(nullptr, le == hipErrorInvalidValue ? FTATTN_EUNSUPPORTED : FTATTN_EHIP, std::string(why) + ": " + hipGetErrorString(le));
      release(c);
      return rc;
    }
  }
  CREATE_TRY(hipDeviceSynchronize());
#undef CREATE_TRY
  *out = c;
  return FTATTN_OK;
}

extern "C" int ftattn_get_config(const ftattn_ctx* ctx, ftattn_config* effective) {
  if (!ctx || !effective) return FTATTN_EINVAL;
  *effective = ctx->cfg;
  return FTATTN_OK;
}

// The launches of one pass on `st`: encode (Algorithm 1: "Encode tensor checksum"), once per key tile for all row tiles, which
// also clears the counters of the report; then the fused pass; then, where row tiles are split by their keys, what puts their shares
// together.  The fused pass alone where in_one_launch says so.
// Allocates nothing.  `timing`: three events recorded before, between and after the launches, or null.
static hipError_t launch_pass(const ftattn_config& e, const Geometry& g, const Buffers& b, const void* q, const void* k,
                              const void* v, void* o, bool inject, hipStream_t st, hipEvent_t* timing) {
  const int D = e.head_dim, N = e.seq;
  const bool ft = e.ft_mode != FTATTN_FT_OFF;
  const int n_resmax = g.BH * g.Ti * 4;
  hipError_t he;
  // (a timed call keeps the launch of the encode, which has a time of its own)
  const bool self = !inject && !timing && in_one_launch(e, g);
  if (timing && (he = hipEventRecord(timing[0], st)) != hipSuccess) return he;
  dim3 eg(g.Tj, g.BH, 2);
  const int bf = e.in_dtype == FTATTN_BF16 ? 1 : 0;
  const int kchk = ft ? 1 : 0, vchk = ft ? 1 + e.rowsum_fold : 0;
  if (self) {}
  else if (D == 128)
    ftattn_prepare<128><<<eg, 256, 0, st>>>(k, v, bf, b.kc, b.vt, N, g.Tj, kchk, vchk, b.ev_count, b.recheck, b.resmax, n_resmax, b.range, b.range_next);
  else
    ftattn_prepare<64><<<eg, 256, 0, st>>>(k, v, bf, b.kc, b.vt, N, g.Tj, kchk, vchk, b.ev_count, b.recheck, b.resmax, n_resmax, b.range, b.range_next);

  KArgs a;
  a.q = q; a.q_bf16 = bf; a.kc = b.kc; a.vt = b.vt; a.o = o; a.out_dtype = e.out_dtype;
  a.N = N; a.H = e.heads; a.Ti = g.Ti; a.Tj = g.Tj;
  a.head_group = head_group(D, ft, g.BH, g.Ti);
  const bool split = b.ws && !inject;
  a.n_tiles = g.BH * g.Ti;
  a.first_split = split ? g.first_split : a.n_tiles;
  a.piece = g.piece;
  a.ws = b.ws;
  a.scale = e.softmax_scale;
  a.scale_log2 = e.softmax_scale * 1.4426950408889634f;
  a.eps1 = e.eps1;
  a.tau_fast = 0.5f * (1.0f - std::exp(-e.eps1));
  a.tau_o = e.tau_o; a.delta_l = e.delta_l;
  a.correct = e.ft_mode == FTATTN_FT_CORRECT ? 1 : 0;
  a.rowsum_fold = e.rowsum_fold;
  a.rescale_margin = e.rescale_margin;
  a.faults = b.faults;
  a.fault_off = inject ? b.fault_off : nullptr;
  a.events = b.events; a.ev_count = b.ev_count; a.max_events = e.max_events;
  a.resmax = b.resmax; a.recheck = b.recheck; a.range = b.range;
  a.k = k; a.v = v;
  a.last = {};
  if (self) {
    a.last = {b.ended, b.ev_count, b.recheck, b.range, b.range_next};
    a.ev_count = (int32_t*)b.work; a.range = (uint32_t*)(b.work + 4); a.recheck = (unsigned long long*)(b.work + 8);
  }
  main_fn f = e.per_step ? select_perstep(D, e.causal != 0, inject, e.per_step)
              : e.stride == 1 ? select_elementwide(D, e.causal != 0, inject)
              : e.rescale_margin > 0.f ? select_lazy(D, ft, e.causal != 0, inject)
              : split ? select_split(D, ft, e.causal != 0)
              : self ? select_self(D, ft, e.causal != 0)
                              : select_kernel(D, ft, e.causal != 0, inject);
  if (timing && (he = hipEventRecord(timing[1], st)) != hipSuccess) return he;
  const int n_split = a.n_tiles - a.first_split;
  hipLaunchKernelGGL(f, dim3(a.first_split + (split ? g.shares : 0)), dim3(nwave_of(D) * 64), lds_bytes(D, ft), st, a);
  if ((he = hipGetLastError()) != hipSuccess) return he;
  if (split) {
    hipLaunchKernelGGL(select_finish(D, ft, e.causal != 0), dim3(n_split * nwave_of(D)), dim3(2 * D), 0, st, a);
    if ((he = hipGetLastError()) != hipSuccess) return he;
  }
  if (timing && (he = hipEventRecord(timing[2], st)) != hipSuccess) return he;
  return hipSuccess;
}

static int n_tiles_for_row(const ftattn_config& e, int row) {
  int last_key = e.causal ? row : e.seq - 1;
  return last_key / BN + 1;
}

extern "C" int ftattn_forward(ftattn_ctx* c, const void* q, const void* k, const void* v, void* o,
                              const ftattn_fault* faults, int32_t n_faults, void* hip_stream) {
  if (!c) return FTATTN_EINVAL;
  if (!q || !k || !v || !o) return fail(c, FTATTN_EINVAL, "null tensor pointer");
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return fail(c, FTATTN_EINVAL, "tensor pointers must be 16-byte aligned");
  if (n_faults < 0 || (n_faults > 0 && !faults)) return fail(c, FTATTN_EINVAL, "bad fault list");
  if (n_faults > c->fault_cap) return fail(c, FTATTN_EINVAL, "too many faults (limit 65536)");
  const ftattn_config& e = c->cfg;
  const int D = e.head_dim, N = e.seq;
  hipStream_t st = (hipStream_t)hip_stream;
  HIP_TRY(c, hipSetDevice(e.device));

  // ---- validate and bucket the fault list by (head, row tile), ordered by key tile
  if (n_faults > 0) {
    struct Keyed { long long key; DevFault f; };
    std::vector<Keyed> ks(n_faults);
    for (int i = 0; i < n_faults; ++i) {
      const ftattn_fault& f = faults[i];
      char msg[160];
      bool ok = f.b >= 0 && f.b < e.batch && f.h >= 0 && f.h < e.heads && f.row >= 0 && f.row < N && f.bit >= 0 && f.bit <= 31 &&
                f.stage >= FTATTN_ST_S && f.stage <= FTATTN_ST_OACC && f.kv_tile >= 0 && f.kv_tile < n_tiles_for_row(e, f.row);
      if (ok && (f.stage == FTATTN_ST_S || f.stage == FTATTN_ST_EXP))
        ok = f.col >= 0 && f.kv_tile == f.col / BN && (c->masked_faults ? f.stage == FTATTN_ST_EXP : f.col < N && (!e.causal || f.col <= f.row));
      if (ok && f.stage == FTATTN_ST_OACC) ok = f.col >= 0 && f.col < D;
      if (!ok) {
        snprintf(msg, sizeof msg, "fault %d (b=%d h=%d stage=%d kv_tile=%d row=%d col=%d bit=%d) names a masked or out-of-range position",
                 i, f.b, f.h, f.stage, f.kv_tile, f.row, f.col, f.bit);
        return fail(c, FTATTN_EINVAL, msg);
      }
      long long bucket = (long long)(f.b * e.heads + f.h) * c->geo.Ti + f.row / c->geo.BM;
      ks[i].key = (bucket << 32) | ((long long)f.kv_tile << 8) | f.stage;
      ks[i].f = DevFault{f.stage, f.kv_tile, f.row, f.col, f.bit};
    }
    std::stable_sort(ks.begin(), ks.end(), [](const Keyed& a, const Keyed& b) { return a.key < b.key; });
    size_t nb = (size_t)c->geo.BH * c->geo.Ti;
    std::fill(c->h_fault_off, c->h_fault_off + nb + 1, 0);
    for (int i = 0; i < n_faults; ++i) { c->h_faults[i] = ks[i].f; c->h_fault_off[(ks[i].key >> 32) + 1]++; }
    for (size_t i = 0; i < nb; ++i) c->h_fault_off[i + 1] += c->h_fault_off[i];
    HIP_TRY(c, hipMemcpyAsync(c->d_faults, c->h_faults, sizeof(DevFault) * n_faults, hipMemcpyHostToDevice, st));
    HIP_TRY(c, hipMemcpyAsync(c->d_fault_off, c->h_fault_off, sizeof(int32_t) * (nb + 1), hipMemcpyHostToDevice, st));
    HIP_TRY(c, hipStreamSynchronize(st));   // the staging buffers may be rewritten by the next call
  }

  Buffers bufs;
  bufs.kc = c->kc; bufs.vt = c->vt; bufs.ws = c->ws; bufs.faults = c->d_faults; bufs.fault_off = n_faults > 0 ? c->d_fault_off : nullptr;
  bufs.events = c->d_events;
  bufs.ev_count = (int32_t*)(c->d_stat + STAT_EVENTS);
  bufs.recheck = (unsigned long long*)(c->d_stat + STAT_RECHECK);
  bufs.resmax = (uint32_t*)(c->d_stat + STAT_RESMAX);
  bufs.work = c->d_stat + STAT_WORK;
  bufs.ended = (uint32_t*)(bufs.work + 16);
  uint32_t* range = (uint32_t*)(c->d_stat + STAT_RANGE);
  bufs.range = range + (c->calls & 1u); bufs.range_next = range + ((c->calls + 1u) & 1u);
  hipError_t le = launch_pass(e, c->geo, bufs, q, k, v, o, n_faults > 0, st, c->timing ? c->ev : nullptr);
  if (le != hipSuccess) return fail(c, FTATTN_EHIP, std::string("launch: ") + hipGetErrorString(le));
  c->last_stream = st;
  c->ran = true;
  ++c->calls;
  return FTATTN_OK;
}

// For the tests, and no part of the interface: fault lists may name the exponential of a masked score from here on.
extern "C" void ftattn_accept_masked_faults(ftattn_ctx* c) { c->masked_faults = true; }

extern "C" int ftattn_report(ftattn_ctx* c, ftattn_report_view* out) {
  if (!c || !out) return FTATTN_EINVAL;
  if (!c->ran) return fail(c, FTATTN_EINVAL, "no forward call to report on");
  const ftattn_config& e = c->cfg;
  HIP_TRY(c, hipSetDevice(e.device));
  // The copy goes over the default stream, behind whatever runs there: a captured call may have been replayed on
  // it.  A call made on that stream needs no wait of its own before.
  if (c->last_stream) HIP_TRY(c, hipStreamSynchronize(c->last_stream));
  HIP_TRY(c, hipMemcpyAsync(c->h_stat, c->d_stat, c->stat_bytes, hipMemcpyDeviceToHost, nullptr));
  HIP_TRY(c, hipStreamSynchronize(nullptr));
  int32_t count = 0;
  unsigned long long recheck = 0;
  uint32_t range = 0;
  std::memcpy(&count, c->h_stat + STAT_EVENTS, sizeof count);
  std::memcpy(&recheck, c->h_stat + STAT_RECHECK, sizeof recheck);
  std::memcpy(&range, c->h_stat + STAT_RANGE + sizeof range * ((c->calls - 1u) & 1u), sizeof range);
  int stored = std::min(count, e.max_events);
  c->events.resize(stored);
  if (stored) HIP_TRY(c, hipMemcpy(c->events.data(), c->d_events, sizeof(ftattn_event) * stored, hipMemcpyDeviceToHost));
  std::sort(c->events.begin(), c->events.end(), [](const ftattn_event& x, const ftattn_event& y) {
    if (x.b != y.b) return x.b < y.b;
    if (x.h != y.h) return x.h < y.h;
    if (x.check != y.check) return x.check < y.check;
    if (x.kv_tile != y.kv_tile) return x.kv_tile < y.kv_tile;
    if (x.row != y.row) return x.row < y.row;
    return x.col < y.col;
  });
  size_t n_rt = (size_t)c->geo.BH * c->geo.Ti;
  c->tile_flags.assign(n_rt * c->geo.Tj, 0);
  c->rowtile_flags.assign(n_rt, 0);
  for (const ftattn_event& ev : c->events) {
    size_t rt = (size_t)(ev.b * e.heads + ev.h) * c->geo.Ti + ev.row / c->geo.BM;
    if (ev.check == FTATTN_CHECK_S) c->tile_flags[rt * c->geo.Tj + ev.kv_tile] |= FTATTN_TF_DET_S | (ev.action ? FTATTN_TF_COR_S : 0);
    else if (ev.check == FTATTN_CHECK_EXP) c->tile_flags[rt * c->geo.Tj + ev.kv_tile] |= FTATTN_TF_DET_EXP | (ev.action ? FTATTN_TF_COR_EXP : 0);
    else if (ev.check == FTATTN_CHECK_L) c->rowtile_flags[rt] |= FTATTN_RF_DET_L | (ev.action ? FTATTN_RF_COR_L : 0);
    else c->rowtile_flags[rt] |= FTATTN_RF_DET_O | (ev.action ? FTATTN_RF_COR_O : 0);
  }
  if (count > stored)
    for (auto& f : c->rowtile_flags) f |= FTATTN_RF_EVENT_OVERFLOW;
  c->resmax.resize(n_rt * 4);
  std::memcpy(c->resmax.data(), c->h_stat + STAT_RESMAX, sizeof(float) * n_rt * 4);
  out->n_events = stored;
  out->n_events_dropped = count - stored;
  out->events = c->events.data();
  out->tiles_m = c->geo.Ti;
  out->tiles_n = c->geo.Tj;
  out->tile_flags = c->tile_flags.data();
  out->rowtile_flags = c->rowtile_flags.data();
  out->residual_max = c->resmax.data();
  out->recheck_entries = (int64_t)recheck;
  out->range_flags = (int32_t)range;
  return FTATTN_OK;
}

extern "C" int ftattn_set_timing(ftattn_ctx* c, int32_t enabled) {
  if (!c) return FTATTN_EINVAL;
  HIP_TRY(c, hipSetDevice(c->cfg.device));
  if (enabled)
    for (hipEvent_t& e : c->ev)
      if (!e) HIP_TRY(c, hipEventCreate(&e));
  c->timing = enabled != 0;
  return FTATTN_OK;
}

extern "C" int ftattn_get_timing(ftattn_ctx* c, float ms[2]) {
  if (!c || !ms) return FTATTN_EINVAL;
  if (!c->timing || !c->ran) return fail(c, FTATTN_EINVAL, "timing is not enabled or no forward has run");
  HIP_TRY(c, hipSetDevice(c->cfg.device));
  HIP_TRY(c, hipEventSynchronize(c->ev[2]));
  HIP_TRY(c, hipEventElapsedTime(&ms[0], c->ev[0], c->ev[1]));
  HIP_TRY(c, hipEventElapsedTime(&ms[1], c->ev[1], c->ev[2]));
  return FTATTN_OK;
}

extern "C" int ftattn_destroy(ftattn_ctx* c) {
  if (!c) return FTATTN_EINVAL;
  (void)hipSetDevice(c->cfg.device);
  (void)hipDeviceSynchronize();
  release(c);
  return FTATTN_OK;
}

extern "C" const char* ftattn_last_error(const ftattn_ctx* c) {
  return c ? c->err.c_str() : g_create_err.c_str();
}

// ------------------------------------------------------------------ the entry point that allocates nothing
//
// Same pass, same kernels, with every device buffer carved out of one file-scope device array
// instead of a context's allocations.  The array exists once per GPU for the life of the process;
// the address a kernel may use is the one hipGetSymbolAddress returns for the current device (the
// array's name is only a host-side handle).

constexpr size_t STATIC_SCRATCH_BYTES = (size_t)FTATTN_STATIC_SCRATCH_MIB << 20;
constexpr int STATIC_MAX_EVENTS = 4096;
constexpr int STATIC_MAX_DEVICES = 64;
// Behind what a workgroup may read past the last encoded tile: Buffers::ended, a word for each number of heads that a call may have
// (a head takes at least one key and one value tile of head_dim 64).
constexpr size_t STATIC_ENDED = STATIC_SCRATCH_BYTES + tiles_beyond(128);
constexpr size_t STATIC_MAX_HEADS = STATIC_SCRATCH_BYTES / (2 * (BN + CKR) * 64 * 2);
static __device__ __align__(256) unsigned char scratch[STATIC_ENDED + (STATIC_MAX_HEADS + 1) * sizeof(uint32_t)];

static std::mutex g_static_mu;
static unsigned char* g_static_ptr[STATIC_MAX_DEVICES];      // per device, null until set up
static bool g_static_lds[STATIC_MAX_DEVICES][8];             // kernels of a head size, protected or not, causal or not, prepared
static unsigned g_static_calls[STATIC_MAX_DEVICES];          // parity picks the range word of a call
static thread_local char g_static_err[256];

static int static_fail(int code, const char* what, hipError_t he = hipSuccess) {
  if (he != hipSuccess) snprintf(g_static_err, sizeof g_static_err, "%s: %s", what, hipGetErrorString(he));
  else snprintf(g_static_err, sizeof g_static_err, "%s", what);
  return code;
}

extern "C" const char* ftattn_static_last_error(void) { return g_static_err; }

extern "C" int ftattn_forward_static(const ftattn_config* cfg, const void* q, const void* k, const void* v, void* o,
                                     int32_t* n_events_dev, void* hip_stream) {
  g_static_err[0] = 0;
  if (!cfg) return static_fail(FTATTN_EINVAL, "null configuration");
  ftattn_config e;
  Geometry g;
  const char* why;
  if (int rc = resolve_config(cfg, e, g, why)) return static_fail(rc, why);
  if (e.per_step != 0 || e.stride != 8 || e.rescale_margin > 0.f)
    return static_fail(FTATTN_EUNSUPPORTED, "the static entry point runs the default verification scheme (per_step 0, stride 8, rescale_margin 0)");
  if (e.device < 0 || e.device >= STATIC_MAX_DEVICES) return static_fail(FTATTN_EINVAL, "device ordinal out of range");
  if (!q || !k || !v || !o) return static_fail(FTATTN_EINVAL, "null tensor pointer");
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return static_fail(FTATTN_EINVAL, "tensor pointers must be 16-byte aligned");
  if ((uintptr_t)n_events_dev & 3) return static_fail(FTATTN_EINVAL, "n_events_dev must be 4-byte aligned");
  if (e.max_events > STATIC_MAX_EVENTS) e.max_events = STATIC_MAX_EVENTS;

  // layout of the array: counters | residual maxima | event log | encoded key tiles | encoded value tiles
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t off_resmax = 256;
  const size_t off_events = off_resmax + up(sizeof(uint32_t) * (size_t)g.BH * g.Ti * 4);
  const size_t off_kc = off_events + up(sizeof(ftattn_event) * (size_t)e.max_events);
  const size_t off_vt = off_kc + up(g.n_kc * 2);
  const size_t off_ws = off_vt + up(g.n_vt * 2), need = off_ws;
  // (where the state of split row tiles does not fit as well, none is split)
  const bool split = g.n_ws != 0 && off_ws + g.n_ws * sizeof(float) <= STATIC_SCRATCH_BYTES;
  if (need > STATIC_SCRATCH_BYTES) {
    snprintf(g_static_err, sizeof g_static_err, "this shape needs %zu bytes of scratch, the static array holds %zu", need, STATIC_SCRATCH_BYTES);
    return FTATTN_EUNSUPPORTED;
  }

  hipError_t he = hipSetDevice(e.device);
  if (he != hipSuccess) return static_fail(FTATTN_EHIP, "hipSetDevice", he);
  unsigned char* base;
  unsigned calls;
  {
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[e.device]) {
      void* ptr = nullptr;
      he = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (he != hipSuccess || !ptr) return static_fail(FTATTN_EHIP, "hipGetSymbolAddress(scratch)", he);
      g_static_ptr[e.device] = (unsigned char*)ptr;
    }
    const int di = (e.head_dim == 128 ? 4 : 0) + (e.ft_mode != FTATTN_FT_OFF ? 2 : 0) + (e.causal != 0 ? 1 : 0);
    if (!g_static_lds[e.device][di]) {
      he = allow_lds(e, true, true, why);
      if (he != hipSuccess) return static_fail(FTATTN_EHIP, why, he);
      g_static_lds[e.device][di] = true;
    }
    base = g_static_ptr[e.device];
    calls = g_static_calls[e.device]++;
  }

  Buffers bufs;
  bufs.ev_count = n_events_dev ? n_events_dev : (int32_t*)base;
  bufs.recheck = (unsigned long long*)(base + 8);
  bufs.work = base + STAT_WORK;
  bufs.ended = (uint32_t*)(base + STATIC_ENDED) + ((size_t)g.BH <= STATIC_MAX_HEADS ? g.BH : 0);
  bufs.range = (uint32_t*)(base + 16) + (calls & 1u);
  bufs.range_next = (uint32_t*)(base + 16) + ((calls + 1u) & 1u);
  bufs.resmax = (uint32_t*)(base + off_resmax);
  bufs.events = (ftattn_event*)(base + off_events);
  bufs.kc = (_Float16*)(base + off_kc);
  bufs.vt = (_Float16*)(base + off_vt);
  bufs.ws = split ? (float*)(base + off_ws) : nullptr;
  he = launch_pass(e, g, bufs, q, k, v, o, false, (hipStream_t)hip_stream, nullptr);
  if (he != hipSuccess) return static_fail(FTATTN_EHIP, "launch", he);
  return FTATTN_OK;
}
