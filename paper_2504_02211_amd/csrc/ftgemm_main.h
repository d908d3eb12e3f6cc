// Fault-tolerant linear layer Y = X W^T for gfx950 / CDNA4: the strided ABFT of Section 3.3 of
// the paper (tensor checksums of eq. (13), (14); checksum products of eq. (15), (16); location
// and repair as stated after eq. (16)) on a plain fp16 or bf16 GEMM with fp32 accumulation.
//
// Execution shape.  A workgroup of four or eight waves computes a tile of BM tokens x BF
// features of Y; a checksum block is 256 features, and a tile never holds less than one block
// (BF = 256, or all features of a matrix that has no more than 128).  A wave owns WT x WF
// accumulator blocks of 16 tokens x 16 features of Y^T = W X^T (16x16x32 fp16 or bf16 MFMA: the
// weight rows are the A operand, the token rows the B operand), and its share of the products of
// the 32 checksum rows.  A lane then holds one token per token block and, per feature block, the
// features 4*(lane/16) + r: feature index mod 8 is 4*((lane/16)%2)+r, so the folds of the four
// checksum classes a lane sees are sums over the registers of the lane and of lane^32; what the waves
// of one token range have to exchange after the last K step is one partial fold per class, through LDS.
//
// What bounds it: the clock that power allows, and a matrix pipe that is 71 % busy at it (1.77 GHz; 16384
// tokens, 4096 -> 16384 features).  With operands in registers and nothing else running, 32x32x16 products
// sustain 1660 TFLOP/s on random fp16 data (1.7 GHz) and 16x16x32 products 1880 (2.0 GHz), against 2420 and
// 2320 on zeros (2.4 GHz): the smaller block reads and writes half as many accumulators per flop.  A wave owns
// a block of blocks because LDS reads and L2-to-LDS traffic are paid from the same budget.
//
// The K dimension is walked in steps of BK through a ring of NST LDS stages filled by direct
// global-to-LDS loads; tiles are stored unpadded with the 16-byte chunk index XOR-ed with a
// function of the row, which keeps the MFMA operand reads free of bank conflicts (those counted, 2 % of the
// LDS cycles, are the results on their way through LDS).  Operands are read
// ahead of their products, also across the stage boundary: the barrier of a stage sits AHEAD rows before
// its end, where the last operands of the stage are in registers, so that no wave waits for LDS after it.
//
// Measured (16384 tokens, 4096 -> 16384 features, fp16): 1810-1950 us protected (by the clock that a card's power allows; 1859 where the
// epilogue in which every wave formed all verdicts took 1884), 1660-1700 us with the checks compiled out, against
// 2250 / 1930 us for one 32-token row of 32x32x16 blocks per wave.  Four waves of 8 x 8 blocks would read a third less
// LDS, but their 288 accumulators do not fit next to the operands without register copies in the loop.
#pragma once
#include "ftattn_main.h"
#include "ftgemm.h"

#include <utility>
#include <vector>

namespace ftgemm {

using ftattn::half8;
using ftattn::uint4v;
using ftattn::as_u;
using ftattn::as_f;
using ftattn::fmax2;
using ftattn::finitef;
using ftattn::flip_if;
using ftattn::gload_lds16_off;
using ftattn::sum32;
using ftattn::xchg32;
using ftattn::phase_barrier;

constexpr int GBN = 256;      // output features per checksum block
constexpr int GCK = 32;       // checksum rows per block: {c1 hi, c1 lo, c2 hi, c2 lo} x 8 classes
constexpr int GFOLD = GBN / 8;

template <int N> __device__ __forceinline__ void wait_vmcnt() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }

// f(0), f(1), ... f(N-1) with the index as a compile-time constant
template <class F, int... I> __device__ __forceinline__ void for_each_index_of(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void for_each_index(F&& f) { for_each_index_of(f, std::make_integer_sequence<int, N>{}); }

constexpr int WS_BLOCKS = 18;  // 16 x 16 blocks of a checksum block's accumulators: 16 of results, 2 of checksum products

struct GFault { int32_t row, col, bit; };

// What one workgroup reports: the events it logged (a run of entries of the event ring, starting at
// `first` modulo the ring's size) and its largest passing statistic.  Every workgroup of every call
// writes its slot, so nothing has to be cleared between calls.
struct GSlot { uint32_t first; int32_t n; float stat; };

typedef float float4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// 16-bit storage helpers (fp16 or bf16 bit patterns)
template <bool BF> __device__ __forceinline__ float to_f32(uint16_t u) {
  if (BF) return as_f((uint32_t)u << 16);
  return (float)__builtin_bit_cast(_Float16, u);
}
// round-to-nearest-even to the storage type (Inf / NaN pass through)
template <bool BF> __device__ __forceinline__ uint16_t from_f32(float x) {
  if (!BF) return __builtin_bit_cast(uint16_t, (_Float16)x);
  const uint32_t u = as_u(x);
  if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

struct GArgs {
  const uint16_t* x;       // [M][K] fp16 or bf16 patterns
  const uint16_t* w;       // [N][K]
  const uint16_t* wc;      // [Tn][GCK][K] checksum rows of W, same type
  void* y;                 // [M][N] fp32, or the input type
  int32_t out_dtype;
  int32_t M, N, K, Tm, Tn; // Tm: token tiles of the launched tile shape, Tn: feature blocks
  float tau_rel, tau_abs;
  int32_t correct;
  const GFault* faults;
  int32_t n_faults;
  ftgemm_event* events;    // ring of ring_mask + 1 entries
  uint32_t* cursor;        // next free entry of the ring, counted without wrapping
  uint32_t ring_mask;
  GSlot* slots;            // one per workgroup (of a problem)
  int32_t* n_slots;        // how many that is: what a report goes by, because the launch that it reports on may be
                           // the replay of a captured one, with another tile shape than the host's last call
  // batch of independent products (blockIdx.y): element strides between consecutive problems of x, w,
  // wc, the event rings and the slots, byte stride of y; one cursor per problem.  All zero for a single product.
  long long bs_x, bs_w, bs_wc, bs_y_bytes, bs_events, bs_slots;
  int32_t skip_upper;      // 1: output tiles that lie entirely above the diagonal (first feature > last token) are
                           // not launched (the score matrix of a causal attention: nobody reads them)
  int32_t k_lower;         // 1: x is lower-triangular (the weights of a causal attention): contraction steps beyond the
                           // last token of the tile multiply zeros and are skipped.  One feature block only
  int32_t tiles;           // with one of these two the batch is in blockIdx.x as well: tiles launched per problem ...
  int32_t head_group;      // ... and (k_lower) problems whose tiles are issued together (causal_row_tile)
  int32_t parts;           // > 1: the K dimension is split over blockIdx.z, the shares go to ws
  float4v* ws;             // [part][16-token block][feature block of 256][WS_BLOCKS][lane]
  int32_t ws_tokens;       // 16-token blocks per part
  int32_t transposed;      // 1: the kernel's (token, feature) is the caller's (column, row) of Y: checksums over the
                           // caller's token rows; results are stored, and events named, with the two exchanged
};

// Tensor checksums of the weight rows of every 256-feature block (eq. (13), (14)): a thread folds 8 of
// the 32 rows c, c+8, ... of its (class c, 16-byte chunk of K) in fp32, four neighbours (lanes 8 apart)
// add up, and the sums are stored as a high word and a low word of the input type (high = the sum
// rounded, low = the remainder rounded).  Rows beyond N count as zero.  Bound: reading W once; with one
// thread per whole (class, chunk) a 2048 x 1024 matrix had 32 workgroups on 256 CUs and took 14 us.
template <bool BF>
__device__ __forceinline__ void encode_weight_rows(const uint16_t* __restrict__ w, uint16_t* __restrict__ wc, int N, int K, int tn, int chunks8) {
  typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
  const int tid = threadIdx.x;
  const int cls = tid >> 5, part = (tid >> 3) & 3, ch = chunks8 * 8 + (tid & 7);
  const bool on = ch * 8 < K;
  float c1[8], c2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { c1[e] = 0.f; c2[e] = 0.f; }
#pragma unroll
  for (int i = 0; i < GFOLD / 4; ++i) {
    const int l = 4 * i + part, n = tn * GBN + cls + 8 * l;
    u16x8 h = (u16x8)(uint16_t)0;
    if (on && n < N) h = *reinterpret_cast<const u16x8*>(w + (size_t)n * K + ch * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = to_f32<BF>(h[e]);
      c1[e] += v;
      c2[e] += (float)(l + 1) * v;
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    c1[e] += __shfl_xor(c1[e], 8); c2[e] += __shfl_xor(c2[e], 8);
    c1[e] += __shfl_xor(c1[e], 16); c2[e] += __shfl_xor(c2[e], 16);
  }
  if (!on) return;
  // each of the four stores one of the four words
  u16x8 out;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float c = part < 2 ? c1[e] : c2[e];
    const uint16_t high = from_f32<BF>(c);
    out[e] = part & 1 ? from_f32<BF>(c - to_f32<BF>(high)) : high;
  }
  *reinterpret_cast<u16x8*>(wc + ((size_t)tn * GCK + 8 * part + cls) * K + ch * 8) = out;
}

template <bool BF>
__global__ __launch_bounds__(256) void ftgemm_encode_w(const uint16_t* __restrict__ w, uint16_t* __restrict__ wc, int N, int K,
                                                       long long bs_w, long long bs_wc) {
  encode_weight_rows<BF>(w + (size_t)blockIdx.z * bs_w, wc + (size_t)blockIdx.z * bs_wc, N, K, blockIdx.x, blockIdx.y);      // z: matrix of a batch
}

// Tile shape: BM tokens x BF features, a wave takes WT x WF blocks of 16 x 16, ring of NST stages, PER_CU workgroups per CU
// (whose epilogue may need more LDS than the ring: EPILOGUE).
template <int BM_, int BF_, int WT_, int WF_, int BK_, int NST_, int PER_CU_ = 1, int EPILOGUE_ = 0> struct GTile {
  static constexpr int PER_CU = PER_CU_;
  static constexpr int BM = BM_, BF = BF_, WT = WT_, WF = WF_, BK = BK_, NST = NST_;
  static constexpr int NWT = BM / (16 * WT), NWF = BF / (16 * WF);   // waves along the tokens / along the features
  static constexpr int NW = NWT * NWF;                               // waves per workgroup
  static_assert(NW == 4 || NW == 8, "one or two waves per SIMD");
  // checksum products: the NWF waves that share a token range split its WT token blocks among them;
  // where there are fewer blocks than waves the last waves have none.  (Splitting the k-steps of a block
  // among waves instead gives false alarms: a class with a single fold passes by having the products of
  // the fold and of its checksum accumulated in the same order.)
  static constexpr int CB = WT >= NWF ? WT / NWF : 1;
  static constexpr int ROWB = BK * 2;                                // bytes per tile row in LDS
  static constexpr int CPR = BK / 8, PR = 1024 / ROWB;               // 16-byte chunks per row; rows per 1 KB piece
  static_assert(CPR == 8, "the swizzle of a row's chunks is one of eight");
  static constexpr int XP = BM / PR, WP = BF / PR, CP = GCK / PR;    // pieces per stage
  // ... per wave.  Where there are fewer pieces of checksum rows than waves the last waves have none (C_SPARE); in the largest
  // tile, which has no registers left for a second form of its loop, and with fewer pieces of token rows than waves, some
  // are fetched twice (to the same place)
  static constexpr bool C_SPARE = CP < NW && BM < 256;
  static constexpr int XW = (XP + NW - 1) / NW, WW = (WP + NW - 1) / NW, CW = 1;
  static_assert((XP % NW == 0 || XP < NW) && (WP % NW == 0) && CP <= NW, "pieces split evenly");
  template <bool FT> static constexpr int nload() { return XW + WW + (FT ? CW : 0); }
  template <bool FT> static constexpr int bytes() { return (BM + BF + (FT ? GCK : 0)) * ROWB; }
  template <bool FT> static constexpr int lds() { return FT && EPILOGUE_ > NST * bytes<FT>() ? EPILOGUE_ : NST * bytes<FT>(); }
  static_assert((NST - 1) * (XW + WW + CW) <= 63, "counted waits use a 6-bit immediate");
  static_assert(PER_CU * NST * (BM + BF + GCK) * ROWB <= 160 * 1024 && PER_CU * EPILOGUE_ <= 160 * 1024 && NST <= 3, "LDS; the waits of the last stages");
};

// The tile shapes in use (see gemm_plan in ftgemm.hip for when).  The tiles of 128 and 64 tokens are spread over eight waves,
// two per SIMD, although four with blocks twice as high would read a third less LDS: a wave alone on its SIMD waits
// for LDS and for its own barrier (2048 x 2048 x 1024 19.2 -> 16.9 us with 64 tokens, 5000 x 1300 x 8000 152 -> 134 with 128).
using TileWide = GTile<256, 256, 4, 8, 64, 2>;
using TileHalf = GTile<128, 256, 4, 4, 64, 3>;
using TileQuarter = GTile<64, 256, 2, 4, 64, 3>;
using TileStrip = GTile<32, 256, 2, 4, 64, 3>;
using TileNarrow = GTile<128, 128, 4, 4, 64, 3>;
using TileFinish = GTile<16, 256, 1, 4, 64, 1>;      // epilogue only
using TileSlim = GTile<256, 64, 4, 4, 64, 3>;
using TileNarrow2 = GTile<64, 128, 2, 4, 64, 2, 2>;
using TileSlim2 = GTile<128, 64, 2, 4, 64, 2, 2>;
// Short contractions with large results: a stage at a time, two workgroups to a CU, so that one loads and multiplies while the
// other's results are on their way out.
using TileLow = GTile<128, 256, 4, 8, 64, 1, 2, 58 * 1024>;

__device__ __forceinline__ void write_slot(const GArgs& a, int logical, const GSlot& s) {
  a.slots[logical] = s;
  if (logical == 0) *a.n_slots = a.tiles ? a.tiles : (int32_t)gridDim.x;
}

// Tiles on or below the diagonal: a block row of 256 tokens, the b-th, has b + 1 feature blocks for each of its token tiles.
__host__ __device__ __forceinline__ int lower_tiles(int Tm, int bm) {
  const int per = GBN / bm, b = Tm / per;
  return per * (b * (b + 1) / 2) + (Tm - b * per) * (b + 1);
}
__device__ __forceinline__ void lower_tile(int t, int bm, int& tm, int& tn) {
  const int per = GBN / bm;
  int b = 0;
  while (t >= per * (b + 1)) { t -= per * (b + 1); ++b; }
  tm = b * per + t / (b + 1);
  tn = t % (b + 1);
}

__device__ __forceinline__ void log_gemm_event(const GArgs& a, uint32_t at, int row, int col, float res, int action) {
  ftgemm_event e;
  e.row = a.transposed ? col : row; e.col = a.transposed ? row : col; e.residual = res; e.action = action;
  a.events[at & a.ring_mask] = e;
}

// What follows the last accumulation step of a tile whose accumulators are in registers: (fault
// injection,) verification, location and repair, and the store.  Needs T's ring of LDS, free.
template <class T, bool FT, bool INJ, bool BF>
__device__ __forceinline__ void finish_tile(const GArgs& a, char* smem, float4v (&acc)[T::WF][T::WT], float4v (&sc)[T::CB][2],
                                            const int m0, const int n0, const int logical) {
  constexpr int WT = T::WT, WF = T::WF, NWF = T::NWF, CB = T::CB;
  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wt = wave / NWF, wf = wave % NWF;
  const int M = a.M, N = a.N;
  const int rot = wf * CB % WT;
  const bool check_wave = FT && wf * CB < WT;
  auto block_of = [&](int t) __attribute__((always_inline)) -> int { return (t + rot) % WT; };
  const int nf0 = n0 + 16 * WF * wf;       // first feature of this wave
  // result r of block (y, t) for the folds: features beyond N (clamped weight rows) count as zero
  auto fold_value = [&](int y, int t, int r, bool edge) __attribute__((always_inline)) -> float {
    return edge && nf0 + 16 * y + 4 * lg + r >= N ? 0.f : acc[y][t][r];
  };
  auto store_one = [&](int row, int col, float v) __attribute__((always_inline)) {
    const size_t at = a.transposed ? (size_t)col * M + row : (size_t)row * N + col;
    if (a.out_dtype == FTGEMM_F32) reinterpret_cast<float*>(a.y)[at] = v;
    else reinterpret_cast<uint16_t*>(a.y)[at] = from_f32<BF>(v);
  };
  auto row_of = [&](int t) __attribute__((always_inline)) -> int { return m0 + 16 * (WT * wt + block_of(t)) + lq; };
  if (INJ) {
    for (int fi = 0; fi < a.n_faults; ++fi) {
      const GFault f = a.faults[fi];
      const int lc = f.col - nf0;
      if (lc < 0 || lc >= 16 * WF) continue;
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        const bool mine = f.row == row_of(t) && lg == ((lc & 15) >> 2);
#pragma unroll
        for (int y = 0; y < WF; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[y][t][r] = flip_if(acc[y][t][r], mine && (lc >> 4) == y && (lc & 3) == r, f.bit);
      }
    }
  }
  // Exchange area, in floats: [token block of the tile][kind][wave along the features][lane][2]; kinds: fold sums of the classes,
  // sums of magnitudes, first checksum products.  A class r = 0..3 of lane % 32 stands with lane % 32 + 32 (r % 2), entry r / 2:
  // where it is after the two halves of two classes were added up in one exchange of lanes (pair_sums).  Behind it a
  // staging area per wave, through which the results go out in whole rows.
  constexpr int EX_BYTES = FT ? T::BM / 16 * 3 * NWF * 64 * 8 : 0, SHARED_BYTES = 64;
  constexpr int OUT_PITCH = 16 * WF * 4 + 16, OUT_PITCH_T = 16 * WT * 4 + 16;
  constexpr int OUT_BYTES = 16 * (OUT_PITCH > OUT_PITCH_T ? OUT_PITCH : OUT_PITCH_T);
  constexpr int TAIL_BYTES = T::NW * OUT_BYTES > EX_BYTES ? T::NW * OUT_BYTES : EX_BYTES;      // staging, or a second exchange area
  static_assert(EX_BYTES + SHARED_BYTES + TAIL_BYTES <= T::template lds<FT>(), "exchange and staging areas fit the ring");
  typedef float float2v __attribute__((ext_vector_type(2)));
  auto ex_pair = [&](int block, int kind, int f) __attribute__((always_inline)) -> float2v& {
    return reinterpret_cast<float2v*>(smem)[((block * 3 + kind) * NWF + f) * 64 + lane];
  };
  auto ex = [&](int t, int val, int f) __attribute__((always_inline)) -> float& {       // val: 4 * kind + class
    const int at = (((WT * wt + block_of(t)) * 3 + (val >> 2)) * NWF + f) * 64 + (lane & 31) + 32 * (val & 1);
    return reinterpret_cast<float*>(smem)[2 * at + ((val >> 1) & 1)];
  };
  // sums of lane and lane^32 of four values: of the first and third in the lower half of the lanes, of the others in the upper half
  auto pair_sums = [&](const float (&v)[4]) __attribute__((always_inline)) -> float2v {
    const auto x = __builtin_amdgcn_permlane32_swap(as_u(v[0]), as_u(v[1]), false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(as_u(v[2]), as_u(v[3]), false, false);
    return float2v{as_f(x[0]) + as_f(x[1]), as_f(y[0]) + as_f(y[1])};
  };
  auto ex2 = [&](int t, int val, int f) __attribute__((always_inline)) -> float& {
    return *reinterpret_cast<float*>(reinterpret_cast<char*>(&ex(t, val, f)) + EX_BYTES + SHARED_BYTES);
  };
  int* shared_n = reinterpret_cast<int*>(smem + EX_BYTES);            // [0] rows flagged, [1] events, [2] first entry
  float* shared_stat = reinterpret_cast<float*>(shared_n + 4);
  char* stage_out = smem + EX_BYTES + SHARED_BYTES + wave * OUT_BYTES;
  const bool edge = n0 + T::BF > N;
  if (FT && tid < 3) shared_n[tid] = 0;

  // One token block: fold sums to the exchange area, results to the staging area and out.  The lane
  // holds features nf0 + 16*y + 4*lg + (0..3) of its token.  Stored from here, a wave-wide store
  // would touch 16 rows for a few bytes each; through LDS it is a few whole rows.
  auto block_out = [&](int t, auto out32_tag, auto edge_tag) __attribute__((always_inline)) {
    constexpr bool OUT32 = decltype(out32_tag)::value, EDGE = decltype(edge_tag)::value;
    constexpr int ES = OUT32 ? 4 : 2, PITCH = 16 * WF * ES + 16;
    float sum1[4] = {0.f, 0.f, 0.f, 0.f}, mag[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int y = 0; y < WF; ++y) {
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = fold_value(y, t, r, EDGE);
        if (FT) { sum1[r] += x[r]; mag[r] += __builtin_fabsf(x[r]); }
      }
      if (!a.transposed) {
        char* at = stage_out + lq * PITCH + (16 * y + 4 * lg) * ES;
        if (OUT32) {
          *reinterpret_cast<float4*>(at) = make_float4(x[0], x[1], x[2], x[3]);
        } else {
          uint16_t hv[4] = {from_f32<BF>(x[0]), from_f32<BF>(x[1]), from_f32<BF>(x[2]), from_f32<BF>(x[3])};
          *reinterpret_cast<uint2*>(at) = *reinterpret_cast<uint2*>(hv);
        }
      }
    }
    if (FT) {
      const int b = WT * wt + block_of(t);
      ex_pair(b, 0, wf) = pair_sums(sum1);
      ex_pair(b, 1, wf) = pair_sums(mag);
      if (t < CB && check_wave) {
        const float4v c = sc[t < CB ? t : 0][0];
        ex_pair(b, 2, 0) = pair_sums({c[0], c[1], c[2], c[3]});
      }
    }
    if (a.transposed) return;
    const int r0 = m0 + 16 * (WT * wt + block_of(t));
    if ((N * ES) % 16 == 0) {
      constexpr int LPR = 16 * WF * ES / 16, RPI = 64 / LPR;          // lanes per row, rows per store
      const int col = nf0 + (lane % LPR) * (16 / ES);
#pragma unroll
      for (int i = 0; i < (16 + RPI - 1) / RPI; ++i) {
        const int r = i * RPI + lane / LPR;
        const uint4v v = *reinterpret_cast<const uint4v*>(stage_out + r * PITCH + (lane % LPR) * 16);
        if (r < 16 && r0 + r < M && (!EDGE || col < N)) *reinterpret_cast<uint4v*>(reinterpret_cast<char*>(a.y) + ((size_t)(r0 + r) * N + col) * ES) = v;
      }
    } else {
      for (int e = lane; e < 16 * 16 * WF; e += 64) {
        const int r = e / (16 * WF), c = e % (16 * WF);
        if (r0 + r < M && nf0 + c < N) {
          const size_t at = (size_t)(r0 + r) * N + nf0 + c;
          if (OUT32) reinterpret_cast<float*>(a.y)[at] = *reinterpret_cast<const float*>(stage_out + r * PITCH + c * ES);
          else reinterpret_cast<uint16_t*>(a.y)[at] = *reinterpret_cast<const uint16_t*>(stage_out + r * PITCH + c * ES);
        }
      }
    }
  };
  // The same for a transposed result, one feature block at a time: Y is [N][M] seen from here.
  auto block_out_transposed = [&](int y, auto out32_tag) __attribute__((always_inline)) {
    constexpr bool OUT32 = decltype(out32_tag)::value;
    constexpr int ES = OUT32 ? 4 : 2, PITCH = 16 * WT * ES + 16;
#pragma unroll
    for (int t = 0; t < WT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        char* at = stage_out + (4 * lg + r) * PITCH + (16 * block_of(t) + lq) * ES;
        if (OUT32) *reinterpret_cast<float*>(at) = acc[y][t][r];
        else *reinterpret_cast<uint16_t*>(at) = from_f32<BF>(acc[y][t][r]);
      }
    const int c0 = nf0 + 16 * y, r0 = m0 + 16 * WT * wt;
    if ((M * ES) % 16 == 0) {
      constexpr int LPR = 16 * WT * ES / 16, RPI = 64 / LPR;
      const int row = r0 + (lane % LPR) * (16 / ES);
#pragma unroll
      for (int i = 0; i < (16 + RPI - 1) / RPI; ++i) {
        const int c = i * RPI + lane / LPR;
        const uint4v v = *reinterpret_cast<const uint4v*>(stage_out + c * PITCH + (lane % LPR) * 16);
        if (c < 16 && c0 + c < N && row < M) *reinterpret_cast<uint4v*>(reinterpret_cast<char*>(a.y) + ((size_t)(c0 + c) * M + row) * ES) = v;
      }
    } else {
      for (int e = lane; e < 16 * 16 * WT; e += 64) {
        const int c = e / (16 * WT), r = e % (16 * WT);
        if (c0 + c < N && r0 + r < M) {
          const size_t at = (size_t)(c0 + c) * M + r0 + r;
          if (OUT32) reinterpret_cast<float*>(a.y)[at] = *reinterpret_cast<const float*>(stage_out + c * PITCH + r * ES);
          else reinterpret_cast<uint16_t*>(a.y)[at] = *reinterpret_cast<const uint16_t*>(stage_out + c * PITCH + r * ES);
        }
      }
    }
  };
  auto all_out = [&](auto out32_tag, auto edge_tag) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < WT; ++t) {
      block_out(t, out32_tag, edge_tag);
      __builtin_amdgcn_sched_barrier(0);      // (one block's results at a time out of the accumulation registers)
    }
    if (a.transposed) {
#pragma unroll
      for (int y = 0; y < WF; ++y) { block_out_transposed(y, out32_tag); __builtin_amdgcn_sched_barrier(0); }
    }
  };
  if (a.out_dtype == FTGEMM_F32) {
    if (edge) all_out(ftattn::yes{}, ftattn::yes{}); else all_out(ftattn::yes{}, ftattn::no{});
  } else {
    if (edge) all_out(ftattn::no{}, ftattn::yes{}); else all_out(ftattn::no{}, ftattn::no{});
  }

  if (FT) {
    __syncthreads();
    // fold of the results of each class against the first checksum product (eq. (15)).  The waves of a token range
    // divide its token blocks; a lane has the two classes whose sums it finds at its own place.  (With every wave forming the
    // verdicts of all blocks, this took 1.7 us of the 3.2 that follow the last product of the smallest tile; now 0.6.)
    auto total = [&](int t, int val, int n) __attribute__((always_inline)) -> float {
      float v = ex(t, val, 0);
#pragma unroll
      for (int f = 1; f < n; ++f) v += ex(t, val, f);
      return v;
    };
    float stat_max = 0.f;
    bool any = false;
#pragma unroll
    for (int u = 0; u < (WT + NWF - 1) / NWF; ++u) {
      const int in_range = wf + u * NWF;
      if (WT % NWF != 0 && in_range >= WT) break;
      const int b = WT * wt + in_range;
      float2v fold = ex_pair(b, 0, 0), mag = ex_pair(b, 1, 0);
      const float2v chk = ex_pair(b, 2, 0);
#pragma unroll
      for (int f = 1; f < NWF; ++f) { fold += ex_pair(b, 0, f); mag += ex_pair(b, 1, f); }
      const bool real = m0 + 16 * b + lq < M;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float R = chk[h] - fold[h], thr = a.tau_abs + a.tau_rel * mag[h];
        const bool d = real && (!(__builtin_fabsf(R) <= thr) || !finitef(R));
        any |= d;
        if (!d && real && thr > 0.f) stat_max = fmax2(stat_max, __builtin_fabsf(R) / thr);
      }
    }
    if (any) shared_n[0] = 1;
    const uint32_t stat = ftattn::wave_max_u32(as_u(stat_max));        // (not negative: ordered like its bits)
    if (lane == 63) shared_stat[wave] = as_f(stat);
    __syncthreads();
    if (shared_n[0]) {
      // ---- rare: the verdicts again, of all blocks of its token range by every wave, in the same order and so alike
      uint32_t det = 0u;
#pragma unroll
      for (int t = 0; t < WT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float R = ex(t, 8 + r, 0) - total(t, r, NWF);
          const float thr = a.tau_abs + a.tau_rel * total(t, 4 + r, NWF);
          if (row_of(t) < M && (!(__builtin_fabsf(R) <= thr) || !finitef(R))) det |= 1u << (4 * t + r);
        }
      // Locate with the second checksum, restore from the first, one token block after the
      // other.  The workgroup's run of the event ring is counted by the waves that log (one per token
      // range).  The results are in Y already: a restored one is stored over the faulty one.
      if (wf == 0 && lane < 32 && det) atomicAdd(&shared_n[1], __popc(det));
      wait_vmcnt<0>();
      __syncthreads();
      if (tid == 0) { shared_n[2] = (int)atomicAdd(a.cursor, (uint32_t)shared_n[1]); shared_n[3] = 0; }
      __syncthreads();
      // (the waves of a token range number its blocks from different ones, so each of these passes covers
      // all blocks; the second checksum products take the place of the magnitudes)
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        if (t < CB && check_wave) {
#pragma unroll
          for (int r = 0; r < 4; ++r) ex(t, 4 + r, 0) = sum32(sc[t][1][r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float sum2 = 0.f, big = -1.f;
          int l_big = -1;
#pragma unroll
          for (int y = 0; y < WF; ++y) {
            const int l = 2 * (WF * wf + y) + (lg >> 1);
            const float v = fold_value(y, t, r, edge);
            sum2 += (float)(l + 1) * v;
            const float m = finitef(v) ? __builtin_fabsf(v) : __builtin_inff();
            if (m > big) { big = m; l_big = l; } else if (m == big) { l_big = -1; }
          }
          const float pb = xchg32(big, lg >> 1);
          const int pl = (int)xchg32((float)l_big, lg >> 1);
          if (pb > big) { big = pb; l_big = pl; } else if (pb == big) { l_big = -1; }
          ex2(t, r, wf) = sum32(sum2); ex2(t, 4 + r, wf) = big; ex2(t, 8 + r, wf) = (float)l_big;
        }
      }
      __syncthreads();
      int lstar[WT];                      // located fold per class, one byte each; 0xff: none
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        lstar[t] = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float s2 = 0.f, b = -1.f;
          int lb = -1;
#pragma unroll
          for (int f = 0; f < NWF; ++f) {
            s2 += ex2(t, r, f);
            const float m = ex2(t, 4 + r, f);
            if (m > b) { b = m; lb = (int)ex2(t, 8 + r, f); } else if (m == b) { lb = -1; }
          }
          const float ratio = (ex(t, 4 + r, 0) - s2) / (ex(t, 8 + r, 0) - total(t, r, NWF));
          int ls = -1;
          if (finitef(ratio)) {
            const float c = __builtin_rintf(ratio) - 1.0f;
            if (c >= 0.f && c < (float)GFOLD) ls = (int)c;
          } else {
            ls = lb;            // residuals left the fp32 range: the fold of overwhelming size
          }
          if (!((det >> (4 * t + r)) & 1u) || (ls >= 0 && n0 + 8 * ls + 4 * (lg & 1) + r >= N)) ls = -1;
          lstar[t] |= (ls & 0xff) << (8 * r);
        }
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < WT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float rest = 0.f;
#pragma unroll
          for (int y = 0; y < WF; ++y)
            if (2 * (WF * wf + y) + (lg >> 1) != ((lstar[t] >> (8 * r)) & 0xff)) rest += fold_value(y, t, r, edge);
          ex2(t, r, wf) = sum32(rest);
        }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < WT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!((det >> (4 * t + r)) & 1u) || lane >= 32) continue;
          const int b8 = (lstar[t] >> (8 * r)) & 0xff, ls = b8 == 0xff ? -1 : b8;
          const int col = ls >= 0 ? n0 + 8 * ls + 4 * (lg & 1) + r : -1;
          const bool fix = a.correct && ls >= 0;
          const float chk1 = ex(t, 8 + r, 0);
          if (wf == 0) log_gemm_event(a, (uint32_t)shared_n[2] + (uint32_t)atomicAdd(&shared_n[3], 1), row_of(t), col, chk1 - total(t, r, NWF), fix ? 1 : 0);
          if (fix && ls >= 2 * WF * wf && ls < 2 * WF * (wf + 1)) {
            float rest = ex2(t, r, 0);
#pragma unroll
            for (int f = 1; f < NWF; ++f) rest += ex2(t, r, f);
            store_one(row_of(t), col, chk1 - rest);
          }
        }
    }
    if (tid == 0) {
      float s = shared_stat[0];
#pragma unroll
      for (int w = 1; w < T::NW; ++w) s = fmax2(s, shared_stat[w]);
      write_slot(a, logical, GSlot{(uint32_t)shared_n[2], shared_n[1], s});
    }
  } else if (tid == 0) {
    write_slot(a, logical, GSlot{0u, 0, 0.f});
  }
}

template <class T, bool FT, bool INJ, bool BF>
__global__ __launch_bounds__(T::NW * 64, T::PER_CU * T::NW / 4 > 8 / T::NW ? T::PER_CU * T::NW / 4 : 8 / T::NW) void ftgemm_main(const GArgs a0) {
  GArgs a = a0;
  // ---- workgroup -> problem of the batch, output tile.  Workgroup ids go round-robin over the 8 XCDs; each XCD gets a
  // contiguous range of tiles, and tiles are numbered in groups of 8 token tiles x all feature
  // tiles, feature-major inside a group, so that the workgroups an XCD runs together share
  // weight rows and token rows in its L2.
  int by, tm, tn, logical;
  if (a.k_lower) {
    // tiles of unequal length (tile t has t + 1 times as many steps as tile 0): longest first
    const ftattn::RowTile rt = ftattn::causal_row_tile((int)blockIdx.x, (int)gridDim.x, a.tiles, a.head_group);
    by = rt.bh; tm = logical = rt.ti; tn = 0;
  } else {
    const int id = blockIdx.x, total = gridDim.x, xcd = id & 7, slot = id >> 3, qn = total >> 3, rn = total & 7;
    logical = xcd * qn + (xcd < rn ? xcd : rn) + slot;
    if (a.skip_upper) {
      by = logical / a.tiles;
      logical -= by * a.tiles;
      lower_tile(logical, T::BM, tm, tn);
    } else {
      by = blockIdx.y;
      constexpr int GM = 8;
      const int gsz = GM * a.Tn, g = logical / gsz, first = g * GM;
      const int gm = a.Tm - first < GM ? a.Tm - first : GM;
      const int in_g = logical - g * gsz;
      tm = first + in_g % gm;
      tn = in_g / gm;
    }
  }
  // (divisions leave the vector unit; everything here is the same in all lanes)
  by = __builtin_amdgcn_readfirstlane(by); tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn); logical = __builtin_amdgcn_readfirstlane(logical);
  {
    a.x += by * a0.bs_x; a.w += by * a0.bs_w; a.wc += by * a0.bs_wc;
    a.y = reinterpret_cast<char*>(a0.y) + by * a0.bs_y_bytes;
    a.events += by * a0.bs_events; a.cursor += by; a.slots += by * a0.bs_slots;
  }
  constexpr int WT = T::WT, WF = T::WF, NST = T::NST, NWF = T::NWF, CB = T::CB;
  constexpr int BK = T::BK, ROWB = T::ROWB, CPR = T::CPR;
  constexpr int STAGE = T::template bytes<FT>(), NLOAD = T::template nload<FT>();
  constexpr int NKS = BK / 32;           // k-steps of 32 per stage
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wt = wave / NWF, wf = wave % NWF;         // the wave's place along tokens and features
  const int M = a.M, N = a.N, K = a.K;
  const int m0 = tm * T::BM, n0 = tn * GBN;
  int nkb = (K + BK - 1) / BK;
  const int krem = K - (nkb - 1) * BK;      // columns of the last K step (BK unless K is ragged; K is a multiple of 8)
  int kb_ragged = krem < BK ? nkb - 1 : -1;
  if (a.k_lower) { const int lim = (m0 + T::BM + BK - 1) / BK; nkb = lim < nkb ? lim : nkb; }
  int kb0 = 0;                              // first K step of this workgroup's share
  if (a.parts > 1) {
    kb0 = nkb * (int)blockIdx.z / a.parts;  // (at most 2^16 steps)
    nkb = nkb * ((int)blockIdx.z + 1) / a.parts - kb0;
    kb_ragged -= kb0;
  }
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

  // ---- per-lane source offsets of this wave's load instructions.  Piece p of an operand tile is its
  // rows PR*p .. PR*p + PR-1; wave w takes pieces w, w + NW, ...  Rows beyond the matrix are clamped to its
  // last row (their results are never used).  The chunk a lane fetches is the same in all its pieces.
  auto swz = [](int row) __attribute__((always_inline)) -> int { return (row >> 1) & 7; };
  auto piece_of = [&](int i) __attribute__((always_inline)) -> int {
    return i < T::XW ? (wave + T::NW * i) % T::XP : i < T::XW + T::WW ? wave + T::NW * (i - T::XW) : wave % T::CP;
  };
  const int chunk = (lane % CPR) ^ swz(T::PR * wave + lane / CPR);
  uint32_t off[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int rows_left = i < T::XW ? M - m0 : i < T::XW + T::WW ? N - n0 : GCK;
    int r = T::PR * piece_of(i) + lane / CPR;
    if (r > rows_left - 1) r = rows_left - 1;
    off[i] = ((uint32_t)r * (uint32_t)K + (uint32_t)chunk * 8u) * 2u;
  }
  const uint16_t* xb = a.x + (size_t)m0 * K + kb0 * BK;
  const uint16_t* wb = a.w + (size_t)n0 * K + kb0 * BK;
  const uint16_t* cb = (FT ? a.wc + (size_t)tn * GCK * K : a.w) + kb0 * BK;
  // Steps are requested in their order: the sources move on by one step behind each (next_step), and a piece's place
  // is its stage's base plus what does not change over the steps.
  const uint32_t wave_at = smem_base + (uint32_t)wave * 1024u;
  const uint32_t x_at = T::XP % T::NW ? (uint32_t)(wave % T::XP - wave) * 1024u : 0u;      // (pieces that are fetched twice)
  const uint32_t c_at = T::CP % T::NW ? (uint32_t)(wave % T::CP - wave) * 1024u : 0u;
  auto piece_lds = [&](int i, uint32_t stage) __attribute__((always_inline)) -> uint32_t {
    if (i < T::XW) return wave_at + stage + x_at + (uint32_t)(T::NW * i * 1024);
    if (i < T::XW + T::WW) return wave_at + stage + (uint32_t)((T::XP + T::NW * (i - T::XW)) * 1024);
    return wave_at + stage + c_at + (uint32_t)((T::XP + T::WP) * 1024);
  };
  auto issue_piece = [&](int i, uint32_t stage) __attribute__((always_inline)) {
    gload_lds16_off(i < T::XW ? xb : i < T::XW + T::WW ? wb : cb, off[i], piece_lds(i, stage));
  };
  auto next_step = [&]() __attribute__((always_inline)) { xb += BK; wb += BK; cb += BK; };
  // the last K step of a ragged K: the chunks beyond column K are filled with zeros instead
  // (a wave without a piece of the checksum rows has one load less; fetching another wave's piece once more to keep the
  // counts alike made the steps of the 64-token tile, whose 48 pieces include 4 such, 10 % longer where rows are not
  // multiples of a cache line: 1733 x 539 x 6344)
  const bool has_c = FT && (!T::C_SPARE || wave < T::CP);
  auto issue_ragged = [&](uint32_t stage) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      if (i == T::XW + T::WW && !has_c) continue;
      if (chunk * 8 < krem) issue_piece(i, stage);
      else *reinterpret_cast<__attribute__((address_space(3))) half8*>((uintptr_t)(piece_lds(i, stage) + 16u * lane)) = (half8)(_Float16)0.f;
    }
  };

  // The token blocks of a wave are numbered from the first one whose checksum products it forms (its
  // share of the checksum work, counted round the WT blocks of its token range), so that the share has
  // fixed register indices in every wave.
  const int rot = wf * CB % WT;
  const bool check_wave = FT && wf * CB < WT;
  auto block_of = [&](int t) __attribute__((always_inline)) -> int { return (t + rot) % WT; };

  float4v acc[WF][WT], sc[CB][2];         // sc: the products of the first and of the second checksum rows
#pragma unroll
  for (int f = 0; f < WF; ++f)
#pragma unroll
    for (int t = 0; t < WT; ++t) acc[f][t] = (float4v)0.f;
#pragma unroll
  for (int t = 0; t < CB; ++t) sc[t][0] = sc[t][1] = (float4v)0.f;

  // operand addresses inside a stage: row 16*y + lq of a tile, chunk (4*ks + lg) XOR-ed with a function of the row.
  // Stages start at multiples of 1 KB, so the chunk bits can be XOR-ed into the complete address.
  const uint32_t lane_at = (uint32_t)(lq * ROWB + ((lg ^ swz(lq)) << 4));
  const uint32_t wrow = smem_base + (uint32_t)((T::BM + 16 * WF * wf) * ROWB) + lane_at;
  const uint32_t crow = smem_base + (uint32_t)((T::BM + T::BF) * ROWB) + lane_at;
  uint32_t xrow[WT];
#pragma unroll
  for (int t = 0; t < WT; ++t) xrow[t] = smem_base + (uint32_t)(16 * (WT * wt + block_of(t)) * ROWB) + lane_at;
  auto lds_rd = [](uint32_t addr) __attribute__((always_inline)) -> half8 {
    return *reinterpret_cast<const __attribute__((address_space(3))) half8*>((uintptr_t)addr);
  };
  auto mma = [&](const half8& av, const half8& bv, float4v& d) __attribute__((always_inline)) {
    if (BF) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, av), __builtin_bit_cast(bf8, bv), d, 0, 0, 0);
    else d = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, d, 0, 0, 0);
  };
  // Operand registers: the token operands of two k-steps (one in use, one being read), a ring of four
  // weight operands (a row of WT products uses one; the one three rows ahead is being read), the checksum
  // operands of the k-step in progress.
  half8 xr[2][WT], wr[4], cr[2];
  constexpr int AHEAD = 3;
  static_assert(WF >= AHEAD + 1 && WT >= 2 && (NKS * WF) % 4 == 0 && NKS % 2 == 0, "operand rings");
  auto read_x = [&](int ks, int t, uint32_t stage) __attribute__((always_inline)) {
    xr[ks & 1][t] = lds_rd((xrow[t] + stage) ^ (uint32_t)(ks << 6));
  };
  auto read_w = [&](int p, uint32_t stage) __attribute__((always_inline)) {       // p: k-step * WF + row
    wr[p & 3] = lds_rd(((wrow + stage) ^ (uint32_t)(p / WF << 6)) + p % WF * 16 * ROWB);
  };
  auto read_c = [&](int ks, int i, uint32_t stage) __attribute__((always_inline)) {
    cr[i] = lds_rd(((crow + stage) ^ (uint32_t)(ks << 6)) + i * 16 * ROWB);
  };
  // keeps `n` LDS reads behind the product they were written after
  auto pin = [](int n) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (n == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    else if (n == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    else if (n == 3) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
  };
  auto wait_lds = []() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0xC07F); };

  // ---- prologue: the first NST stages are requested, the first one's first operands read
#pragma unroll
  for (int st = 0; st < NST; ++st)
    if (st < nkb) {
      if (st == kb_ragged) issue_ragged((uint32_t)(st * STAGE));
      else {
#pragma unroll
        for (int i = 0; i < NLOAD; ++i)
          if (i < T::XW + T::WW || has_c) issue_piece(i, (uint32_t)(st * STAGE));
      }
      next_step();
    }
  if (nkb < NST) wait_vmcnt<0>();
  else if (has_c) wait_vmcnt<(NST - 1) * NLOAD>();
  else wait_vmcnt<(NST - 1) * (T::XW + T::WW)>();
  wait_lds();
  phase_barrier();
  const int nfull = kb_ragged >= 0 && kb_ragged < nkb ? nkb - 1 : nkb;      // steps that are requested in the stream
  auto contract = [&](auto chk_tag, auto c_tag) __attribute__((always_inline)) {
    constexpr bool CHK = decltype(chk_tag)::value;
    constexpr int NL = T::XW + T::WW + (decltype(c_tag)::value ? 1 : 0);      // loads per step of this wave
    constexpr int NCHK = CHK ? 2 * CB : 0;
    uint32_t stage = 0;                      // base of the stage in use
    // Row y of k-step ks: its products, and the LDS reads behind them.  `tail`: the last AHEAD rows of a
    // stage, behind its barrier, which read the next stage's first operands (after the last stage: what the
    // ring still holds, in bounds and unused) and request (LD) the stage that takes this one's place.
    auto row_step = [&](auto row_tag, uint32_t stage, uint32_t next, auto ld_tag) __attribute__((always_inline)) {
      constexpr bool LD = decltype(ld_tag)::value;
      constexpr int ks = decltype(row_tag)::value / WF, y = decltype(row_tag)::value % WF;
      constexpr bool last = ks == NKS - 1, tail = last && y >= WF - AHEAD;
      constexpr int np = WT + (y == WF - 1 ? NCHK : 0);                   // products of this row
      constexpr int TAILP = AHEAD * WT + NCHK;                        // ... of all tail rows
      // token operands of the next k-step: read over the rows of this one, or over the tail
      constexpr int rows = last ? AHEAD : WF, r = last ? y - (WF - AHEAD) : y;
      constexpr int x0 = last && !tail ? 0 : WT * r / rows, x1 = last && !tail ? 0 : WT * (r + 1) / rows;
      int nread[WT + 2 * CB];
#pragma unroll
      for (int m = 0; m < np; ++m) {
        if (m < WT) mma(wr[(ks * WF + y) & 3], xr[ks & 1][m], acc[y][m]);
        else mma(cr[(m - WT) / CB], xr[ks & 1][(m - WT) % CB], sc[(m - WT) % CB][(m - WT) / CB]);
        int n = 0;
        const int p = ks * WF + y + AHEAD;
        if (m == 0 && (NST > 1 || p < NKS * WF)) {
          read_w(p % (NKS * WF), p < NKS * WF ? stage : next);
          ++n;
        }
        if (CHK && y == 0 && m == 1) { read_c(ks, 0, stage); read_c(ks, 1, stage); n += 2; }     // (ahead of the barrier of the last k-step)
        // one token operand behind every product but the first
        if (m >= 1 && x0 + m - 1 < x1 && (NST > 1 || !last)) { read_x((ks + 1) % NKS, x0 + m - 1, last ? next : stage); ++n; }
        nread[m] = n;
        if (LD && tail) {
          const int q = (y - (WF - AHEAD)) * WT + m;
#pragma unroll
          for (int i = NL * q / TAILP; i < NL * (q + 1) / TAILP; ++i) issue_piece(i, stage);
        }
      }
#pragma unroll
      for (int m = 0; m < np; ++m) pin(nread[m]);
    };
    auto first_operands = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < WT; ++t) read_x(0, t, 0u);
#pragma unroll
      for (int p = 0; p < AHEAD; ++p) read_w(p, 0u);
    };
    auto stage_step = [&](int kb, auto ld_tag) __attribute__((always_inline)) {
      constexpr bool LD = decltype(ld_tag)::value;
      const uint32_t next = stage == (uint32_t)((NST - 1) * STAGE) ? 0u : stage + (uint32_t)STAGE;
      for_each_index<NKS * WF - AHEAD>([&](auto row) __attribute__((always_inline)) { row_step(row, stage, next, ld_tag); });
      wait_lds();                            // the operands of the last rows are in registers: this wave is done with the stage
      // the next stage has landed; up to NST-2 younger ones may be in flight
      if constexpr (NST > 1) {
        if (LD || kb + NST - 1 < nkb) wait_vmcnt<(NST - 2) * NL>();
        else wait_vmcnt<0>();
      }
      phase_barrier();                       // everyone's pieces of the next stage have landed, and everyone is done with this one
      if (!LD && kb + NST < nkb) issue_ragged(stage);
      for_each_index<AHEAD>([&](auto row) __attribute__((always_inline)) {
        row_step(std::integral_constant<int, NKS * WF - AHEAD + decltype(row)::value>{}, stage, next, ld_tag);
      });
      if (LD) next_step();
      stage = next;
      if constexpr (NST == 1) {
        if (kb + 1 < nkb) {                  // the one stage again, once everyone's pieces have landed
          wait_vmcnt<0>();
          wait_lds();
          phase_barrier();
          first_operands();
        }
      }
    };
    first_operands();
    int kb = 0;
    for (; kb + NST < nfull; ++kb) stage_step(kb, ftattn::yes{});
    for (; kb < nkb; ++kb) stage_step(kb, ftattn::no{});
  };
  auto contract_as = [&](auto chk_tag) __attribute__((always_inline)) {
    if constexpr (!FT) contract(chk_tag, ftattn::no{});
    else if constexpr (!T::C_SPARE) contract(chk_tag, ftattn::yes{});
    else if (has_c) contract(chk_tag, ftattn::yes{});
    else contract(chk_tag, ftattn::no{});
  };
  if (FT && WT < NWF) {
    if (check_wave) contract_as(ftattn::yes{}); else contract_as(ftattn::no{});
  } else if (FT) {
    contract_as(ftattn::yes{});
  } else {
    contract_as(ftattn::no{});
  }

  wait_lds();
  phase_barrier();                         // the ring is free
  if (a.parts > 1) {
    // this workgroup's share of the contraction, for ftgemm_finish
    float4v* out = a.ws + ((size_t)blockIdx.z * a.ws_tokens + m0 / 16 + WT * wt) * a.Tn * WS_BLOCKS * 64 + lane;
    for_each_index<WT>([&](auto t) __attribute__((always_inline)) {
      float4v* at = out + ((size_t)block_of(t) * a.Tn + tn) * WS_BLOCKS * 64;
#pragma unroll
      for (int y = 0; y < WF; ++y) at[(WF * wf + y) * 64] = acc[y][t];
      if (t < CB && check_wave) { at[16 * 64] = sc[t < CB ? t : 0][0]; at[17 * 64] = sc[t < CB ? t : 0][1]; }
    });
    return;
  }
  finish_tile<T, FT, INJ, BF>(a, smem, acc, sc, m0, n0, logical);
}

// Sums up the shares of the K dimension (in their order) and finishes 16 tokens x 256 features per
// workgroup: the split contraction of ftgemm_main, whose workgroups would each have a whole tile's shares
// to read if the last of them did this.
template <bool FT, bool BF>
__global__ __launch_bounds__(256) void ftgemm_finish(const GArgs a) {
  using T = TileFinish;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tm = blockIdx.x / a.Tn, tn = blockIdx.x % a.Tn, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float4v acc[T::WF][T::WT], sc[T::CB][2];
#pragma unroll
  for (int y = 0; y < T::WF; ++y) acc[y][0] = (float4v)0.f;
  sc[0][0] = sc[0][1] = (float4v)0.f;
  const float4v* in = a.ws + ((size_t)tm * a.Tn + tn) * WS_BLOCKS * 64 + lane;
  const size_t step = (size_t)a.ws_tokens * a.Tn * WS_BLOCKS * 64;
  // up to eight shares are requested before the first is added: what this kernel takes is the latency of its loads
  auto add = [&](const int first, auto n_tag) __attribute__((always_inline)) {
    constexpr int NP = decltype(n_tag)::value;
    float4v x[NP][T::WF], c[NP][2];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const float4v* at = in + (first + i) * step;
#pragma unroll
      for (int y = 0; y < T::WF; ++y) x[i][y] = at[(T::WF * wave + y) * 64];
      if (FT && wave == 0) { c[i][0] = at[16 * 64]; c[i][1] = at[17 * 64]; }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
#pragma unroll
      for (int y = 0; y < T::WF; ++y) acc[y][0] += x[i][y];
      if (FT && wave == 0) { sc[0][0] += c[i][0]; sc[0][1] += c[i][1]; }
    }
  };
  int p = 0;
  for (; p + 8 <= a.parts; p += 8) add(p, std::integral_constant<int, 8>{});
  if (p + 4 <= a.parts) { add(p, std::integral_constant<int, 4>{}); p += 4; }
  for (; p < a.parts; ++p) add(p, std::integral_constant<int, 1>{});
  finish_tile<T, FT, false, BF>(a, smem, acc, sc, tm * T::BM, tn * GBN, blockIdx.x);
}

typedef void (*gemm_fn)(const GArgs);
enum TileId { TILE_WIDE, TILE_HALF, TILE_QUARTER, TILE_STRIP, TILE_NARROW, TILE_SLIM, TILE_NARROW2, TILE_SLIM2, TILE_LOW, N_TILES };
struct TileInfo { int bm, threads, per_cu, lds[2]; };       // lds: dynamic LDS bytes without / with the checksum rows

// kernel of one tile shape, instantiated per type (ftgemm_f16.hip, ftgemm_bf16.hip); the fault
// injector exists for TILE_QUARTER only
gemm_fn tile_kernel_f16(int tile, bool ft, bool inject);
gemm_fn tile_kernel_bf16(int tile, bool ft, bool inject);
gemm_fn finish_kernel_f16(bool ft);
gemm_fn finish_kernel_bf16(bool ft);
template <bool BF> gemm_fn tile_kernel_of(int tile, bool ft, bool inject) {
  if (inject) return ft ? ftgemm_main<TileQuarter, true, true, BF> : ftgemm_main<TileQuarter, false, true, BF>;
  switch (tile) {
    case TILE_WIDE: return ft ? ftgemm_main<TileWide, true, false, BF> : ftgemm_main<TileWide, false, false, BF>;
    case TILE_HALF: return ft ? ftgemm_main<TileHalf, true, false, BF> : ftgemm_main<TileHalf, false, false, BF>;
    case TILE_QUARTER: return ft ? ftgemm_main<TileQuarter, true, false, BF> : ftgemm_main<TileQuarter, false, false, BF>;
    case TILE_STRIP: return ft ? ftgemm_main<TileStrip, true, false, BF> : ftgemm_main<TileStrip, false, false, BF>;
    case TILE_NARROW2: return ft ? ftgemm_main<TileNarrow2, true, false, BF> : ftgemm_main<TileNarrow2, false, false, BF>;
    case TILE_SLIM2: return ft ? ftgemm_main<TileSlim2, true, false, BF> : ftgemm_main<TileSlim2, false, false, BF>;
    case TILE_LOW: return ft ? ftgemm_main<TileLow, true, false, BF> : ftgemm_main<TileLow, false, false, BF>;
    case TILE_NARROW: return ft ? ftgemm_main<TileNarrow, true, false, BF> : ftgemm_main<TileNarrow, false, false, BF>;
    default: return ft ? ftgemm_main<TileSlim, true, false, BF> : ftgemm_main<TileSlim, false, false, BF>;
  }
}

// Launch helpers (ftgemm.hip), for other host code of the library that runs the same protected
// product on buffers of its own (the decoupled attention baseline).  None of them allocates or
// synchronises.
hipError_t gemm_launch_encode_w(const uint16_t* w, uint16_t* wc, int n, int k, bool bf16, hipStream_t st,
                                int batch = 1, long long bs_w = 0, long long bs_wc = 0);
// How a product is run: its tile shape, and over how many workgroups a tile's K dimension is split.
struct GPlan { int tile, parts; };
GPlan gemm_plan(long long m, long long n, long long k, int batch, bool inject, bool may_split);
hipError_t gemm_allow_lds(GPlan plan, bool ft, bool bf16);       // once, before the launches of a plan
int gemm_slots(long long m, long long n, GPlan plan, bool skip_upper = false);      // report slots of one problem
size_t gemm_workspace(long long m, long long n, GPlan plan);    // bytes of GArgs::ws (0: not split)
hipError_t gemm_launch(GArgs a, bool ft, bool inject, bool bf16, GPlan plan, hipStream_t st, int batch = 1);
// What the slots of one call (host copies) say: the events logged and the largest passing statistic.
struct GStats { long long events; float stat; };
GStats gemm_stats(const GSlot* slots, int n_slots);
// Event ring of at least max_events entries: a power of two.
inline uint32_t ring_size(int max_events) { uint32_t n = 1; while (n < (uint32_t)max_events) n <<= 1; return n; }
// The events of one call out of the ring: at most max_events.  Where a call logs more than the ring holds, each entry
// is one of those that were written there, whichever workgroup's store came last.
hipError_t gemm_fetch_events(const GSlot* slots, int n_slots, const ftgemm_event* ring, uint32_t ring_n, int max_events,
                             std::vector<ftgemm_event>& out);

}  // namespace ftgemm
