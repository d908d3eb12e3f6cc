// The decoupled, operation-level fault-tolerant attention of Section 3.1 (the comparison system of
// Section 4.1): ABFT-GEMM I -> DMR row-softmax -> ABFT-GEMM II, with S and P in device memory between
// the kernels.  The C ABI of include/ftdecoupled.h.  The two GEMMs are the library's strided-ABFT
// GEMM kernel (ftgemm_main.h) on buffers of this context, one launch for all heads (with a fault list one
// per head); the softmax kernels and the kernel that prepares both products are here.
#include "ftdecoupled.h"
#include "ftgemm_main.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

namespace ftdec {

using ftattn::as_f;
using ftattn::as_u;

struct SFault { int32_t key, col, bit, stage; };   // key = bh * seq + row; sorted by key

struct SArgs {
  const float* S;          // [BH][N][N]
  _Float16* P;             // [BH][N][Np]
  int32_t N, Np, H, causal;
  float scale_log2, eps;
  int32_t use_lds;         // the row is staged in LDS (it fits), else re-read from memory
  const SFault* faults;
  int32_t n_faults;
  ftdec_event* events;
  int32_t* ev_count;
  int32_t max_events;
  unsigned long long* retried;
};

__device__ __forceinline__ float opaque(float x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float flip(float x, int bit) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) ^ (1u << bit)); }

__device__ __forceinline__ void log_softmax_event(const SArgs& a, int bh, int stage, int row, int col) {
  const int idx = atomicAdd(a.ev_count, 1);
  if (idx < a.max_events) {
    ftdec_event e;
    e.b = bh / a.H; e.h = bh % a.H; e.stage = stage; e.row = row; e.col = col; e.action = 1;
    a.events[idx] = e;
  }
}

// block-wide reductions over 256 threads (4 waves); every thread gets the result
__device__ __forceinline__ float block_max(float v, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = __builtin_fmaxf(v, __shfl_xor(v, off));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
}
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}
__device__ __forceinline__ int block_or(int v, int* red) {
  v = __builtin_amdgcn_ballot_w64(v != 0) != 0ull ? 1 : 0;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] | red[1] | red[2] | red[3];
}

// Row softmax by dual modular redundancy (eq. (11), (12)).  One workgroup per (row, head).
//   evaluation a, evaluation b: maximum and exponentials, the second on values the compiler cannot
//   merge with the first; |e_a - e_b| < eps element by element, DMR(e) = (e_a + e_b) / 2;
//   P = DMR(e) / rowsum(DMR(e)); |rowsum(P) - 1| < eps.
// A row that fails either test is evaluated again; injected faults hit the first attempt only (a
// soft error does not repeat).  FT == false: one evaluation, no test.
template <bool FT, bool INJ>
__global__ __launch_bounds__(256) void ftdec_softmax(const SArgs a) {
  extern __shared__ __attribute__((aligned(16))) float rowbuf[];
  __shared__ float red[4];
  __shared__ int redi[4];
  const int row = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
  const int N = a.N, nvalid = a.causal ? row + 1 : N;
  const float* src = a.S + ((size_t)bh * N + row) * N;
  _Float16* dst = a.P + ((size_t)bh * N + row) * a.Np;
  if (a.use_lds) {
    for (int j = tid; j < nvalid; j += 256) rowbuf[j] = src[j];
    __syncthreads();
    src = rowbuf;
  }
  // faults of this row: [f0, f1)
  int f0 = 0, f1 = 0;
  if (INJ) {
    const int key = bh * N + row;
    int lo = 0, hi = a.n_faults;
    while (lo < hi) { const int mid = (lo + hi) >> 1; if (a.faults[mid].key < key) lo = mid + 1; else hi = mid; }
    f0 = lo;
    while (lo < a.n_faults && a.faults[lo].key == key) ++lo;
    f1 = lo;
  }
  const float sl2 = a.scale_log2;
  for (int attempt = 0; attempt < 3; ++attempt) {
    // ---- maximum, twice
    float ma = -__builtin_inff(), mb = -__builtin_inff();
    for (int j = tid; j < nvalid; j += 256) {
      const float s = src[j];
      ma = __builtin_fmaxf(ma, s);
      if (FT) mb = __builtin_fmaxf(mb, opaque(s));
    }
    ma = block_max(ma, red);
    if (FT) mb = block_max(mb, red);
    const float na = -ma * sl2, nb = -mb * sl2;
    // ---- exponentials, twice; eq. (11)
    float sum = 0.f;
    int bad = 0;
    for (int j = tid; j < nvalid; j += 256) {
      const float s = src[j];
      float ea = ex2(__builtin_fmaf(s, sl2, na));
      if (INJ && attempt == 0)
        for (int f = f0; f < f1; ++f)
          if (a.faults[f].stage == FTDEC_ST_EXP && a.faults[f].col == j) ea = flip(ea, a.faults[f].bit);
      if (FT) {
        const float eb = ex2(__builtin_fmaf(opaque(s), sl2, nb));
        if (!(__builtin_fabsf(ea - eb) < a.eps)) {
          bad = 1;
          log_softmax_event(a, bh, FTDEC_ST_EXP, row, j);
        }
        sum += 0.5f * (ea + eb);
      } else {
        sum += ea;
      }
    }
    if (FT && block_or(bad, redi)) {
      if (tid == 0) atomicAdd(a.retried, 1ull);
      continue;
    }
    const float l = block_sum(sum, red);
    const float inv = 1.0f / l;
    // ---- normalised weights; eq. (12)
    float psum = 0.f;
    // (causal: GEMM II stops at the last query of the row's 256-query tile; the weights beyond are never read)
    const int jend = a.causal && (row / 256 + 1) * 256 < a.Np ? (row / 256 + 1) * 256 : a.Np;
    for (int j = tid; j < jend; j += 256) {
      float p = 0.f;
      if (j < nvalid) {
        const float s = src[j];
        float ea = ex2(__builtin_fmaf(s, sl2, na));
        if (INJ && attempt == 0)
          for (int f = f0; f < f1; ++f)
            if (a.faults[f].stage == FTDEC_ST_EXP && a.faults[f].col == j) ea = flip(ea, a.faults[f].bit);
        const float e = FT ? 0.5f * (ea + ex2(__builtin_fmaf(opaque(s), sl2, nb))) : ea;
        p = opaque(e * inv);            // (one value for the sum and the store, as below)
        if (INJ && attempt == 0)
          for (int f = f0; f < f1; ++f)
            if (a.faults[f].stage == FTDEC_ST_PNORM && a.faults[f].col == j) p = flip(p, a.faults[f].bit);
        psum += p;
      }
      dst[j] = (_Float16)p;
    }
    if (!FT) break;
    psum = block_sum(psum, red);
    if (__builtin_fabsf(psum - 1.0f) < a.eps) break;
    if (tid == 0) {
      log_softmax_event(a, bh, FTDEC_ST_PNORM, row, -1);
      atomicAdd(a.retried, 1ull);
    }
  }
}

// The same for rows of at most 256 * CH scores: a wave per row, four rows per workgroup, and the row in
// registers from the one read of S to the one write of P.  Lane l holds the scores 256 c + 4 l .. + 3
// of chunk c; chunks beyond the row's last valid score are skipped (wave-uniform), so a causal row
// pays for its own length only.  S has rows of N floats, 16 bytes at a time from any multiple of 4 bytes.
// Bound: memory (S once, P once; 268 + 151 MB for the lower half of 32 x 2048 x 2048, at 4.5 TB/s).  There a workgroup
// per row with eight barriers and four passes over LDS took 232 us, a wave per row whose loads waited for one another
// and whose reductions went through LDS 109, this takes 94.  Rows beyond 4096
// scores do not fit a wave's registers and keep the workgroup-per-row kernel.
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

template <int I> struct index_t { static constexpr int value = I; };

// op over the 64 lanes, in every lane: register moves within rows of 16 lanes, then between rows.  (As six LDS permutes, each
// waiting for the one before, four of these were 3100 cycles of a row's time.)
template <class F> __device__ __forceinline__ float wave_reduce(float v, const F& op) {
  auto moved = [&](auto ctrl) __attribute__((always_inline)) -> float {
    return as_f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)as_u(v), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v = op(v, moved(index_t<0xB1>{}));         // quads: 1 0 3 2, 2 3 0 1
  v = op(v, moved(index_t<0x4E>{}));
  v = op(v, moved(index_t<0x141>{}));        // mirrored in 8, in 16 lanes
  v = op(v, moved(index_t<0x140>{}));
  const auto r = __builtin_amdgcn_permlane16_swap(as_u(v), as_u(v), false, false);
  v = op(as_f(r[0]), as_f(r[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(as_u(v), as_u(v), false, false);
  return op(as_f(q[0]), as_f(q[1]));
}
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float x, float y) { return __builtin_fmaxf(x, y); }); }
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, [](float x, float y) { return x + y; }); }

// f(0) .. f(E - 1) with the index as a constant from the start.  (Loops over the registers of a row are
// unrolled only after the row has become one wide vector, which is then copied whole around every load.)
template <int E, int I = 0, class F> __device__ __forceinline__ void each(const F& f) {
  if constexpr (I < E) {
    f(index_t<I>{});
    each<E, I + 1>(f);
  }
}

// (Waves per SIMD: the most whose registers hold a row, but for rows of more than 2048 scores with their second evaluations, where four waves
// spill 5 values and three none: with a causal mask four are the faster ones, without it three: 1 x 4 x 4096 x 64 causal 144.2 and 146.5 us for the
// whole pass, 1 x 3 x 2500 x 64 causal 66.6 and 67.3, 1 x 2 x 4001 x 64 140.2 and 137.7, 1 x 7 x 2900 x 128 221.9 and 219.6.)
template <bool FT, bool INJ, int CH>
__global__ __launch_bounds__(256, INJ ? 1 : CH <= 4 ? 8 : CH == 8 ? 7 : 4) void ftdec_softmax_wave(const SArgs a) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the heads whose scores were written last come first: they are still in the memory-side cache; 2 x 16 x 2048 x 128 without a
  // mask 437 -> 425 us)
  const int N = a.N, row = blockIdx.x * 4 + wave, bh = gridDim.y - 1 - blockIdx.y;
  if (row >= N) return;
  const int nvalid = a.causal ? row + 1 : N;
  const float* src = a.S + ((size_t)bh * N + row) * N + 4 * lane;
  _Float16* dst = a.P + ((size_t)bh * N + row) * a.Np + 4 * lane;
  int f0 = 0, f1 = 0;             // faults of this row: [f0, f1)
  if (INJ) {
    const int key = bh * N + row;
    int lo = 0, hi = a.n_faults;
    while (lo < hi) { const int mid = (lo + hi) >> 1; if (a.faults[mid].key < key) lo = mid + 1; else hi = mid; }
    f0 = lo;
    while (lo < a.n_faults && a.faults[lo].key == key) ++lo;
    f1 = lo;
  }
  const float sl2 = a.scale_log2;
  // (causal: GEMM II stops at the last query of the row's 256-query tile; the weights beyond are never read)
  const int jend = a.causal && (row / 256 + 1) * 256 < a.Np ? (row / 256 + 1) * 256 : a.Np;
  for (int attempt = 0; attempt < 3; ++attempt) {
    float4u s[CH];            // (chunks beyond the row's last valid score are never written, nor read)
    // the lane's scores of chunk c are valid below left - 256 c (formed here: the masks of all chunks would
    // otherwise be kept in scalar registers across the attempts, more than there are)
    int left = nvalid - 4 * lane;
    asm volatile("" : "+v"(left));
    // the first attempt's faults (a soft error does not repeat)
    auto inject = [&](const int stage, const int col, float v) __attribute__((always_inline)) -> float {
      if (INJ && attempt == 0)
        for (int f = f0; f < f1; ++f)
          if (a.faults[f].stage == stage && a.faults[f].col == col) v = flip(v, a.faults[f].bit);
      return v;
    };
    // ---- the row, and its maximum, twice
    // All loads first, in registers that stay where they are: with the choice between a whole chunk and the last
    // one made around each load, its values were moved together behind it, and every load waited for the one before.
    each<CH>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = decltype(ci)::value;
      // (up to three scores beyond the last valid one are read with it, and not used: S ends in 16 bytes more)
      if (256 * c < nvalid && left > 256 * c) s[c] = *reinterpret_cast<const float4u*>(src + 256 * c);
    });
    each<CH>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = decltype(ci)::value;
      if (256 * c < nvalid && 256 * c + 256 > nvalid)
        each<4>([&](auto xi) __attribute__((always_inline)) {
          constexpr int x = decltype(xi)::value;
          s[c][x] = left > 256 * c + x ? s[c][x] : -__builtin_inff();
        });
    });
    // The second evaluations are made on the registers of the first, renewed: the compiler cannot merge them, and keeps
    // no copy for it.
    auto renew = [&](float4u& v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); };
    float ma = -__builtin_inff(), mb = -__builtin_inff();
    auto row_max = [&](float& m) __attribute__((always_inline)) {
      each<CH>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        if (256 * c < nvalid) each<4>([&](auto xi) __attribute__((always_inline)) { m = __builtin_fmaxf(m, s[c][decltype(xi)::value]); });
      });
    };
    row_max(ma);
    if (FT) {
      each<CH>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        if (256 * c < nvalid) renew(s[c]);
      });
      row_max(mb);
    }
    ma = wave_max(ma);
    if (FT) mb = wave_max(mb);
    const float na = -ma * sl2, nb = -mb * sl2;
    // ---- exponentials, twice; eq. (11).  s becomes DMR(e): zero, and equal, beyond the last valid score
    // (unless no score of the row is a number, and then the valid ones fail as well)
    float sum = 0.f;
    uint32_t bad[(CH + 7) / 8] = {};        // a bit per score of the lane
    each<CH>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = decltype(ci)::value;
      if (256 * c < nvalid) {
        float4u e;
        float d[4];
        each<4>([&](auto xi) __attribute__((always_inline)) {
          constexpr int x = decltype(xi)::value;
          e[x] = inject(FTDEC_ST_EXP, 256 * c + 4 * lane + x, ex2(__builtin_fmaf(s[c][x], sl2, na)));
        });
        if (FT) {
          renew(s[c]);
          each<4>([&](auto xi) __attribute__((always_inline)) {
            constexpr int x = decltype(xi)::value;
            const float eb = ex2(__builtin_fmaf(s[c][x], sl2, nb));
            d[x] = e[x] - eb;
            e[x] = 0.5f * (e[x] + eb);
          });
          // the largest difference of the four (a NaN stays one); which ones it was only where one is too large
          float m;
          asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(d[0]), "v"(d[1]), "v"(d[2]));
          asm("v_maximum3_f32 %0, %0, %0, |%1|" : "+v"(m) : "v"(d[3]));
          if (__builtin_amdgcn_ballot_w64(!(m < a.eps)) != 0ull)
            each<4>([&](auto xi) __attribute__((always_inline)) {
              constexpr int x = decltype(xi)::value;
              bad[c / 8] |= __builtin_fabsf(d[x]) < a.eps ? 0u : 1u << (4 * (c % 8) + x);
            });
        }
        each<4>([&](auto xi) __attribute__((always_inline)) {
          constexpr int x = decltype(xi)::value;
          sum += e[x];
        });
        s[c] = e;
      }
    });
    uint32_t any = 0u;
    each<(CH + 7) / 8>([&](auto bi) __attribute__((always_inline)) { any |= bad[decltype(bi)::value]; });
    if (FT && __builtin_amdgcn_ballot_w64(any != 0u) != 0ull) {
      each<(CH + 7) / 8>([&](auto bi) __attribute__((always_inline)) {
        constexpr int b = decltype(bi)::value;
        for (uint32_t m = bad[b]; m; m &= m - 1) {
          const int k = __builtin_ctz(m), col = 256 * (8 * b + (k >> 2)) + 4 * lane + (k & 3);
          if (col < nvalid) log_softmax_event(a, bh, FTDEC_ST_EXP, row, col);
        }
      });
      if (lane == 0) atomicAdd(a.retried, 1ull);
      continue;
    }
    const float inv = 1.0f / wave_sum(sum);
    // ---- normalised weights; eq. (12).  The weight that is summed and the one that is stored are one value:
    // without `opaque` the product is contracted into the sum and into the conversion, each with a
    // multiplication of its own, and the sum says nothing of what is stored (the lower half of 32 x 2048 x
    // 2048: 2 us).
    float psum = 0.f;
    each<CH>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = decltype(ci)::value;
      if (256 * c < jend) {
        half4 h = (half4)(_Float16)0.f;
        if (256 * c < nvalid) {
          each<4>([&](auto xi) __attribute__((always_inline)) {
            constexpr int x = decltype(xi)::value;
            const float p = opaque(inject(FTDEC_ST_PNORM, 256 * c + 4 * lane + x, s[c][x] * inv));
            if (FT) psum += p;
            h[x] = (_Float16)p;
          });
        }
        if (256 * c + 4 * lane < jend) *reinterpret_cast<half4*>(dst + 256 * c) = h;      // (jend is a multiple of 8)
      }
    });
    if (!FT) break;
    psum = wave_sum(psum);
    if (__builtin_fabsf(psum - 1.0f) < a.eps) break;
    if (lane == 0) {
      log_softmax_event(a, bh, FTDEC_ST_PNORM, row, -1);
      atomicAdd(a.retried, 1ull);
    }
  }
}

// Everything the two products need before they start, in one launch: grid (tiles, heads, roles).
// Role 0, 64 keys per workgroup: V [N][d] (fp16 or bf16 patterns) -> V^T [d][Np] in fp16, columns beyond N zero, and (FT)
// the tensor checksums of its rows (eq. (13), (14): 32 rows [32][Np], as encode_weight_rows forms them).  A
// 64 x 64 block at a time: 16 bytes per lane from memory, transposed through LDS (rows of 33 words: the eight keys
// a lane gathers, and the 16 lanes of a row, fall on banks of their own), 16 bytes per lane back; four threads per key
// fold its features from the same block.  The first workgroup also clears the counters of the softmax log.
// Role 1: the checksum rows of K.
// Bound: memory, one read of K and V and one write of V^T; for short sequences the launches.  Three launches (V^T with
// 16 bytes per lane, the checksums of K, those of V^T read back) took 23 us for 2 x 16 x 2048 x 128, this takes 14; for 2 x 5 x 151 x 128 they took 15.
// The second product gave that back at the larger size (76 us, 69 with three launches; 59 since its longest tiles come first): it reads
// V^T from memory, which the launch that read V^T back had just brought into the caches.
template <bool FT, bool BF>
__global__ __launch_bounds__(256) void ftdec_prepare(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, uint16_t* __restrict__ wc1,
                                                     _Float16* __restrict__ vt, _Float16* __restrict__ wc2, int N, int Np, int d, int Tn1,
                                                     int32_t* s_count, unsigned long long* retried) {
  typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
  typedef _Float16 half8 __attribute__((ext_vector_type(8)));
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));
  const int bh = blockIdx.y, tid = threadIdx.x;
  if (blockIdx.z == 1) {
    const int chunks = (d / 8 + 7) / 8, tn = blockIdx.x / chunks;
    if (tn < Tn1)
      ftgemm::encode_weight_rows<BF>(k + (size_t)bh * N * d, wc1 + (size_t)bh * Tn1 * ftgemm::GCK * d, N, d, tn, blockIdx.x % chunks);
    return;
  }
  __shared__ __attribute__((aligned(16))) _Float16 tile[64][66];
  __shared__ __attribute__((aligned(16))) _Float16 cks[ftgemm::GCK][64];
  const int k0 = blockIdx.x * 64;
  if (k0 >= Np) return;                     // (the whole workgroup, before any barrier)
  if (tid == 0 && blockIdx.x == 0 && bh == 0) { *s_count = 0; *retried = 0ull; }
  const uint16_t* src = v + (size_t)bh * N * d;
  _Float16* dst = vt + (size_t)bh * d * Np;
  // thread: key tid / 4 of the 64, classes 2 (tid % 4) and the next
  float c1[2] = {0.f, 0.f}, c2[2] = {0.f, 0.f};
  u16x8 u[2];                               // the thread's part of the block to come, requested while one is worked on
  auto request = [&](const int f0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int key = k0 + (tid >> 3) + 32 * i, c = (tid & 7) * 8;
      u[i] = (u16x8)(uint16_t)0;
      if (key < N && f0 + c < d) u[i] = *reinterpret_cast<const u16x8*>(src + (size_t)key * d + f0 + c);      // (d is a multiple of 8)
    }
  };
  request(0);
  for (int f0 = 0; f0 < d; f0 += 64) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (tid >> 3) + 32 * i, c = (tid & 7) * 8;
#pragma unroll
      for (int x = 0; x < 8; x += 2) {
        half2v h;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const uint16_t w = u[i][x + y];
          h[y] = BF ? (_Float16)__builtin_bit_cast(float, (uint32_t)w << 16) : __builtin_bit_cast(_Float16, w);
        }
        *reinterpret_cast<half2v*>(&tile[r][c + x]) = h;
      }
    }
    __syncthreads();
    request(f0 + 64);
#pragma unroll
    for (int e = tid; e < 64 * 8; e += 256) {
      const int f = e >> 3, r = (e & 7) * 8, key = k0 + r;
      half8 h;
#pragma unroll
      for (int x = 0; x < 8; ++x) h[x] = tile[r + x][f];
      if (f0 + f < d && key < Np) *reinterpret_cast<half8*>(dst + (size_t)(f0 + f) * Np + key) = h;      // (Np is a multiple of 8)
    }
    if (FT) {
      // (features beyond d are zeros in the tile)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const half2v h = *reinterpret_cast<const half2v*>(&tile[tid >> 2][8 * i + 2 * (tid & 3)]);
        const float weight = (float)(f0 / 8 + i + 1);
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          c1[y] += (float)h[y];
          c2[y] += weight * (float)h[y];
        }
      }
    }
    __syncthreads();
  }
  if (!FT) return;
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    const int cls = 2 * (tid & 3) + y, key = tid >> 2;
    const _Float16 h1 = (_Float16)c1[y], h2 = (_Float16)c2[y];
    cks[cls][key] = h1;
    cks[8 + cls][key] = (_Float16)(c1[y] - (float)h1);
    cks[16 + cls][key] = h2;
    cks[24 + cls][key] = (_Float16)(c2[y] - (float)h2);
  }
  __syncthreads();
  const int row = tid >> 3, at = (tid & 7) * 8;
  if (k0 + at < Np)
    *reinterpret_cast<half8*>(wc2 + ((size_t)bh * ftgemm::GCK + row) * Np + k0 + at) = *reinterpret_cast<const half8*>(&cks[row][at]);
}

typedef void (*prepare_fn)(const uint16_t*, const uint16_t*, uint16_t*, _Float16*, _Float16*, int, int, int, int, int32_t*, unsigned long long*);
static prepare_fn select_prepare(bool ft, bool bf) {
  if (ft) return bf ? ftdec_prepare<true, true> : ftdec_prepare<true, false>;
  return bf ? ftdec_prepare<false, true> : ftdec_prepare<false, false>;
}

}  // namespace ftdec

using namespace ftdec;

// Counters that a report goes by, all written by the kernels of a call (also where the call is the replay of a
// captured one): report slots per head of the two GEMMs, the softmax log's counter, rows evaluated again.
struct DStat { int32_t slots[2], s_count, pad; unsigned long long retried; };

struct ftdec_ctx {
  ftdec_config cfg;
  int BH = 0, N = 0, Np = 0, d = 0, Tn1 = 0;
  int slots1 = 0, slots2 = 0;    // report slots per head of the two GEMMs (allocated)
  uint32_t ring_n = 0;
  // device
  float* S = nullptr;
  _Float16* P = nullptr;
  void* scratch = nullptr;       // the allocation that holds all of the following
  _Float16* vt = nullptr;
  uint16_t* wc1 = nullptr;       // [BH][Tn1][32][d]
  uint16_t* wc2 = nullptr;       // [BH][1][32][Np]
  ftgemm_event* g_events = nullptr;   // [2*BH][ring_n] event rings of the GEMMs
  uint32_t* cursors = nullptr;        // [2*BH]
  ftgemm::GSlot* g_slots = nullptr;   // [BH][slots1], then [BH][slots2]
  DStat* stat = nullptr;
  ftdec_event* s_events = nullptr;
  ftgemm::GFault* d_gfaults = nullptr;
  SFault* d_sfaults = nullptr;
  ftgemm::GFault* h_gfaults = nullptr;   // pinned
  SFault* h_sfaults = nullptr;           // pinned
  int fault_cap = 0;
  int64_t bytes_total = 0, bytes_sp = 0;
  size_t softmax_lds = 0;
  std::vector<ftdec_event> events;
  std::vector<ftgemm::GSlot> h_slots;
  std::vector<ftgemm_event> h_gev;
  hipStream_t last_stream = nullptr;
  bool ran = false, timing = false;
  hipEvent_t ev[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};   // ends of the stages; before V^T, which counts with GEMM II
  std::string err;
};

static thread_local std::string g_dec_err;
static int dfail(ftdec_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg; else g_dec_err = msg;
  return code;
}
#define DHIP_TRY(ctx, expr)                                                                     \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return dfail(ctx, e_ == hipErrorOutOfMemory ? FTDEC_ENOMEM : FTDEC_EHIP,                  \
                   std::string(#expr) + ": " + hipGetErrorString(e_));                          \
  } while (0)

static void drelease(ftdec_ctx* c) {
  if (!c) return;
  (void)hipFree(c->S); (void)hipFree(c->P); (void)hipFree(c->scratch);
  if (c->h_gfaults) (void)hipHostFree(c->h_gfaults);
  if (c->h_sfaults) (void)hipHostFree(c->h_sfaults);
  for (hipEvent_t e : c->ev) if (e) (void)hipEventDestroy(e);
  delete c;
}

typedef void (*softmax_fn)(const SArgs);
// chunks of 256 scores a wave holds in registers for rows of N scores, or 0: the row is too long
static int softmax_chunks(int N) { return N <= 512 ? 2 : N <= 1024 ? 4 : N <= 2048 ? 8 : N <= 4096 ? 16 : 0; }
template <int CH> static softmax_fn pick_wave(bool ft, bool inject) {
  if (ft) return inject ? ftdec_softmax_wave<true, true, CH> : ftdec_softmax_wave<true, false, CH>;
  return inject ? ftdec_softmax_wave<false, true, CH> : ftdec_softmax_wave<false, false, CH>;
}
static softmax_fn select_softmax_wave(int chunks, bool ft, bool inject) {
  return chunks == 2 ? pick_wave<2>(ft, inject) : chunks == 4 ? pick_wave<4>(ft, inject)
         : chunks == 8 ? pick_wave<8>(ft, inject) : pick_wave<16>(ft, inject);
}
static softmax_fn select_softmax(bool ft, bool inject) {
  if (ft) return inject ? ftdec_softmax<true, true> : ftdec_softmax<true, false>;
  return inject ? ftdec_softmax<false, true> : ftdec_softmax<false, false>;
}

extern "C" int ftdec_create(const ftdec_config* cfg, ftdec_ctx** out) {
  if (!cfg || !out) return dfail(nullptr, FTDEC_EINVAL, "null argument");
  *out = nullptr;
  if (cfg->struct_size != sizeof(ftdec_config)) return dfail(nullptr, FTDEC_EINVAL, "struct_size mismatch");
  if (cfg->batch < 1 || cfg->heads < 1 || cfg->seq < 1) return dfail(nullptr, FTDEC_EINVAL, "batch, heads, seq must be >= 1");
  if ((long long)cfg->batch * cfg->heads > 65535) return dfail(nullptr, FTDEC_EUNSUPPORTED, "batch*heads > 65535");
  if (cfg->head_dim < 8 || cfg->head_dim % 8 != 0 || cfg->head_dim > 256) return dfail(nullptr, FTDEC_EUNSUPPORTED, "head_dim must be a multiple of 8, at most 256");
  if (cfg->in_dtype != FTDEC_F16 && cfg->in_dtype != FTDEC_BF16) return dfail(nullptr, FTDEC_EINVAL, "in_dtype must be F16 or BF16");
  if (cfg->causal != 0 && cfg->causal != 1) return dfail(nullptr, FTDEC_EINVAL, "causal must be 0 or 1");
  if (cfg->ft_mode != FTDEC_FT_OFF && cfg->ft_mode != FTDEC_FT_CORRECT) return dfail(nullptr, FTDEC_EINVAL, "ft_mode must be OFF or CORRECT");
  if ((long long)cfg->batch * cfg->heads * cfg->seq > 0x7FFFFFFFll) return dfail(nullptr, FTDEC_EUNSUPPORTED, "batch*heads*seq too large");
  ftdec_ctx* c = new (std::nothrow) ftdec_ctx();
  if (!c) return dfail(nullptr, FTDEC_ENOMEM, "out of host memory");
  c->cfg = *cfg;
  ftdec_config& e = c->cfg;
  if (!(e.softmax_scale > 0.f)) e.softmax_scale = 1.0f / std::sqrt((float)e.head_dim);
  if (!(e.tau_rel > 0.f)) e.tau_rel = 1.0f / 32768.0f;
  if (!(e.eps_dmr > 0.f)) e.eps_dmr = 1.0f / 4096.0f;
  if (e.max_events <= 0) e.max_events = 4096;
  c->BH = e.batch * e.heads; c->N = e.seq; c->Np = (e.seq + 7) & ~7; c->d = e.head_dim;
  c->Tn1 = (c->N + ftgemm::GBN - 1) / ftgemm::GBN;
  c->slots1 = std::max(ftgemm::gemm_slots(c->N, c->N, ftgemm::gemm_plan(c->N, c->N, c->d, c->BH, false, false)), ftgemm::gemm_slots(c->N, c->N, ftgemm::gemm_plan(c->N, c->N, c->d, c->BH, true, false)));
  c->slots2 = std::max(ftgemm::gemm_slots(c->N, c->d, ftgemm::gemm_plan(c->N, c->d, c->Np, c->BH, false, false)), ftgemm::gemm_slots(c->N, c->d, ftgemm::gemm_plan(c->N, c->d, c->Np, c->BH, true, false)));
  c->ring_n = ftgemm::ring_size(e.max_events);
  c->fault_cap = 1 << 16;
  hipError_t he = hipSetDevice(e.device);
  if (he != hipSuccess) { int rc = dfail(nullptr, FTDEC_EHIP, std::string("hipSetDevice: ") + hipGetErrorString(he)); delete c; return rc; }
  const size_t BH = c->BH, N = c->N, Np = c->Np, d = c->d, cap = e.max_events;
  struct { void** p; size_t bytes; bool sp; } allocs[] = {
      {(void**)&c->S, BH * N * N * 4, true}, {(void**)&c->P, BH * N * Np * 2, true}, {(void**)&c->vt, BH * d * Np * 2, false},
      {(void**)&c->wc1, BH * c->Tn1 * ftgemm::GCK * d * 2, false}, {(void**)&c->wc2, BH * ftgemm::GCK * Np * 2, false},
      {(void**)&c->g_events, 2 * BH * c->ring_n * sizeof(ftgemm_event), false}, {(void**)&c->cursors, 2 * BH * 4, false},
      {(void**)&c->g_slots, BH * (c->slots1 + c->slots2) * sizeof(ftgemm::GSlot), false}, {(void**)&c->stat, sizeof(DStat), false}, {(void**)&c->s_events, cap * sizeof(ftdec_event), false},
      {(void**)&c->d_gfaults, sizeof(ftgemm::GFault) * c->fault_cap, false},
      {(void**)&c->d_sfaults, sizeof(SFault) * c->fault_cap, false}};
  // S and P by themselves, everything else in one allocation: each one and its memset cost tens of microseconds
  auto room = [](size_t x) { return (x + 255) & ~(size_t)255; };
  size_t rest = 0;
  for (auto& al : allocs) rest += al.sp ? 0 : room(al.bytes);
  auto allocate = [&](void** p, size_t bytes) {
    he = hipMalloc(p, bytes);
    if (he == hipSuccess) he = hipMemset(*p, 0, bytes);
    if (he == hipSuccess) return (int)FTDEC_OK;
    int rc = dfail(nullptr, he == hipErrorOutOfMemory ? FTDEC_ENOMEM : FTDEC_EHIP, std::string("allocating device scratch: ") + hipGetErrorString(he));
    drelease(c);
    return rc;
  };
  if (const int rc = allocate(&c->scratch, rest)) return rc;
  size_t at = 0;
  for (auto& al : allocs) {
    if (al.sp) {
      if (const int rc = allocate(al.p, al.bytes + 16)) return rc;      // (the softmax reads up to three scores past a row)
      c->bytes_sp += (int64_t)al.bytes;
    } else {
      *al.p = static_cast<char*>(c->scratch) + at;
      at += room(al.bytes);
    }
    c->bytes_total += (int64_t)al.bytes;
  }
  he = hipHostMalloc((void**)&c->h_gfaults, sizeof(ftgemm::GFault) * c->fault_cap, hipHostMallocDefault);
  if (he == hipSuccess) he = hipHostMalloc((void**)&c->h_sfaults, sizeof(SFault) * c->fault_cap, hipHostMallocDefault);
  if (he == hipSuccess) he = ftgemm::gemm_allow_lds(ftgemm::gemm_plan(N, N, d, c->BH, false, false), e.ft_mode != FTDEC_FT_OFF, e.in_dtype == FTDEC_BF16);
  if (he == hipSuccess) he = ftgemm::gemm_allow_lds(ftgemm::gemm_plan(N, d, Np, c->BH, false, false), e.ft_mode != FTDEC_FT_OFF, false);
  // where a row takes a workgroup (more than 4096 scores) it is staged in LDS up to 8192 scores
  c->softmax_lds = N * 4 <= 32 * 1024 ? N * 4 : 0;
  if (he == hipSuccess) he = hipDeviceSynchronize();
  if (he != hipSuccess) {
    int rc = dfail(nullptr, FTDEC_EHIP, std::string("context set-up: ") + hipGetErrorString(he));
    drelease(c);
    return rc;
  }
  *out = c;
  return FTDEC_OK;
}

extern "C" int ftdec_get_config(const ftdec_ctx* c, ftdec_config* effective) {
  if (!c || !effective) return FTDEC_EINVAL;
  *effective = c->cfg;
  return FTDEC_OK;
}

extern "C" int ftdec_footprint(const ftdec_ctx* c, int64_t* total_bytes, int64_t* s_and_p_bytes) {
  if (!c || !total_bytes || !s_and_p_bytes) return FTDEC_EINVAL;
  *total_bytes = c->bytes_total;
  *s_and_p_bytes = c->bytes_sp;
  return FTDEC_OK;
}

extern "C" int ftdec_forward(ftdec_ctx* c, const void* q, const void* k, const void* v, void* o,
                             const ftdec_fault* faults, int32_t n_faults, void* hip_stream) {
  if (!c) return FTDEC_EINVAL;
  if (!q || !k || !v || !o) return dfail(c, FTDEC_EINVAL, "null tensor pointer");
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return dfail(c, FTDEC_EINVAL, "tensor pointers must be 16-byte aligned");
  if (n_faults < 0 || (n_faults > 0 && !faults)) return dfail(c, FTDEC_EINVAL, "bad fault list");
  if (n_faults > c->fault_cap) return dfail(c, FTDEC_EINVAL, "too many faults (limit 65536)");
  const ftdec_config& e = c->cfg;
  const int BH = c->BH, N = c->N, Np = c->Np, d = c->d;
  const bool ft = e.ft_mode != FTDEC_FT_OFF, bf = e.in_dtype == FTDEC_BF16;
  hipStream_t st = (hipStream_t)hip_stream;
  DHIP_TRY(c, hipSetDevice(e.device));

  // ---- fault list: GEMM faults grouped by (stage, head), softmax faults sorted by (head, row)
  std::vector<int> g_off(2 * (size_t)BH + 1, 0);
  int n_g = 0, n_s = 0;
  if (n_faults > 0) {
    std::vector<std::pair<long long, ftgemm::GFault>> gf;
    std::vector<SFault> sf;
    for (int i = 0; i < n_faults; ++i) {
      const ftdec_fault& f = faults[i];
      bool ok = f.b >= 0 && f.b < e.batch && f.h >= 0 && f.h < e.heads && f.row >= 0 && f.row < N && f.bit >= 0 && f.bit <= 31 &&
                f.stage >= FTDEC_ST_GEMM1 && f.stage <= FTDEC_ST_GEMM2 && f.col >= 0;
      if (ok && f.stage == FTDEC_ST_GEMM2) ok = f.col < d;
      if (ok && f.stage == FTDEC_ST_GEMM1) ok = f.col < N;
      if (ok && (f.stage == FTDEC_ST_EXP || f.stage == FTDEC_ST_PNORM)) ok = f.col < N && (!e.causal || f.col <= f.row);
      if (!ok) {
        char msg[160];
        snprintf(msg, sizeof msg, "fault %d (b=%d h=%d stage=%d row=%d col=%d bit=%d) names a masked or out-of-range position",
                 i, f.b, f.h, f.stage, f.row, f.col, f.bit);
        return dfail(c, FTDEC_EINVAL, msg);
      }
      const int bh = f.b * e.heads + f.h;
      if (f.stage == FTDEC_ST_GEMM1 || f.stage == FTDEC_ST_GEMM2)
        gf.push_back({(long long)(f.stage == FTDEC_ST_GEMM1 ? 0 : BH) + bh, ftgemm::GFault{f.row, f.col, f.bit}});
      else
        sf.push_back(SFault{bh * N + f.row, f.col, f.bit, f.stage});
    }
    std::stable_sort(gf.begin(), gf.end(), [](const auto& x, const auto& y) { return x.first < y.first; });
    std::stable_sort(sf.begin(), sf.end(), [](const SFault& x, const SFault& y) { return x.key < y.key; });
    n_g = (int)gf.size(); n_s = (int)sf.size();
    for (int i = 0; i < n_g; ++i) { c->h_gfaults[i] = gf[i].second; g_off[gf[i].first + 1]++; }
    for (size_t i = 0; i < 2 * (size_t)BH; ++i) g_off[i + 1] += g_off[i];
    for (int i = 0; i < n_s; ++i) c->h_sfaults[i] = sf[i];
    if (n_g) DHIP_TRY(c, hipMemcpyAsync(c->d_gfaults, c->h_gfaults, sizeof(ftgemm::GFault) * n_g, hipMemcpyHostToDevice, st));
    if (n_s) DHIP_TRY(c, hipMemcpyAsync(c->d_sfaults, c->h_sfaults, sizeof(SFault) * n_s, hipMemcpyHostToDevice, st));
    DHIP_TRY(c, hipStreamSynchronize(st));     // the staging buffers may be rewritten by the next call
  }

  // ---- V^T and the checksum rows of both products, one launch; while the stages are timed V^T alone, and the checksum
  // rows in launches of their own beside their products, so that every encode counts with its product
  const uint16_t* q16 = reinterpret_cast<const uint16_t*>(q);
  const uint16_t* k16 = reinterpret_cast<const uint16_t*>(k);
  const long long wc1_stride = (long long)c->Tn1 * ftgemm::GCK * d, wc2_stride = (long long)ftgemm::GCK * Np;
  const bool fused = ft && !c->timing;
  if (c->timing) DHIP_TRY(c, hipEventRecord(c->ev[4], st));
  hipLaunchKernelGGL(select_prepare(fused, bf), dim3(std::max((Np + 63) / 64, c->Tn1 * ((d / 8 + 7) / 8)), BH, fused ? 2 : 1), dim3(256), 0, st,
                     k16, reinterpret_cast<const uint16_t*>(v), c->wc1, c->vt, reinterpret_cast<_Float16*>(c->wc2), N, Np, d, c->Tn1,
                     &c->stat->s_count, &c->stat->retried);
  DHIP_TRY(c, hipGetLastError());
  if (c->timing) DHIP_TRY(c, hipEventRecord(c->ev[0], st));
  if (ft && !fused) DHIP_TRY(c, ftgemm::gemm_launch_encode_w(k16, c->wc1, N, d, bf, st, BH, (long long)N * d, wc1_stride));
  // (with a fault list every head runs the injecting tile shape, so that all slots have one stride)
  const ftgemm::GPlan plan1 = ftgemm::gemm_plan(N, N, d, BH, n_g > 0, false), plan2 = ftgemm::gemm_plan(N, d, Np, BH, n_g > 0, false);
  auto gemm_args = [&](int which, int bh) {
    ftgemm::GArgs a;
    std::memset(&a, 0, sizeof a);
    a.out_dtype = FTGEMM_F32;
    a.tau_rel = e.tau_rel; a.tau_abs = 0.f; a.correct = 1; a.transposed = 0;
    const int slot = which * BH + bh;
    a.faults = c->d_gfaults + g_off[slot];
    a.n_faults = g_off[slot + 1] - g_off[slot];
    a.events = c->g_events + (size_t)slot * c->ring_n;
    a.cursor = c->cursors + slot;
    a.ring_mask = c->ring_n - 1;
    const int per_head = which ? ftgemm::gemm_slots(N, d, plan2) : ftgemm::gemm_slots(N, N, plan1, e.causal && !n_g);
    a.n_slots = &c->stat->slots[which];
    a.slots = c->g_slots + (which ? (size_t)BH * c->slots1 : 0) + (size_t)bh * per_head;
    if (!n_g) { a.bs_events = c->ring_n; a.bs_slots = per_head; }
    return a;
  };

  // ---- 1. ABFT-GEMM I: S = Q K^T (tokens = queries, weight rows = keys).  Without a fault list all
  // heads go out as one batched launch; a fault list is applied head by head.
  for (int bh = 0; bh < (n_g ? BH : 1); ++bh) {
    ftgemm::GArgs a = gemm_args(0, bh);
    a.x = q16 + (size_t)bh * N * d; a.w = k16 + (size_t)bh * N * d; a.wc = c->wc1 + (size_t)bh * wc1_stride;
    a.y = c->S + (size_t)bh * N * N;
    a.M = N; a.N = N; a.K = d;
    if (!n_g) {
      a.bs_x = a.bs_w = (long long)N * d; a.bs_wc = wc1_stride; a.bs_y_bytes = (long long)N * N * 4;
      a.skip_upper = e.causal;      // score tiles above the diagonal are never read by the softmax (with a fault
                                    // list the matrix is computed in full: a fault may name any score)
    }
    DHIP_TRY(c, ftgemm::gemm_launch(a, ft, n_g > 0, bf, plan1, st, n_g ? 1 : BH));
  }
  if (c->timing) DHIP_TRY(c, hipEventRecord(c->ev[1], st));

  // ---- 2. DMR row-softmax, all heads in one launch
  {
    SArgs a;
    a.S = c->S; a.P = c->P; a.N = N; a.Np = Np; a.H = e.heads; a.causal = e.causal;
    a.scale_log2 = e.softmax_scale * 1.4426950408889634f;
    a.eps = e.eps_dmr;
    a.use_lds = c->softmax_lds ? 1 : 0;
    a.faults = c->d_sfaults; a.n_faults = n_s;
    a.events = c->s_events; a.ev_count = &c->stat->s_count; a.max_events = e.max_events;
    a.retried = &c->stat->retried;
    if (const int ch = softmax_chunks(N))
      hipLaunchKernelGGL(select_softmax_wave(ch, ft, n_s > 0), dim3((N + 3) / 4, BH), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL(select_softmax(ft, n_s > 0), dim3(N, BH), dim3(256), c->softmax_lds, st, a);
    DHIP_TRY(c, hipGetLastError());
  }
  if (c->timing) DHIP_TRY(c, hipEventRecord(c->ev[2], st));

  // ---- 3. ABFT-GEMM II: O = P V per head (tokens = queries, weight rows = the features of V^T)
  const uint16_t* vt16 = reinterpret_cast<const uint16_t*>(c->vt);
  const uint16_t* p16 = reinterpret_cast<const uint16_t*>(c->P);
  if (ft && !fused) DHIP_TRY(c, ftgemm::gemm_launch_encode_w(vt16, c->wc2, d, Np, false, st, BH, (long long)d * Np, wc2_stride));
  for (int bh = 0; bh < (n_g ? BH : 1); ++bh) {
    ftgemm::GArgs a = gemm_args(1, bh);
    a.x = p16 + (size_t)bh * N * Np; a.w = vt16 + (size_t)bh * d * Np; a.wc = c->wc2 + (size_t)bh * wc2_stride;
    a.y = reinterpret_cast<float*>(o) + (size_t)bh * N * d;
    a.M = N; a.N = d; a.K = Np;
    if (!n_g) {
      a.bs_x = (long long)N * Np; a.bs_w = (long long)d * Np; a.bs_wc = wc2_stride; a.bs_y_bytes = (long long)N * d * 4;
      a.k_lower = e.causal;         // P is lower-triangular: keys beyond a tile's last query contribute nothing
    }
    DHIP_TRY(c, ftgemm::gemm_launch(a, ft, n_g > 0, false, plan2, st, n_g ? 1 : BH));
  }
  if (c->timing) DHIP_TRY(c, hipEventRecord(c->ev[3], st));
  c->last_stream = st;
  c->ran = true;
  return FTDEC_OK;
}

extern "C" int ftdec_report(ftdec_ctx* c, ftdec_report_view* out) {
  if (!c || !out) return FTDEC_EINVAL;
  if (!c->ran) return dfail(c, FTDEC_EINVAL, "no forward call to report on");
  const ftdec_config& e = c->cfg;
  DHIP_TRY(c, hipSetDevice(e.device));
  DHIP_TRY(c, hipStreamSynchronize(c->last_stream));
  const int BH = c->BH, cap = e.max_events;
  DStat stat;
  DHIP_TRY(c, hipMemcpy(&stat, c->stat, sizeof stat, hipMemcpyDeviceToHost));
  c->events.clear();
  int dropped = 0;
  for (int which = 0; which < 2; ++which) {
    const int per_head = stat.slots[which];
    if (!per_head) continue;       // (captured, and never run)
    c->h_slots.resize((size_t)BH * per_head);
    DHIP_TRY(c, hipMemcpy(c->h_slots.data(), c->g_slots + (which ? (size_t)BH * c->slots1 : 0), c->h_slots.size() * sizeof(ftgemm::GSlot), hipMemcpyDeviceToHost));
    for (int bh = 0; bh < BH; ++bh) {
      const ftgemm::GSlot* sl = c->h_slots.data() + (size_t)bh * per_head;
      c->h_gev.clear();
      DHIP_TRY(c, ftgemm::gemm_fetch_events(sl, per_head, c->g_events + ((size_t)which * BH + bh) * c->ring_n, c->ring_n, cap, c->h_gev));
      dropped += (int)(ftgemm::gemm_stats(sl, per_head).events - (long long)c->h_gev.size());
      for (const ftgemm_event& g : c->h_gev)
        c->events.push_back(ftdec_event{bh / e.heads, bh % e.heads, which ? FTDEC_ST_GEMM2 : FTDEC_ST_GEMM1, g.row, g.col, g.action});
    }
  }
  {
    const int stored = std::min(stat.s_count, cap);
    dropped += stat.s_count - stored;
    const size_t base = c->events.size();
    c->events.resize(base + stored);
    if (stored) DHIP_TRY(c, hipMemcpy(c->events.data() + base, c->s_events, sizeof(ftdec_event) * stored, hipMemcpyDeviceToHost));
  }
  std::sort(c->events.begin(), c->events.end(), [](const ftdec_event& x, const ftdec_event& y) {
    if (x.b != y.b) return x.b < y.b;
    if (x.h != y.h) return x.h < y.h;
    if (x.stage != y.stage) return x.stage < y.stage;
    if (x.row != y.row) return x.row < y.row;
    return x.col < y.col;
  });
  out->n_events = (int32_t)c->events.size();
  out->n_events_dropped = dropped;
  out->events = c->events.data();
  out->retried_rows = (int64_t)stat.retried;
  return FTDEC_OK;
}

extern "C" int ftdec_set_timing(ftdec_ctx* c, int32_t enabled) {
  if (!c) return FTDEC_EINVAL;
  DHIP_TRY(c, hipSetDevice(c->cfg.device));
  if (enabled)
    for (hipEvent_t& e : c->ev)
      if (!e) DHIP_TRY(c, hipEventCreate(&e));
  c->timing = enabled != 0;
  return FTDEC_OK;
}

extern "C" int ftdec_get_timing(ftdec_ctx* c, float ms[3]) {
  if (!c || !ms) return FTDEC_EINVAL;
  if (!c->timing || !c->ran) return dfail(c, FTDEC_EINVAL, "timing is not enabled or no forward has run");
  DHIP_TRY(c, hipSetDevice(c->cfg.device));
  DHIP_TRY(c, hipEventSynchronize(c->ev[3]));
  for (int i = 0; i < 3; ++i) DHIP_TRY(c, hipEventElapsedTime(&ms[i], c->ev[i], c->ev[i + 1]));
  float vt = 0.f;
  DHIP_TRY(c, hipEventElapsedTime(&vt, c->ev[4], c->ev[0]));
  ms[2] += vt;
  return FTDEC_OK;
}

extern "C" int ftdec_destroy(ftdec_ctx* c) {
  if (!c) return FTDEC_EINVAL;
  (void)hipSetDevice(c->cfg.device);
  (void)hipDeviceSynchronize();
  drelease(c);
  return FTDEC_OK;
}

extern "C" const char* ftdec_last_error(const ftdec_ctx* c) {
  return c ? c->err.c_str() : g_dec_err.c_str();
}
