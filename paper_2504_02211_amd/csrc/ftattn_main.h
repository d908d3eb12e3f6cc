// The fused fault-tolerant attention kernel (gfx950 / CDNA4): Algorithm 1 of the paper from
// GEMM I to the final store, for one (batch, head, query row tile) per workgroup.
//
// Execution shape.  Wave w of a workgroup owns queries 32w .. 32w+31 of the row tile.
//  * head_dim 128: eight waves (256-query row tiles), one workgroup per CU.  The waves form two
//    groups of four (one wave of each group per SIMD) that run half an iteration apart: while one
//    group is in its MATRIX phase (GEMM II of key tile i and GEMM I of key tile i+1, back to back
//    on the MFMA pipe) the other is in its SOFTMAX phase (max, exp, product-form check, row-sum,
//    rescale: vector ALU only), and at every workgroup barrier they trade places.  Key / value
//    tiles arrive in LDS by direct global-to-LDS loads into a ring of three stages.
//  * head_dim 64: four waves (128-query row tiles), two independent workgroups per CU, so that a
//    SIMD again holds two waves, which the hardware interleaves as it finds them; one barrier per
//    iteration, a ring of two stages.  With the smaller head the softmax phase is about twice the
//    matrix phase, and the strict alternation would leave the matrix pipe and one of the two waves
//    idle half of the time; free-running waves keep the vector ALU busy from both.
// In either shape stage u of the ring holds V_u^T and K_{u+1}, the two operands one matrix phase reads.
//
// Register layout: see ftattn_device.h (scores transposed, one query per lane, the four
// stride-8 checksum classes of a lane and all their folds in the lane's own registers).
#pragma once
#include "ftattn_device.h"

namespace ftattn {

// waves per workgroup, query rows per workgroup and ring stages, by head_dim (see above)
constexpr int nwave_of(int d) { return d == 64 ? 4 : 8; }
constexpr int bm_of(int d) { return nwave_of(d) * 32; }
constexpr int nstage_of(int d) { return nwave_of(d) == 8 ? 3 : 2; }

// ---- workgroup id -> (head, row tile).  Workgroup ids go round-robin over the 8 XCDs (id & 7), and
// each XCD takes its ids in order as slots become free.
struct RowTile { int bh, ti; };

// Row tiles of equal length: each XCD a contiguous range of work, so that workgroups that share the
// K / V of a head share an L2.
__host__ __device__ __forceinline__ RowTile even_row_tile(int id, int total, int Ti) {
  const int xcd = id & 7, slot = id >> 3, qn = total >> 3, rn = total & 7;
  const int logical = xcd * qn + (xcd < rn ? xcd : rn) + slot;
  return RowTile{logical / Ti, logical % Ti};
}

// Causal row tiles (tile t visits (t + 1) times as many keys as tile 0).  With the contiguous ranges
// above an XCD may own more heavy tiles than another, and the heaviest tiles of its last head start
// when everything else is nearly done.  Here every XCD owns the same number of whole heads, taken in
// groups of `group` heads whose tiles are issued heaviest first across the group; the group that is not
// full comes first, so that what runs last are the light tiles of a full group.  The heads left over
// by the division by 8 come before all of these, dealt to the XCDs tile by tile.
// Measured against contiguous ranges: 8 x 16 x 2048 x 64 with checks 222 -> 201 us, 4 x 16 x 3000 x 64
// without 146 -> 128, 4 x 32 x 4096 x 128 988 -> 976.
__host__ __device__ __forceinline__ RowTile causal_row_tile(int id, int total, int Ti, int group) {
  const int BH = total / Ti, h8 = BH >> 3, left = BH & 7;
  if (id < left * Ti) return RowTile{8 * h8 + id % left, Ti - 1 - id / left};
  const int xcd = id & 7, first = h8 % group;
  int slot = (id - left * Ti) >> 3, head = xcd * h8, n = first;
  if (slot >= first * Ti) {
    slot -= first * Ti;
    const int full = slot / (group * Ti);
    slot -= full * group * Ti;
    head += first + full * group;
    n = group;
  }
  return RowTile{head + slot % n, Ti - 1 - slot / n};
}

// ---- the share of the keys of a row tile that a workgroup takes.  In a split call the row tiles from launch number
// `first_split` on are divided among up to `parts` workgroups each, by their key tiles: a row tile of L key tiles has
// ceil(L / piece) shares, of equal length to within one.  The first shares of all these row tiles are launched first, then
// the second ones of those that have one, and so on (longest row tiles first, and no workgroup without work: those
// would still be dealt to the shader engines in turn, and leave some with more than others).  The shares of a row
// tile leave their state in memory (store_part), ftattn_finish puts it together.
__host__ __device__ __forceinline__ int row_tiles_with(int part, bool causal, int n_split, int heads, int Ti, int piece, int tiles_per_row) {
  return causal ? heads * (Ti - part * piece / tiles_per_row) : n_split;      // those of more than `part` shares
}
struct Share {
  RowTile rt;
  int nj;                  // key tiles of the row tile
  int part, nparts;
  int first, count;        // key tiles of this share
  int rank, slot;          // number of the row tile among the split ones, of this share's state in memory
};
template <int D, bool CAUSAL> __device__ __forceinline__ void place_share(const KArgs& a, Share& h, bool split) {
  const int end = (h.rt.ti + 1) * bm_of(D), last_row = (end < a.N ? end : a.N) - 1;
  h.nj = CAUSAL ? last_row / BN + 1 : a.Tj;
  h.nparts = split ? (h.nj + a.piece - 1) / a.piece : 1;
  h.first = split ? h.nj * h.part / h.nparts : 0;
  h.count = split ? h.nj * (h.part + 1) / h.nparts - h.first : h.nj;
}
template <int D, bool CAUSAL> __device__ __forceinline__ RowTile split_row_tile(const KArgs& a, int rank) {
  const int heads = a.n_tiles / a.Ti;
  return CAUSAL ? RowTile{rank % heads, a.Ti - 1 - rank / heads} : even_row_tile(a.first_split + rank, a.n_tiles, a.Ti);
}
template <int D, bool CAUSAL, bool SPLIT> __device__ __forceinline__ Share share_of(const KArgs& a, int id) {
  Share h;
  h.part = h.slot = h.rank = 0;
  if (SPLIT && id >= a.first_split) {
    const int n_split = a.n_tiles - a.first_split, heads = a.n_tiles / a.Ti;
    h.slot = h.rank = id - a.first_split;
    for (int n = n_split; h.rank >= n; n = row_tiles_with(h.part, CAUSAL, n_split, heads, a.Ti, a.piece, bm_of(D) / BN)) {
      h.rank -= n;
      ++h.part;
    }
    h.rt = split_row_tile<D, CAUSAL>(a, h.rank);
    place_share<D, CAUSAL>(a, h, true);
    return h;
  }
  h.rt = CAUSAL ? causal_row_tile(id, a.n_tiles, a.Ti, a.head_group) : even_row_tile(id, a.n_tiles, a.Ti);
  place_share<D, CAUSAL>(a, h, false);
  return h;
}

// Heads per group: the fewest whose row tiles fill the workgroup slots of an XCD (32 CUs) once.  Larger
// groups would let fewer workgroups share the K / V of a head in the L2.  Never 0, and at most the heads of an XCD.
inline int head_group_of(int slots, int BH, int Ti) {
  const int h8 = BH >> 3, g = (slots + Ti - 1) / Ti;
  return g < h8 ? g : h8 > 0 ? h8 : 1;
}
inline int head_group(int D, bool ft, int BH, int Ti) { return head_group_of(32 * (D == 128 ? 1 : ft ? 2 : 3), BH, Ti); }

typedef void (*kernel_fn)(const KArgs);

template <int D, bool FT> struct Unit {
  static constexpr int KROWS = FT ? BN + CKR : BN;
  static constexpr int VROWS = FT ? D + CKR : D;
  static constexpr int KBYTES = KROWS * D * 2;
  static constexpr int VBYTES = VROWS * BN * 2;
  static constexpr int K_INSTR = KBYTES / 1024;     // one instruction moves 64 lanes x 16 bytes
  static constexpr int V_INSTR = VBYTES / 1024;
  static constexpr int NWAVE = nwave_of(D), NSTAGE = nstage_of(D);
  static constexpr int KPW = K_INSTR / NWAVE;
  static constexpr int VPW = (V_INSTR + NWAVE - 1) / NWAVE;
  // Every wave issues NLOAD instructions per unit.  A wave that has no piece left (uneven split) fetches its
  // first one again, into a 1 KB dump area at the end of the stage, so that the counted waits below hold for every wave.
  static constexpr int NLOAD = KPW + VPW;
  static constexpr int DUMP = V_INSTR % NWAVE ? 1024 : 0;
  static constexpr int BYTES = KBYTES + VBYTES + DUMP;
  static constexpr int LDS_TOTAL = NSTAGE * BYTES;
  static_assert(K_INSTR % NWAVE == 0 && V_INSTR >= NWAVE, "every wave owns as many pieces of a key tile, and at least one of a value tile");
  static_assert((NSTAGE - 1) * NLOAD <= 15, "counted waits use a 4-bit immediate");
  static_assert(NWAVE == 8 || 2 * LDS_TOTAL <= 160 * 1024, "two workgroups per CU");
};

// 16 bytes per lane from (uniform base + per-lane byte offset) straight into LDS at
// (uniform LDS address + 16*lane).  Opaque to the compiler on purpose (see gload_lds16 above); no
// memory clobber, so that operand reads of other ring stages may be scheduled around it.  Ordering
// against barriers and counted waits is kept because all of them are side-effecting instructions.
__device__ __forceinline__ void gload_lds16_off(const void* base, uint32_t byte_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr) : "m0");
}

// The queries of a lane (NQ times 16 bytes, 32 bytes apart), then the pieces of a unit (KPW of the key tile, VPW of the value tile, all but the last
// a fixed distance apart in memory and in LDS), then the wait for everything but these.
#define FTATTN_LOAD_Q(r, off) "global_load_dwordx4 %" #r ", %[q], off offset:" #off "\n\t"
#define FTATTN_PIECE(m, v, b) "s_mov_b32 m0, %[" #m "]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[" #v "], %[" #b "]\n\t"
template <int NQ, int KPW, int VPW>
__device__ __forceinline__ void queries_and_unit(const void* q, uint4v (&r)[NQ], uint32_t koff, uint32_t voff, const _Float16* k, const _Float16* v, int step,
                                                 uint32_t lds, uint32_t lds_step, const _Float16* last_v, uint32_t last_v_lds, uint32_t vbase) {
  static_assert((NQ == 4 || NQ == 8) && ((KPW == 2 && VPW == 2) || (KPW == 3 && VPW == 3)), "the shapes of Unit");
#define FTATTN_Q4 FTATTN_LOAD_Q(0, 0) FTATTN_LOAD_Q(1, 32) FTATTN_LOAD_Q(2, 64) FTATTN_LOAD_Q(3, 96)
#define FTATTN_Q8 FTATTN_Q4 FTATTN_LOAD_Q(4, 128) FTATTN_LOAD_Q(5, 160) FTATTN_LOAD_Q(6, 192) FTATTN_LOAD_Q(7, 224)
#define FTATTN_U2 FTATTN_PIECE(m0, ko, k0) FTATTN_PIECE(m1, ko, k1) FTATTN_PIECE(n0, vo, v0) FTATTN_PIECE(nl, vo, vl) "s_waitcnt vmcnt(4)"
#define FTATTN_U3 FTATTN_PIECE(m0, ko, k0) FTATTN_PIECE(m1, ko, k1) FTATTN_PIECE(m2, ko, k2) FTATTN_PIECE(n0, vo, v0) FTATTN_PIECE(n1, vo, v1) FTATTN_PIECE(nl, vo, vl) "s_waitcnt vmcnt(6)"
#define FTATTN_IN2 [q] "v"(q), [ko] "v"(koff), [vo] "v"(voff), [k0] "s"(k), [k1] "s"(k + step), [v0] "s"(v), [vl] "s"(last_v), \
                   [m0] "s"(lds), [m1] "s"(lds + lds_step), [n0] "s"(lds + vbase), [nl] "s"(last_v_lds)
#define FTATTN_IN3 FTATTN_IN2, [k2] "s"(k + 2 * step), [v1] "s"(v + step), [m2] "s"(lds + 2 * lds_step), [n1] "s"(lds + vbase + lds_step)
  if constexpr (NQ == 4 && KPW == 2)
    asm volatile(FTATTN_Q4 FTATTN_U2 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : FTATTN_IN2 : "m0", "memory");
  else if constexpr (NQ == 4)
    asm volatile(FTATTN_Q4 FTATTN_U3 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : FTATTN_IN3 : "m0", "memory");
  else if constexpr (KPW == 2)
    asm volatile(FTATTN_Q8 FTATTN_U2 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4 % NQ]), "=&v"(r[5 % NQ]), "=&v"(r[6 % NQ]), "=&v"(r[7 % NQ])
                 : FTATTN_IN2 : "m0", "memory");
  else
    asm volatile(FTATTN_Q8 FTATTN_U3 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4 % NQ]), "=&v"(r[5 % NQ]), "=&v"(r[6 % NQ]), "=&v"(r[7 % NQ])
                 : FTATTN_IN3 : "m0", "memory");
#undef FTATTN_Q4
#undef FTATTN_Q8
#undef FTATTN_U2
#undef FTATTN_U3
#undef FTATTN_IN2
#undef FTATTN_IN3
}
#undef FTATTN_LOAD_Q
#undef FTATTN_PIECE

struct yes { static constexpr bool value = true; };
struct no { static constexpr bool value = false; };

template <int N> __device__ __forceinline__ void wait_vmcnt() { __builtin_amdgcn_s_waitcnt(0x0F70 | N); }

__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// Value that the compiler must take as new: a second evaluation built on it is not merged with the first.
__device__ __forceinline__ float opaque(float x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ int opaque(int x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ half2v opaque(half2v x) { asm volatile("" : "+v"(x)); return x; }

// largest of 32 values, in two chains of three-input maxima
template <class T> __device__ __forceinline__ float max_of(const T& x, const T& y) {
  float a = fmax2(fmax2(x[0], x[1]), x[2]), b = fmax2(fmax2(y[0], y[1]), y[2]);
#pragma unroll
  for (int v = 3; v < 15; v += 2) {
    a = fmax2(fmax2(a, x[v]), x[v + 1]);
    b = fmax2(fmax2(b, y[v]), y[v + 1]);
  }
  a = fmax2(fmax2(a, x[15]), y[15]);
  return fmax2(a, b);
}

// Sum-form check of the output accumulator against its checksums (Algorithm 1, last "if"; text
// after eq. (16) for location and repair): class r of the lane, folds o[fb][4*gg + r].  `thr` is
// the threshold in the units the accumulator is in, `tile` the key tile reported with an event
// (-1 after the loop), `xfold` / `xv` the extra fold of class 0 in the exact row-sum mode.
template <int D, bool EW>
__device__ __forceinline__ bool sum_check(const KArgs& a, float16v (&o)[D / 32], const float16v& oc, const int bh, const int row, const int hi,
                                          const float thr, const int tile, const bool real, const bool xf, const float xv,
                                          const bool track, float& rmax_o) {
  constexpr int NFB = D / 32, NFOLD_V = D / 8;
  if (EW) {
    // one class over all D features of the row (fold index = feature), from both lanes of the query
    float sum1 = 0.f, chk1 = 0.f;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum1 += o[fb][v];
#pragma unroll
    for (int r = 0; r < 4; ++r) chk1 += oc[r] + oc[4 + r];
    sum1 = sum32(sum1); chk1 = sum32(chk1);
    const float R1 = chk1 - sum1;
    const bool d = real && !(__builtin_fabsf(R1) <= thr);
    if (track && !d && real) rmax_o = fmax2(rmax_o, __builtin_fabsf(R1));
    if (!wave_any(d)) return false;
    float chk2 = 0.f, sum2 = 0.f, big = -1.f;
    int l_big = -1;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      chk2 += 8.0f * (oc[8 + r] + oc[12 + r]) + (float)(4 * hi + r - 7) * (oc[r] + oc[4 + r]);
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int l = 32 * fb + 8 * (v >> 2) + 4 * hi + (v & 3);
        const float ov = o[fb][v];
        sum2 += (float)(l + 1) * ov;
        const float mag = finitef(ov) ? __builtin_fabsf(ov) : __builtin_inff();
        if (mag > big) { big = mag; l_big = l; } else if (mag == big) { l_big = -1; }
      }
    chk2 = sum32(chk2); sum2 = sum32(sum2);
    {
      const float bigp = xchg32(big, hi);
      const int lp = (int)xchg32((float)l_big, hi);
      if (bigp > big) l_big = lp; else if (bigp == big) l_big = -1;
    }
    int lstar = -1;
    {
      const float ratio = (chk2 - sum2) / R1;
      if (finitef(ratio)) {
        const float c = __builtin_rintf(ratio) - 1.0f;
        if (c >= 0.f && c < (float)D) lstar = (int)c;
      } else {
        lstar = l_big;
      }
    }
    if (!d) lstar = -1;
    float rest = 0.f;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (32 * fb + 8 * (v >> 2) + 4 * hi + (v & 3) != lstar) rest += o[fb][v];
    rest = sum32(rest);
    if (d) {
      const bool fix = a.correct && lstar >= 0;
      if (hi == 0) log_event(a, bh, FTATTN_CHECK_O, tile, row, lstar, R1, fix ? 1 : 0);
      if (fix) {
        const float val = chk1 - rest;
#pragma unroll
        for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (32 * fb + 8 * (v >> 2) + 4 * hi + (v & 3) == lstar) o[fb][v] = val;
      }
    }
    return true;       // events may have been written
  }
  bool bad = false;
  float R[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float sum1 = 0.f;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) sum1 += o[fb][4 * gg + r];
    if (r == 0 && xf) sum1 += xv;      // the normalised extra fold of class 0
    R[r] = (oc[r] + oc[4 + r]) - sum1;
    bool d = real && !(__builtin_fabsf(R[r]) <= thr);
    bad |= d;
    if (track && !d && real) rmax_o = fmax2(rmax_o, __builtin_fabsf(R[r]));
  }
  if (wave_any(bad)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (real && !(__builtin_fabsf(R[r]) <= thr)) {
        float chk1 = oc[r] + oc[4 + r], chk2 = oc[8 + r] + oc[12 + r];
        float sum2 = 0.f, big = -1.f;
        int l_big = -1;
#pragma unroll
        for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) {
            float ov = o[fb][4 * gg + r];
            sum2 += (float)(4 * fb + gg + 1) * ov;
            float mag = finitef(ov) ? __builtin_fabsf(ov) : __builtin_inff();
            if (mag > big) { big = mag; l_big = 4 * fb + gg; } else if (mag == big) { l_big = -1; }
          }
        const bool xfold = r == 0 && xf;      // class 0 has the row-sum as fold NFOLD_V
        if (xfold) {
          sum2 += (float)(NFOLD_V + 1) * xv;
          float mag = finitef(xv) ? __builtin_fabsf(xv) : __builtin_inff();
          if (mag > big) { big = mag; l_big = NFOLD_V; } else if (mag == big) { l_big = -1; }
        }
        float ratio = (chk2 - sum2) / R[r];
        int lstar = -1;
        if (finitef(ratio)) {
          float c = __builtin_rintf(ratio) - 1.0f;
          if (c >= 0.f && c < (float)(xfold ? NFOLD_V + 1 : NFOLD_V)) lstar = (int)c;
        } else {
          lstar = l_big;
        }
        if (xfold && lstar == NFOLD_V) continue;             // the row-sum itself: reported by its own check
        int col = lstar >= 0 ? 8 * lstar + 4 * hi + r : -1;
        bool fix = a.correct && lstar >= 0;
        log_event(a, bh, FTATTN_CHECK_O, tile, row, col, R[r], fix ? 1 : 0);
        if (fix) {
          float rest = xfold ? xv : 0.f;
#pragma unroll
          for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
              if (4 * fb + gg != lstar) rest += o[fb][4 * gg + r];
          float val = chk1 - rest;
#pragma unroll
          for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
              if (4 * fb + gg == lstar) o[fb][4 * gg + r] = val;
        }
      }
    }
    return true;       // events may have been written
  }
  return false;
}

// The largest statistics that passed, per row tile (non-negative floats order like their bits), and the re-evaluations.
__device__ __forceinline__ void note_statistics(const KArgs& a, const int bh, const int ti, const int lane, const float (&vals)[4], const unsigned rechecks) {
  uint32_t* rm = a.resmax + ((size_t)bh * a.Ti + ti) * 4;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const uint32_t v = wave_max_u32(as_u(vals[x]));
    if (lane == 63) atomicMax(rm + x, v);
  }
  if (lane == 0 && rechecks) atomicAdd(a.recheck, (unsigned long long)rechecks);
}

// What follows the last key tile of 32 query rows whose state a wave holds: row-sum range check, normalisation,
// sum-form check, store, statistics.
template <int D, bool FT, bool CAUSAL, int PS, class NOTE>
__device__ __forceinline__ void finish_rows(const KArgs& a, float16v (&o)[D / 32], float16v& oc, const int bh, const int ti, const int row,
                                            const int lane, const float l_part, const float l_low, const float m_run, const float m_true,
                                            const float dev_max, const NOTE& note) {
  constexpr int NFB = D / 32, NFOLD_V = D / 8;
  constexpr bool DMR = PS == 2, LAZY = PS == 4;
  const int N = a.N, hi = lane >> 5;
  const float sl2 = a.scale_log2;
  float rmax_o = 0.f, rmax_u = 0.f, rmax_l = 0.f;
  {
    const bool real = row < N;
    float l = sum32(l_part);
    const bool lfold = FT && a.rowsum_fold != 0;
    if (FT && lfold) {
      // The row-sum as fold NFOLD_V of checksum class 0 (held by the lane half hi == 0, register
      // r == 0): the row-sum the checksum implies against the accumulated one, in units of the
      // row-sum; on a mismatch the location rule over the NFOLD_V + 1 folds decides whether the
      // row-sum is the wrong element, and if so it is replaced by the implied one.
      float sumx = 0.f;
#pragma unroll
      for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) sumx += o[fb][4 * gg];
      const float chk1 = oc[0] + oc[4];
      const float lc = chk1 - sumx;
      const float rr = (lc - l) / lc;
      const bool detl = real && hi == 0 && (!(__builtin_fabsf(rr) <= a.tau_o) || !finitef(rr));
      if (!detl && real && hi == 0) rmax_u = fmax2(rmax_u, __builtin_fabsf(rr));
      if (wave_any(detl)) {
        if (detl) {
          const float chk2 = oc[8] + oc[12];
          float sum2 = (float)(NFOLD_V + 1) * l;
          float big = finitef(l) ? __builtin_fabsf(l) : __builtin_inff();
          int l_big = NFOLD_V;
#pragma unroll
          for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {
              const float ov = o[fb][4 * gg];
              sum2 += (float)(4 * fb + gg + 1) * ov;
              const float mag = finitef(ov) ? __builtin_fabsf(ov) : __builtin_inff();
              if (mag > big) { big = mag; l_big = 4 * fb + gg; } else if (mag == big) { l_big = -1; }
            }
          const float ratio = (chk2 - sum2) / (lc - l);
          int lstar = -1;
          if (finitef(ratio)) {
            const float c = __builtin_rintf(ratio) - 1.0f;
            if (c >= 0.f && c < (float)(NFOLD_V + 1)) lstar = (int)c;
          } else {
            lstar = l_big;
          }
          if (lstar == NFOLD_V) {
            log_event(a, bh, FTATTN_CHECK_L, -1, row, 0, rr, a.correct ? 1 : 0);
            if (a.correct) l = lc;
          }
        }
      }
      // the other half of the row takes the row-sum of the half that checked it
      const float lp = xchg32(l, hi);
      if (hi == 1) l = lp;
    }
    if (FT && !lfold && !DMR) {
      float Ub = CAUSAL ? (float)(row + 1 < N ? row + 1 : N) : (float)N;
      if (LAZY) Ub *= ex2((m_true - m_run) * sl2);      // exponentials reach exp(running maximum - reference)
      float lo = l_low;
      bool detl = real && !(lo * (1.f - a.delta_l) <= l && l <= Ub * (1.f + a.delta_l));
      if (!detl && real) { rmax_u = fmax2(rmax_u, l / Ub); rmax_l = fmax2(rmax_l, lo / l); }
      if (detl) {
        if (hi == 0) log_event(a, bh, FTATTN_CHECK_L, -1, row, 0, l, a.correct ? 1 : 0);
        if (a.correct) l = lo;     // the approximation of Section 3.4, "optimized EFTA"
      }
    }
    float inv = 1.0f / l;
#pragma unroll
    for (int fb = 0; fb < NFB; ++fb) o[fb] *= inv;
    if (FT) {
      oc *= inv;
      (void)sum_check<D, PS == 3>(a, o, oc, bh, row, hi, a.tau_o, -1, real, lfold && hi == 0, l * inv, true, rmax_o);
    }
    // ---- store: lane holds features 32*fb + 8*gg + 4*hi + (0..3) of its query
    if (real) {
      size_t base = ((size_t)bh * N + row) * D;
#pragma unroll
      for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) {
          int f = 32 * fb + 8 * gg + 4 * hi;
          float x0 = o[fb][4 * gg], x1 = o[fb][4 * gg + 1], x2 = o[fb][4 * gg + 2], x3 = o[fb][4 * gg + 3];
          if (a.out_dtype == FTATTN_F32) {
            float4 v = make_float4(x0, x1, x2, x3);
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + base + f) = v;
          } else if (a.out_dtype == FTATTN_F16) {
            _Float16 hv[4] = {(_Float16)x0, (_Float16)x1, (_Float16)x2, (_Float16)x3};
            *reinterpret_cast<uint2*>(reinterpret_cast<_Float16*>(a.o) + base + f) = *reinterpret_cast<uint2*>(hv);
          } else {
            uint32_t u[4] = {as_u(x0), as_u(x1), as_u(x2), as_u(x3)};
            uint16_t bv16[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              uint32_t rnd = ((u[x] >> 16) & 1u) + 0x7FFFu;
              bv16[x] = (u[x] & 0x7F800000u) == 0x7F800000u ? (uint16_t)(u[x] >> 16) : (uint16_t)((u[x] + rnd) >> 16);
            }
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.o) + base + f) = *reinterpret_cast<uint2*>(bv16);
          }
        }
    }
  }
  if (FT) {
    const float vals[4] = {dev_max, rmax_o, rmax_u, rmax_l};
    note(vals);
  }
}

// The state of 32 query rows after a share of their keys, as 64 lanes hold it: [slot][wave][value][lane].
template <int D, bool FT> constexpr int part_values() { return D / 2 + (FT ? 16 : 0) + (FT ? 3 : 2); }

template <int D, bool FT>
__device__ __forceinline__ void store_part(const KArgs& a, const float16v (&o)[D / 32], const float16v& oc, const Share& sh, const int wave,
                                           const int lane, const float l_part, const float l_low, const float m_run, const float dev_max,
                                           const unsigned rechecks) {
  float* at = a.ws + ((size_t)sh.slot * nwave_of(D) + wave) * (part_values<D, FT>() * 64) + lane;
  at[0] = m_run; at[64] = l_part;
  if (FT) at[128] = l_low;
  at += (FT ? 3 : 2) * 64;
#pragma unroll
  for (int fb = 0; fb < D / 32; ++fb)
#pragma unroll
    for (int v = 0; v < 16; ++v) at[(16 * fb + v) * 64] = o[fb][v];
  if (FT) {
    at += D / 2 * 64;
#pragma unroll
    for (int v = 0; v < 16; ++v) at[v * 64] = oc[v];
    const float vals[4] = {dev_max, 0.f, 0.f, 0.f};
    note_statistics(a, sh.rt.bh, sh.rt.ti, lane, vals, rechecks);
  }
}

// Row tiles whose keys were split: the shares brought to one maximum and added up (row-sum, its lower bound, output
// and output checksums are linear in the same factor e^{m_share - m}), then what the unsplit pass does after its
// last key tile.  A workgroup per 32 rows; wave w adds up feature block w, the first wave the checksums as well, and
// finishes.  Bound: the latency of reading one share after the other, so all maxima are requested at once and a share
// ahead of the one being added (12 row tiles of two shares took 20 us with a wave per 32 rows that read value by value).
// The maximum of a share is not checked: it scales row-sum, bound, output and checksums of its share alike, as a wrong
// running maximum does in the register of an unsplit pass.  Between the two launches it stands in memory, which the fault
// model leaves to ECC; every wave reads it and forms the factor by itself, so that an error in either by one wave shows
// in the sum-form check.
constexpr int MAX_PARTS = 16;
template <int D, bool FT, bool CAUSAL>
__global__ __launch_bounds__(D * 2) void ftattn_finish(const KArgs a) {
  constexpr int NV = part_values<D, FT>(), HEAD = FT ? 3 : 2, NFB = D / 32;
  __shared__ __attribute__((aligned(16))) float4 block[NFB - 1][4][64];
  const int rows = blockIdx.x % nwave_of(D), lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Share sh;
  sh.part = 0;
  sh.rank = (int)blockIdx.x / nwave_of(D);
  sh.rt = split_row_tile<D, CAUSAL>(a, sh.rank);
  place_share<D, CAUSAL>(a, sh, true);
  const int row0 = sh.rt.ti * bm_of(D) + 32 * rows, np = sh.nparts;
  if (np == 1 || row0 >= a.N) return;         // (the whole workgroup)
  const int n_split = a.n_tiles - a.first_split, heads = a.n_tiles / a.Ti;
  const float* in = a.ws + ((size_t)sh.rank * nwave_of(D) + rows) * (NV * 64) + lane;
  float mp[MAX_PARTS], m = -__builtin_inff();
  uint32_t at_part[MAX_PARTS];          // where the shares stand, in states
  {
    uint32_t at = 0;
#pragma unroll
    for (int p = 0; p < MAX_PARTS; ++p) {
      at_part[p] = at * (uint32_t)nwave_of(D);
      mp[p] = in[(size_t)at_part[p] * (NV * 64)];
      if (p + 1 < np) at += (uint32_t)row_tiles_with(p, CAUSAL, n_split, heads, a.Ti, a.piece, bm_of(D) / BN);
    }
  }
  // (a share past the last one is the last one again, not added)
  float16v x = (float16v)0.f, y = (float16v)0.f;
  float xl = 0.f, xlow = 0.f;
  auto request = [&](const int p) __attribute__((always_inline)) {
    const float* at = in + (size_t)at_part[p < MAX_PARTS ? p : MAX_PARTS - 1] * (NV * 64);
    if (wave == 0) {
      xl = at[64];
      if (FT) {
        xlow = at[128];
#pragma unroll
        for (int v = 0; v < 16; ++v) y[v] = at[(HEAD + D / 2 + v) * 64];
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = at[(HEAD + 16 * wave + v) * 64];
  };
  request(0);
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p) m = fmax2(m, mp[p]);
  float16v ob = (float16v)0.f, oc = (float16v)0.f;
  float l = 0.f, l_low = 0.f;
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p) {
    if (p >= np) break;
    const float f = ex2((mp[p] - m) * a.scale_log2);
    const float16v xp = x, yp = y;
    const float xlp = xl, xlowp = xlow;
    request(p + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 16; ++v) { ob[v] = __builtin_fmaf(xp[v], f, ob[v]); oc[v] = __builtin_fmaf(yp[v], f, oc[v]); }
    l = __builtin_fmaf(xlp, f, l);
    l_low = __builtin_fmaf(xlowp, f, l_low);
  }
  if (wave > 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) block[wave - 1][q][lane] = make_float4(ob[4 * q], ob[4 * q + 1], ob[4 * q + 2], ob[4 * q + 3]);
  }
  __syncthreads();
  if (wave > 0) return;
  float16v o[NFB];
  o[0] = ob;
#pragma unroll
  for (int fb = 1; fb < NFB; ++fb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = block[fb - 1][q][lane];
      o[fb][4 * q] = t.x; o[fb][4 * q + 1] = t.y; o[fb][4 * q + 2] = t.z; o[fb][4 * q + 3] = t.w;
    }
  finish_rows<D, FT, CAUSAL, 0>(a, o, oc, sh.rt.bh, sh.rt.ti, row0 + (lane & 31), lane, l, l_low, m, m, 0.f,
                                [&](const float (&vals)[4]) __attribute__((always_inline)) { note_statistics(a, sh.rt.bh, sh.rt.ti, lane, vals, 0u); });
}

// PS >= 1: verification after every step (the paper's EFTA before the unified verification of
// Section 3.4): GEMM I is verified on its own in every iteration, the row-sum against its range
// and the unnormalised output accumulator against its checksum after every GEMM II.
// PS == 2: in addition the softmax is protected by duplication (eq. (11), (12)) instead of the
// product-form check and the range restriction: maximum, exponentials and reduce-sum are
// evaluated twice and compared bit by bit; a third evaluation settles a difference.
// PS == 3: unified verification with the traditional checksum instead of the strided one (the
// comparison of Section 3.3 / 4.2): one class over the whole tile row (64 keys) and one over all
// features, i.e. stride 1 in eq. (13).  Its checksum values are the sums over the eight stride-8
// classes of the same encoded tiles (c1 = sum_c c1_c, c2 = sum_c 8 c2_c + (c - 7) c1_c), so the
// matrix work is the same; what changes is that a row has one residual per key tile, formed by
// the two lanes of a query together, and can name one element of 64 (of D for the output).
// SELF: the whole call in one launch, for heads of one row tile whose key and value tiles fit the ring (see self_encodes):
// the workgroup encodes them into LDS itself, each by one wave, in place of a launch that does so in memory.  Nothing else
// reads them, and what the first launch clears is written whole instead, or cleared by the workgroup that ends last.
// Measured, in two launches and in one: 1 x 1 x 128 x 64 12.5 and 9.3 us, 9 x 31 x 128 x 64 causal 22.6 and 16.7, 1 x 4 x 64 x 128 12.6
// and 10.9, 2 x 3 x 100 x 128 17.1 and 16.1, 2 x 3 x 150 x 128 causal 23.5 and 21.7, 9 x 31 x 64 x 128 25.7 and 23.2 (without checks 19.2
// and 17.4), 16 x 32 x 192 x 128 70 and 50.
template <int D, bool FT, bool CAUSAL, bool INJ, int PS = 0, bool SPLIT = false, bool SELF = false>
__global__ __launch_bounds__(nwave_of(D) * 64, nwave_of(D) == 8 ? 1 : FT ? 2 : 3) void ftattn_main(const KArgs a) {
  static_assert(!(SPLIT || SELF) || (PS == 0 && !INJ && SPLIT != SELF), "these run the default verification scheme without a fault list");
  static_assert(FT || PS == 0 || PS == 4, "the verification modes are modes of the protected kernel");
  constexpr bool DMR = PS == 2;
  constexpr bool STEP = PS == 1 || PS == 2;
  constexpr bool EW = PS == 3;
  // PS == 4 (an extension): the subtracted maximum is a reference that is renewed only when the running
  // maximum exceeds it by more than a margin; in all other iterations the rescale factor is exactly
  // one and the rescale of the output falls away.  Exponentials then reach e^margin; every identity of
  // Algorithm 1 holds with the reference in place of the maximum (Section 3.4, case 1).
  constexpr bool LAZY = PS == 4;
  // What becomes of a masked tile (see there): FILTER, looked through for anything to re-evaluate exactly; else always re-evaluated.  CONSTANT: the
  // weights of its masked keys are chosen to be 0 behind their exponentials, so that none of those is used; else they are checked like any other.
  constexpr bool FILTER = FT && !INJ && (PS == 0 || LAZY) && (CAUSAL || D == 128 || SELF);
  constexpr bool CONSTANT = FT && !INJ && (PS == 0 || LAZY) && !FILTER && !SPLIT;
  using U = Unit<D, FT>;
  constexpr int NWAVE = U::NWAVE, BM = NWAVE * 32, NSTAGE = U::NSTAGE;
  constexpr bool ALT = NWAVE == 8;      // two wave groups alternating between the phases (else: free-running waves)
  constexpr int NSLAB = D / 16;     // k-slabs of GEMM I
  constexpr int NFB = D / 32;       // 32-feature blocks of O^T
  constexpr int NFOLD_V = D / 8;
  constexpr int KCH = D / 8;        // 16-byte chunks per key row
  constexpr int KT_ELEMS = (BN + CKR) * D, VT_ELEMS = (D + CKR) * BN;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const Share sh = share_of<D, CAUSAL, SPLIT>(a, (int)blockIdx.x);
  const int bh = sh.rt.bh, ti = sh.rt.ti;
  const int j0 = sh.first;                  // the loop counts the key tiles of the share, from here
  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = ALT ? wave >> 2 : 0;
  const int N = a.N;
  const int row0_cta = ti * BM;
  const int row0_w = row0_cta + wave * 32;
  const int nj = sh.count;                                        // key tiles of the workgroup
  int nj_w = 0;                                                   // key tiles this wave takes part in
  if (row0_w < N) {
    int last_row_w = (row0_w + 32 < N ? row0_w + 32 : N) - 1;
    nj_w = (CAUSAL ? (last_row_w / BN + 1) : a.Tj) - j0;
    nj_w = nj_w < nj ? nj_w : nj;
  }
  const int row = row0_w + lq;
  const int row_end = (CAUSAL && row + 1 < N ? row + 1 : N) - 4 * hi;      // (see `valid`)
  const float sl2 = a.scale_log2;

  const _Float16* kc_head = a.kc + ((size_t)bh * a.Tj + j0) * KT_ELEMS;
  const _Float16* vt_head = a.vt + ((size_t)bh * a.Tj + j0) * VT_ELEMS;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

  // ---- per-lane source offsets of this wave's load instructions (the same for every tile).
  // Instruction wave + 8*i of a tile reads rows 512/chunks-per-row further down than instruction
  // wave, i.e. 8192 bytes further in either tile, and the swizzle of a row does not change over
  // that distance: one offset per tile kind is kept, the rest is added to the scalar base.
  uint32_t koff0, voff0;
  {
    const int L = wave * 64 + lane;
    const int rk = L / KCH, ck = (L % KCH) ^ swz_k<D>(rk);
    koff0 = (uint32_t)(rk * D + ck * 8) * 2u;
    const int rv = L / 8, cv = (L % 8) ^ swz_v(rv);
    voff0 = (uint32_t)(rv * BN + cv * 8) * 2u;
  }
  constexpr int PIECE_STEP = NWAVE * 64 * 8;      // halfs between the sources of consecutive pieces of a wave
  static_assert((NWAVE * 64 / KCH) * D == PIECE_STEP && (NWAVE * 64 / 8) * BN == PIECE_STEP, "piece stride");
  // unit u = { V_u^T, K_{u+1} } goes to stage (u+1) mod NSTAGE.  A unit is fetched in NLOAD pieces per wave; the pieces
  // of one unit are spread over a matrix phase (see matrix_stream).  Units are requested in their order, also
  // the one or two after the last key tile: those land in a stage that nobody reads any more, and what they fetch from
  // is the next tile in memory (the buffers end in TILES_BEYOND tiles nobody writes), so that neither addresses nor
  // destinations have to be selected in the stream.
  uint32_t ld_lds = smem_base + (uint32_t)wave * 1024u;
  const _Float16* ld_kt = kc_head;
  const _Float16* ld_vt = vt_head;
  constexpr bool UNEVEN = U::DUMP != 0;
  const bool last_v = !UNEVEN || U::VPW * NWAVE <= U::V_INSTR + NWAVE - 1 - wave;      // this wave has a VPW-th piece of a value tile
  const uint32_t last_v_lds = last_v ? (uint32_t)(U::KBYTES + (U::VPW - 1) * NWAVE * 1024) : (uint32_t)(U::KBYTES + U::VBYTES) - (uint32_t)wave * 1024u;
  const int last_v_src = last_v ? (U::VPW - 1) * PIECE_STEP : 0;
  auto issue_piece = [&](int n) __attribute__((always_inline)) {
    if (n < U::KPW) {
      gload_lds16_off(ld_kt + n * PIECE_STEP, koff0, ld_lds + (uint32_t)(n * NWAVE * 1024));
    } else {
      const int m = n - U::KPW;
      if (UNEVEN && m == U::VPW - 1) gload_lds16_off(ld_vt + last_v_src, voff0, ld_lds + last_v_lds);
      else gload_lds16_off(ld_vt + m * PIECE_STEP, voff0, ld_lds + (uint32_t)(U::KBYTES + m * NWAVE * 1024));
    }
  };
  auto next_unit = [&]() __attribute__((always_inline)) {
    ld_kt += KT_ELEMS;
    ld_vt += VT_ELEMS;
    ld_lds = ld_lds == smem_base + (uint32_t)((NSTAGE - 1) * U::BYTES) + (uint32_t)wave * 1024u ? smem_base + (uint32_t)wave * 1024u : ld_lds + (uint32_t)U::BYTES;
  };
  auto issue_unit = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < U::NLOAD; ++n) issue_piece(n);
    next_unit();
  };

  // faults of this workgroup
  int fcur = 0, fend = 0;
  const DevFault* __restrict__ F = a.faults;
  if (INJ && a.fault_off != nullptr) { fcur = a.fault_off[bh * a.Ti + ti]; fend = a.fault_off[bh * a.Ti + ti + 1]; }

  half8 qf[NSLAB];
  if constexpr (SELF) {
    // (queries requested first, converted last; registers for both and no more: see encode_v_rows)
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)bh * N + (row < N ? row : 0)) * D + 8 * hi;
    uint4v raw[D / 16];
#pragma unroll
    for (int sl = 0; sl < D / 16; ++sl) raw[sl] = *reinterpret_cast<const uint4v*>(qp + 16 * sl);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t rbits = 0u;
    // (a key tile is as many tasks as it has lanes' worth of work, 2.3 us each; a value tile is one, of 3.5 us at head_dim 64.  Value
    // tiles in two or three tasks gain nothing: 2 x 3 x 100 x 128 18.0 and 18.7 us, 1 x 1 x 16 x 64 8.7 and 8.9.)
    constexpr int KTASKS = D / 64;
    for (int task = wave; task < (KTASKS + 1) * nj; task += NWAVE) {
      if (task >= KTASKS * nj) {
        const int j = task - KTASKS * nj;
        rbits |= encode_v_rows<D, FT>(a.v, a.q_bf16, N, a.rowsum_fold != 0, j, bh, lane, smem + (j + 1) % NSTAGE * U::BYTES + U::KBYTES);
      } else {
        const int j = task / KTASKS;
        char* tile = smem + j % NSTAGE * U::BYTES;
        rbits |= encode_k_tile<D>(a.k, a.q_bf16, N, FT, j, bh, lane + 64 * (task % KTASKS), [&](const int r, const int ch, const half8& h) __attribute__((always_inline)) {
          *reinterpret_cast<half8*>(tile + r * (D * 2) + ((ch ^ swz_k<D>(r)) << 4)) = h;
        });
      }
    }
    RangeCheck operands;
#pragma unroll
    for (int sl = 0; sl < D / 16; ++sl) {
      if (row >= N) raw[sl] = (uint4v)0u;
      if (a.q_bf16) operands.add(raw[sl]);
      qf[sl] = to_half8(raw[sl], a.q_bf16 != 0);
    }
    rbits |= operands.bits();
    if (rbits) atomicOr(a.range, rbits);
    __syncthreads();
  } else {
  // The first key tile and the queries are waited for, unit 0 is not: GEMM I of the first tile needs nothing else.  From one
  // workgroup per CU on, unit 0 is requested right behind them, and its latency no longer stands between
  // the first two key tiles: 16 x 12 x 512 x 64 48.9 -> 45.7 us, 4 x 16 x 1000 x 64 causal 38.9 -> 37.6, 8 x 32 x 512 x 128 causal 97.8 -> 95.2,
  // 1 x 32 x 16384 x 128 causal 2845 -> 2818.  (Loads are waited for in their order, and the compiler, which counts the queries
  // only, would wait for unit 0 as well: so the queries are loaded, unit 0 requested and the wait made in one block.)  Elsewhere
  // it is requested when the queries are there: the first workgroup of every CU at once would only get its queries
  // later (2 x 8 x 300 x 128 27.6 and 28.0 us), and beside a second workgroup with many key tiles nothing is gained (8 x 16 x 2048 x 64
  // causal 183.7 and 186.2; 16 key tiles still gain, 32 lose; where two share a CU and 256 row tiles fill half of their places it gains
  // or loses 1 %: 4 x 16 x 512 x 64 23.5 and 23.6, 4 x 8 x 1000 x 64 34.8 and 34.7, 3 x 8 x 1500 x 64 causal 42.2 and 42.6).
  const bool early = a.n_tiles >= 256 && (D == 128 || a.Tj <= 24);
#pragma unroll
  for (int n = 0; n < U::KPW; ++n) issue_piece(n);
  next_unit();
  ld_vt = vt_head;          // (unit -1 has no value tile)

  // ---- Q_i^T as MFMA B operand: lane (query lq, half hi) holds Q[row][16*slab + 8*hi .. +7]
  // (bf16 queries are converted here: exact for magnitudes in the fp16 normal range)
  {
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)bh * N + (row < N ? row : 0)) * D + 8 * hi;
    RangeCheck operands;
    auto take = [&](const int sl, uint4v raw) __attribute__((always_inline)) {
      if (row >= N) raw = (uint4v)0u;
      if (a.q_bf16) operands.add(raw);
      qf[sl] = to_half8(raw, a.q_bf16 != 0);
    };
    if (early) {
      uint4v raw[NSLAB];
      queries_and_unit<NSLAB, U::KPW, U::VPW>(qp, raw, koff0, voff0, ld_kt, ld_vt, PIECE_STEP, ld_lds, (uint32_t)(NWAVE * 1024),
                                              ld_vt + last_v_src, ld_lds + last_v_lds, (uint32_t)U::KBYTES);
      next_unit();
#pragma unroll
      for (int sl = 0; sl < NSLAB; ++sl) take(sl, raw[sl]);
      if (const uint32_t qbits = operands.bits()) atomicOr(a.range, qbits);
    } else {
#pragma unroll
      for (int sl = 0; sl < NSLAB; ++sl) take(sl, *reinterpret_cast<const uint4v*>(qp + 16 * sl));
      if (const uint32_t qbits = operands.bits()) atomicOr(a.range, qbits);
      wait_vmcnt<0>();
      issue_unit();
    }
  }
  if (ALT) issue_unit();
  }

  float16v o[NFB], oc, s[2], sc;
  half8 ph[2][2];             // P^T in fp16, B operand of GEMM II: [key block][8-key half]
  float p[2][16];             // exp(S - m) of the key tile in flight, fp32
  float ps[2][2];             // (duplication mode) its row-sum, one partial per quarter
  float4a rs = (float4a)0.f;  // its row-sum (four times the same value)
  float ps2[2][2];            // (duplication mode) the second evaluation of the same
  float l2_part = 0.f, l_prev = 0.f;
  float al = 1.f;             // e^{m_old - m_new} of the key tile in flight
#pragma unroll
  for (int fb = 0; fb < NFB; ++fb) o[fb] = (float16v)0.f;
  oc = (float16v)0.f;
  // A share may begin with key tiles that hold only -inf for a row whose other shares hold finite scores (a pass over all keys
  // has met those by then): it starts from a maximum below every finite score (at most 128 * 65504^2 in magnitude), so
  // that these keys weigh 0, where -inf - -inf would make the row NaN.
  float m_run = SPLIT ? -1e20f : -__builtin_inff(), l_part = 0.f, l_low = 0.f, dev_max = 0.f;
  float m_true = -__builtin_inff();       // (LAZY) the running maximum; m_run is then the reference
  // the maximum to subtract after a key tile whose maximum is mxv (Algorithm 1: m_ij = max(m_i,j-1, rowmax))
  auto renewed = [&](const float mxv) __attribute__((always_inline)) -> float {
    if (!LAZY) return fmax2(m_run, mxv);
    const float mt = fmax2(m_true, mxv);
    return (mt - m_run) * a.scale > a.rescale_margin ? mt : m_run;      // (a reference of -inf is always renewed)
  };
  unsigned rechecks = 0;

  // The matrix phase as one stream of (LDS operand read, MFMA) pairs: first GEMM II of a key tile,
  //   O^T += V_j^T P^T (+ checksum block; the rescale was applied in the softmax phase),
  // then GEMM I of the next key tile,
  //   S^T = K_j Q^T, checksum block = K^c Q^T  (eq. (15), (16)).
  // The wave that runs this phase has the MFMA pipe of its SIMD to itself (its partner wave is in
  // the softmax phase), so the LDS latency must be hidden inside the stream: operand k+RING-1 is
  // requested before MFMA k is issued, and the scheduler is told to keep exactly that order.
  constexpr int NA2 = FT ? NFB + 1 : NFB;      // A operands per k-step of GEMM II
  constexpr int NA1 = FT ? 3 : 2;              // A operands per k-slab of GEMM I
  constexpr int RING = 6;
  // P -> fp16 in B-operand order: registers 8n..8n+7 of key block kb feed the MFMAs of k-step
  // t = 2*kb + n of GEMM II.  The row-sum adds up the converted pairs, the values GEMM II
  // multiplies (dot product with (1, 1), fp32 accumulation).  Quarter 0 is converted at the end of
  // the softmax phase; quarters 1..3 are converted inside the matrix phase, each ahead of its
  // k-step, where the vector instructions run in the shadow of the wave's own MFMAs.
  auto convert_quarter = [&](const int t) __attribute__((always_inline)) {
    const int kb = t >> 1, n = t & 1;
    if (DMR) ps[kb][n] = 0.f;
#pragma unroll
    for (int x = 0; x < 8; x += 2) {
      half2v pr2;
      pr2[0] = (_Float16)p[kb][8 * n + x]; pr2[1] = (_Float16)p[kb][8 * n + x + 1];
      ph[kb][n][x] = pr2[0]; ph[kb][n][x + 1] = pr2[1];
      const half2v ones = {(_Float16)1.f, (_Float16)1.f};
      if (DMR) ps[kb][n] = __builtin_amdgcn_fdot2(pr2, ones, ps[kb][n], false);
      if (DMR) ps2[kb][n] = __builtin_amdgcn_fdot2(opaque(pr2), ones, x == 0 ? 0.f : ps2[kb][n], false);
    }
  };
  // The row-sum of a quarter, on the matrix pipe: with ones as the A operand of the 4x4x4 product a lane's column is the sum of the
  // lane's own four values.  (As 16 dot products of fp16 pairs, which wait for the other wave's matrix instructions: one takes 40 cycles
  // while that wave keeps the pipe busy, a multiplication 9.  With that and the shorter requests of units
  // 8 x 16 x 2048 x 64 takes 280 us instead of 290, 1 x 32 x 16384 x 128 causal 2907 instead of 2967, 4 x 16 x 3000 x 64
  // without checks 124 instead of 128.)
  auto rowsum_quarter = [&](const int t) __attribute__((always_inline)) {
    const half8 h = ph[t >> 1][t & 1];
    const half4v one = {(_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f};
    rs = __builtin_amdgcn_mfma_f32_4x4x4f16(one, __builtin_shufflevector(h, h, 0, 1, 2, 3), t == 0 ? (float4a)0.f : rs, 0, 0, 0);
    rs = __builtin_amdgcn_mfma_f32_4x4x4f16(one, __builtin_shufflevector(h, h, 4, 5, 6, 7), rs, 0, 0, 0);
  };
  // reduce sum (Algorithm 1): one expression for every evaluation, so that they round alike
  auto rowsum_update = [&](float l_old, const float (&q4)[2][2]) __attribute__((always_inline)) -> float {
    return l_old * al + ((q4[0][0] + q4[0][1]) + (q4[1][0] + q4[1][1]));
  };
  // Operand addresses.  Row 32*y + lq of a K tile, chunk (2*sl + hi) XOR swizzle(lq), is at
  //   (tile + lq*row_bytes + ((hi ^ swizzle) << 4)) ^ (sl << 5), plus y*32 rows as an immediate:
  // the XOR only touches the chunk bits because every tile starts at a multiple of the row size.
  // One per-lane constant per tile kind serves all operands (likewise for V^T, whose chunk is
  // 4*(t>>1) + (t&1) XOR 2*hi); nothing per-lane has to follow the ring of stages.
  const uint32_t lane_k = (uint32_t)(lq * (D * 2) + ((hi ^ swz_k<D>(lq)) << 4));
  const uint32_t lane_v = (uint32_t)(lq * (BN * 2) + (((2 * hi) ^ swz_v(lq)) << 4));
  static_assert(U::BYTES % (D * 2) == 0 && U::KBYTES % (D * 2) == 0 && U::BYTES % (BN * 2) == 0 && U::KBYTES % (BN * 2) == 0,
                "tiles start at multiples of their row size");
  auto lds_rd = [](uint32_t addr) __attribute__((always_inline)) -> half8 {
    return *reinterpret_cast<const __attribute__((address_space(3))) half8*>((uintptr_t)addr);
  };
  auto matrix_stream = [&](uint32_t bv, uint32_t bk, auto do2_tag, auto do1_tag, auto ld_tag) __attribute__((always_inline)) {
    const uint32_t ak = bk + lane_k, av0 = bv + lane_v;
    constexpr bool DO2 = decltype(do2_tag)::value, DO1 = decltype(do1_tag)::value, LD = decltype(ld_tag)::value;
    constexpr int N2 = DO2 ? 4 * NA2 : 0, N1 = DO1 ? NSLAB * NA1 : 0, NOPS = N2 + N1;
    if (DO1) {
      s[0] = (float16v)0.f; s[1] = (float16v)0.f;
      if (FT) sc = (float16v)0.f;
    }
    half8 buf[RING];
    auto load_op = [&](int k) __attribute__((always_inline)) -> half8 {
      if (k < N2) {
        const int t = k / NA2, x = k % NA2;
        return lds_rd((av0 ^ (uint32_t)((4 * (t >> 1) + (t & 1)) << 4)) + (uint32_t)(x * 32 * BN * 2));
      }
      const int kk = k - N2, sl = kk / NA1, y = kk % NA1;
      return lds_rd((ak ^ (uint32_t)(sl << 5)) + (uint32_t)(y * 32 * D * 2));
    };
#pragma unroll
    for (int k = 0; k < RING - 1 && k < NOPS; ++k) buf[k] = load_op(k);
#pragma unroll
    for (int k = 0; k < NOPS; ++k) {
      if (k + RING - 1 < NOPS) buf[(k + RING - 1) % RING] = load_op(k + RING - 1);
      // one piece of the next-but-one unit every few MFMAs, so that the memory pipeline never backs up
      if (LD && k % (NOPS / U::NLOAD) == 1 && k / (NOPS / U::NLOAD) < U::NLOAD) issue_piece(k / (NOPS / U::NLOAD));
      const half8 av = buf[k % RING];
      if (DO2 && k < 3 * NA2 && k % NA2 == 0) convert_quarter(k / NA2 + 1);     // one k-step ahead of its use
      if (DMR && DO2 && k == 3 * NA2) {
        l_part = rowsum_update(l_part, ps);
        l2_part = rowsum_update(opaque(l2_part), ps2);
      }
      if (k < N2) {
        const int t = k / NA2, x = k % NA2;
        if (x < NFB) o[x] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, ph[t >> 1][t & 1], o[x], 0, 0, 0);
        else oc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, ph[t >> 1][t & 1], oc, 0, 0, 0);
        if (!DMR && x == 0) rowsum_quarter(t);
      } else {
        const int kk = k - N2, sl = kk / NA1, y = kk % NA1;
        if (y < 2) s[y] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, qf[sl], s[y], 0, 0, 0);
        else sc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, qf[sl], sc, 0, 0, 0);
        if (!DMR && DO2 && kk == 2) l_part = l_part * al + rs[0];      // reduce sum (Algorithm 1)
      }
    }
    // pin the order: RING-1 reads, then (MFMA, read) pairs, then the remaining MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, RING - 1, 0);
#pragma unroll
    for (int k = 0; k + RING - 1 < NOPS; ++k) {
      if (!DMR && k < N2 && k % NA2 == 0) __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
      else __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, RING - 1, 0);
  };
  // ---- prologue: the first key tile's scores; group 1 starts one barrier later than group 0
  phase_barrier();                                // everyone's pieces of the first key tile have landed

  if (ALT && grp == 1) phase_barrier();
  if (nj_w > 0) matrix_stream(smem_base, smem_base, no{}, yes{}, no{});
  if (ALT) {
    if (grp == 1) wait_vmcnt<U::NLOAD>();         // unit 0
    phase_barrier();
  }

  for (int i = 0; i < nj; ++i) {
    const int k0 = (j0 + i) * BN;
    const bool on = i < nj_w;
    const uint32_t stage = smem_base + (uint32_t)((i + 1) % NSTAGE) * U::BYTES;
    const bool tile_has_fault = INJ && fcur < fend && F[fcur].kv_tile == i;

    // =========================================================== softmax phase
    if (on) {
      const bool g_mask = (CAUSAL && k0 + BN - 1 > row0_w) || (k0 + BN > N);
      // keys of this tile that the row attends to, less what the lane half shifts its keys by: one comparison with a
      // constant tells whether a score is masked.  (With the key of every score compared with the row and the end of the
      // sequence, for the maximum, the exponentials and the filter each, 8 x 32 x 512 x 128 causal took 102.6 us and takes
      // 99.4, 2 x 3 x 333 x 128 28.9 and 26.7, 16 x 12 x 512 x 64 42.1 and 40.1.)
      int n_ok = row_end - k0;
      auto valid = [&](const int kb, const int v) __attribute__((always_inline)) -> bool { return 32 * kb + 8 * (v >> 2) + (v & 3) < n_ok; };

      // ---- injection point: raw scores
      if (tile_has_fault) {
        for (int fi = fcur; fi < fend && F[fi].kv_tile == i; ++fi) {
          if (F[fi].stage != FTATTN_ST_S) continue;
          int lr = F[fi].row - row0_w, kl = F[fi].col - k0, bit = F[fi].bit;
          bool mine = lr >= 0 && lr < 32 && lane == lr + 32 * ((kl & 7) >> 2);
          int tkb = kl >> 5, tv = 4 * ((kl & 31) >> 3) + (kl & 3);
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[kb][v] = flip_if(s[kb][v], mine && tkb == kb && tv == v, bit);
        }
      }

      float mx, m_new, negm;
      bool recheck = g_mask;

      if (!g_mask) {
        // ============ reduce max, exp (fast path: no masked entry in this tile)
        mx = max32(max_of(s[0], s[1]));
        m_new = renewed(mx);
        negm = -m_new * sl2;
        // all 32 arguments first, then all 32 exponentials, in place: neighbouring instructions are
        // independent, where (argument, exponential) pairs through one temporary would each wait
        // for the other
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) p[kb][v] = __builtin_fmaf(s[kb][v], sl2, negm);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) p[kb][v] = ex2(p[kb][v]);
      } else {
        // ============ same with the causal / sequence-end mask: a masked score counts as -inf, whose exponential is 0
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) p[kb][v] = valid(kb, v) ? s[kb][v] : -__builtin_inff();
        mx = max32(max_of(p[0], p[1]));
        m_new = renewed(mx);
        negm = -m_new * sl2;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int v = 0; v < 16; ++v) p[kb][v] = ex2(__builtin_fmaf(p[kb][v], sl2, negm));
        if (CONSTANT)
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) p[kb][v] = valid(kb, v) ? p[kb][v] : 0.f;
      }

      // ---- injection point: exponentials
      if (tile_has_fault) {
        for (int fi = fcur; fi < fend && F[fi].kv_tile == i; ++fi) {
          if (F[fi].stage != FTATTN_ST_EXP) continue;
          int lr = F[fi].row - row0_w, kl = F[fi].col - k0, bit = F[fi].bit;
          bool mine = lr >= 0 && lr < 32 && lane == lr + 32 * ((kl & 7) >> 2);
          int tkb = kl >> 5, tv = 4 * ((kl & 31) >> 3) + (kl & 3);
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) p[kb][v] = flip_if(p[kb][v], mine && tkb == kb && tv == v, bit);
        }
      }

      if (FT) {
        if (!g_mask) {
          // ============ unified product-form check of GEMM I, subtraction and exp
          // (Algorithm 1, first "if"; Section 3.4 case 2).  For class c the product of its 8
          // exponentials must equal exp2(sl2*check1 - 8*m).  Both sides are divided by that
          // prediction, two factors at a time, so the running product stays near one.
          bool bad = false;
          float dv[4] = {0.f, 0.f, 0.f, 0.f};
          // (2^(-e/4) per pair of factors, e = sl2*check1 + 8*negm the predicted log2 of the product)
          const float c_chk = sl2 * (-2.0f / NFOLD_K), c_m = -2.0f * negm;
          if (DMR) {
            // second evaluation of the maximum and of every exponential (eq. (11), (12)), compared bit
            // by bit; a third evaluation settles a differing maximum here, a differing exponential in
            // the exact path below
            float m0 = fmax2(opaque(s[0][0]), s[0][1]), m1 = fmax2(opaque(s[1][0]), s[1][1]);
#pragma unroll
            for (int v = 2; v < 16; v += 2) {
              m0 = fmax2(fmax2(m0, s[0][v]), s[0][v + 1]);
              m1 = fmax2(fmax2(m1, s[1][v]), s[1][v + 1]);
            }
            const float mxb = max32(fmax2(m0, m1));
            if (wave_any(as_u(mxb) != as_u(mx))) {
              float mc = opaque(s[0][0]);
#pragma unroll
              for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) mc = fmax2(mc, s[kb][v]);
              mc = max32(mc);
              if (as_u(mc) == as_u(mxb)) mx = mxb;          // two of three agree on the duplicate
              m_new = renewed(mx);
              negm = -m_new * sl2;
              bad = true;                                    // every exponential is looked at again below
            }
            uint32_t diff = 0u;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v) diff |= as_u(ex2(__builtin_fmaf(opaque(s[kb][v]), sl2, negm))) ^ as_u(p[kb][v]);
            bad |= diff != 0u;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float chk = sc[r] + sc[4 + r];
            if (!DMR) {
              float s2 = ex2(__builtin_fmaf(chk, c_chk, c_m));
              float pr = ((p[0][r] * p[0][4 + r]) * s2) * ((p[0][8 + r] * p[0][12 + r]) * s2);
              pr *= ((p[1][r] * p[1][4 + r]) * s2) * ((p[1][8 + r] * p[1][12 + r]) * s2);
              dv[r] = EW ? pr : pr - 1.0f;
            }
            if (STEP) {
              // strided ABFT of GEMM I alone (eq. (15)): same sum order as the exact evaluation below
              float sum1 = 0.f;
#pragma unroll
              for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int gg = 0; gg < 4; ++gg) sum1 += s[kb][4 * gg + r];
              bad |= !(a.scale * __builtin_fabsf(chk - sum1) <= 0.5f * a.eps1);
            }
          }
          if (EW) {
            // one class per row: the product of all 64 exponentials, from both lanes of the query
            const float pl = (dv[0] * dv[1]) * (dv[2] * dv[3]);
            dv[0] = pl * xchg32(pl, hi) - 1.0f;
            bad = !(__builtin_fabsf(dv[0]) <= a.tau_fast);
          }
          float dev = dev_max;           // the largest deviation that passed so far, and these (a NaN stays one)
          if (!EW && !DMR) {
            asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(dev) : "v"(dv[0]), "v"(dv[1]));
            asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(dev) : "v"(dv[2]), "v"(dv[3]));
            bad |= !(dev <= a.tau_fast);
          }
          recheck = wave_any(bad);
          if (recheck) ++rechecks;
          else if (EW) dev_max = fmax2(dev_max, __builtin_fabsf(dv[0]));
          else if (!DMR) dev_max = dev;
        }
        else if (FILTER) {
          // ============ masked tile: is there anything for the exact re-evaluation below to report?  With
          // every exponential equal to its second evaluation, and every masked weight 0, its lambda is -sigma*R1, so the tile passes
          // there exactly if it passes here.  (Every row tile ends in masked key tiles when causal; the
          // exact path costs about four times as many instructions, with a branch per element: 8 x 16 x 2048 x 64
          // took 201 us with it on every masked tile and 195 with this filter, 4 x 32 x 4096 x 128 976 and 938.
          // The kernels with the injection code have no registers left for it and take the exact path.
          // Without a causal mask only the last key tile can be masked, and at head_dim 64 the filter's registers
          // and code cost the others more than that tile gains where there are many: 8 x 16 x 2048 x 64 takes 278.7 us without it and
          // 281.3 with it, 16 x 12 x 512 x 64 44.1 and 44.6, 333 keys 18.0 and 17.2.  (There choosing masked weights costs 0.1 us, their
          // check 0.4 to 0.7 of the exact path: 2 x 3 x 333 x 64 17.6 and 18.0, 4 x 3 x 891 x 64 29.1 and 29.6; where keys are divided the choice
          // made the loop longer instead, also without a masked tile: 1 x 5 x 3008 x 64 47.9 and 46.0.)  Calls in one launch have two
          // tiles at most: 9 x 31 x 100 x 64 15.1 and 14.0.  The second evaluation is chosen to be 0 where masked, not skipped there: skipped, it
          // compiled to 32 regions with an execution mask of their own, 2 x 3 x 333 x 128 causal 26.1 us, like this 25.7.)
          bool bad = false;
          uint32_t diff = 0u;
          n_ok = opaque(n_ok);      // (the 32 comparisons are made again: kept, they would take 64 scalar registers)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float sum1 = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int gg = 0; gg < 4; ++gg) {
                const int v = 4 * gg + r;
                sum1 += s[kb][v];
                const uint32_t pe = as_u(ex2(__builtin_fmaf(opaque(s[kb][v]), sl2, negm)));
                diff |= (valid(kb, v) ? pe : 0u) ^ as_u(p[kb][v]);       // (a masked weight is 0)
              }
            bad |= !(a.scale * __builtin_fabsf((sc[r] + sc[4 + r]) - sum1) <= a.eps1);
          }
          recheck = wave_any(bad || diff != 0u);
        }
        if (recheck) {
          // ============ exact re-evaluation (rare: a fast check tripped, or the filter of a masked tile did).
          // lambda = ln prod P - (sigma*check1_eff - n_valid*m) = sum_l (ln P_l - x_l) - sigma*R1.
          bool lin_fixed = false, logged = false;
          n_ok = opaque(n_ok);
          // (hi, formed again: nothing of this path is kept in registers outside it)
          const int half = __builtin_amdgcn_mbcnt_hi((uint32_t)opaque(-1), __builtin_amdgcn_mbcnt_lo((uint32_t)opaque(-1), 0u)) >> 5;
          auto exponent = [&](const int kb, const int v) __attribute__((always_inline)) -> float {      // (-inf where masked: the weight is 0)
            return __builtin_fmaf(valid(kb, v) ? s[kb][v] : -__builtin_inff(), sl2, negm);
          };
          // Weights of masked scores are in no sum: they are 0 (or NaN, where the row has no finite maximum).  One that is not, is replaced below.
          uint32_t masked = 0u;
          if (g_mask && !CONSTANT)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v) masked |= valid(kb, v) ? 0u : as_u(p[kb][v]);
          auto none = [&]() __attribute__((always_inline)) -> float { return ex2(__builtin_fmaf(-__builtin_inff(), sl2, negm)); };
          const bool stray = !CONSTANT && masked != 0u && none() == 0.f;
          n_ok = opaque(n_ok);      // (comparisons made again, as above)
          if (EW) {
            // the whole tile row as one class (fold index = position of the key in the tile): every
            // sum is the lane's half plus its partner's, formed by all lanes alike (the exchanges
            // are wave-wide operations); only the event and the writes depend on the outcome
            float sum1 = 0.f, sum2 = 0.f, E = 0.f, chk1 = 0.f, chk2 = 0.f, big = -1.f;
            int nvalid = 0, l_big = -1;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float c1 = sc[r] + sc[4 + r];
              chk1 += c1;
              chk2 += 8.0f * (sc[8 + r] + sc[12 + r]) + (float)(4 * half + r - 7) * c1;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int l = key_of(kb, v, half);
                const bool ok = valid(kb, v);
                const float sv = s[kb][v];
                sum1 += sv;
                sum2 += (float)(l + 1) * sv;
                const float mag = finitef(sv) ? __builtin_fabsf(sv) : __builtin_inff();
                if (mag > big) { big = mag; l_big = l; } else if (mag == big) { l_big = -1; }
                const float t = __builtin_fmaf(sv, sl2, negm);
                const float pe = ex2(t);
                if (ok) {
                  ++nvalid;
                  if (as_u(pe) != as_u(p[kb][v])) E += lg2(p[kb][v]) - t;
                }
              }
            sum1 = sum32(sum1); sum2 = sum32(sum2); E = sum32(E); chk1 = sum32(chk1); chk2 = sum32(chk2);
            nvalid += (int)xchg32((float)nvalid, half);
            {
              const float bigp = xchg32(big, half);
              const int lp = (int)xchg32((float)l_big, half);
              if (bigp > big) l_big = lp; else if (bigp == big) l_big = -1;
            }
            const float R1 = chk1 - sum1;
            const float lam = LN2 * E - a.scale * R1;
            const bool linear = !(a.scale * __builtin_fabsf(R1) <= 0.5f * a.eps1);
            const bool det = nvalid > 0 && !(__builtin_fabsf(lam) <= a.eps1);
            int lstar = -1;
            {
              const float ratio = (chk2 - sum2) / R1;
              if (finitef(ratio)) {
                const float c = __builtin_rintf(ratio) - 1.0f;
                if (c >= 0.f && c < (float)BN) lstar = (int)c;
              } else {
                lstar = l_big;
              }
            }
            if (!(det && linear)) lstar = -1;
            float rest = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v)
                if (key_of(kb, v, half) != lstar) rest += s[kb][v];
            rest = sum32(rest);
            if (det || stray) {
              logged = true;
              if (det && linear) {
                const bool fix = a.correct && lstar >= 0;
                if (half == 0) log_event(a, bh, FTATTN_CHECK_S, j0 + i, row, lstar >= 0 ? k0 + lstar : -1, lam, fix ? 1 : 0);
                if (fix) {
                  const float val = chk1 - rest;
#pragma unroll
                  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                      if (key_of(kb, v, half) == lstar) s[kb][v] = val;
                  lin_fixed = true;
                }
              } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                  for (int v = 0; v < 16; ++v) {
                    const int key = k0 + key_of(kb, v, half);
                    const float pe = ex2(exponent(kb, v));
                    if (as_u(pe) != as_u(p[kb][v])) {
                      log_event(a, bh, FTATTN_CHECK_EXP, j0 + i, row, key, lam, a.correct ? 1 : 0);
                      if (a.correct) p[kb][v] = pe;
                    }
                  }
              }
            }
          }
#pragma unroll
          for (int r = 0; r < 4 && !EW; ++r) {
            float chk1 = sc[r] + sc[4 + r];
            float sum1 = 0.f, E = 0.f;
            int nvalid = 0;
            bool differs = false;       // an exponential that is not what its re-evaluation gives
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int gg = 0; gg < 4; ++gg) {
                int v = 4 * gg + r;
                bool ok = valid(kb, v);
                float sv = s[kb][v];
                sum1 += sv;
                float t = __builtin_fmaf(sv, sl2, negm);
                float pe = ex2(t);
                if (ok) {
                  ++nvalid;
                  if (as_u(pe) != as_u(p[kb][v])) { E += lg2(p[kb][v]) - t; differs = true; }
                }
              }
            float R1 = chk1 - sum1;
            float lam = LN2 * E - a.scale * R1;
            const bool linear = !(a.scale * __builtin_fabsf(R1) * 2.0f <= a.eps1);
            bool det = nvalid > 0 && (DMR ? (linear || differs) : (!(__builtin_fabsf(lam) <= a.eps1) || (STEP && linear)));
            if (det || stray) {
              logged = true;
              if (det && linear) {
                float chk2 = sc[8 + r] + sc[12 + r];
                float sum2 = 0.f, big = -1.f;
                int l_big = -1;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                  for (int gg = 0; gg < 4; ++gg) {
                    float sv = s[kb][4 * gg + r];
                    sum2 += (float)(4 * kb + gg + 1) * sv;
                    float mag = finitef(sv) ? __builtin_fabsf(sv) : __builtin_inff();
                    if (mag > big) { big = mag; l_big = 4 * kb + gg; } else if (mag == big) { l_big = -1; }
                  }
                float ratio = (chk2 - sum2) / R1;
                int lstar = -1;
                if (finitef(ratio)) {
                  float c = __builtin_rintf(ratio) - 1.0f;
                  if (c >= 0.f && c < (float)NFOLD_K) lstar = (int)c;
                } else {
                  lstar = l_big;   // residuals left the fp32 range: the fold of overwhelming size
                }
                int col = lstar >= 0 ? k0 + 32 * (lstar >> 2) + 8 * (lstar & 3) + 4 * half + r : -1;
                bool fix = a.correct && lstar >= 0;
                log_event(a, bh, FTATTN_CHECK_S, j0 + i, row, col, lam, fix ? 1 : 0);
                if (fix) {
                  float rest = 0.f;
#pragma unroll
                  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int gg = 0; gg < 4; ++gg)
                      if (4 * kb + gg != lstar) rest += s[kb][4 * gg + r];
                  float val = chk1 - rest;
#pragma unroll
                  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int gg = 0; gg < 4; ++gg)
                      if (4 * kb + gg == lstar) s[kb][4 * gg + r] = val;
                  lin_fixed = true;
                }
              } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                  for (int gg = 0; gg < 4; ++gg) {
                    int v = 4 * gg + r, key = k0 + key_of(kb, v, half);
                    // (a masked weight by the same choice as its first evaluation)
                    float pe = !CONSTANT ? ex2(exponent(kb, v)) : valid(kb, v) ? ex2(__builtin_fmaf(s[kb][v], sl2, negm)) : none();
                    if (as_u(pe) != as_u(p[kb][v])) {
                      log_event(a, bh, FTATTN_CHECK_EXP, j0 + i, row, key, lam, a.correct ? 1 : 0);
                      if (a.correct) p[kb][v] = pe;
                    }
                  }
              }
            }
          }
          // the event log's stores complete out of order with loads: drain before the counted waits
          if (wave_any(logged)) wait_vmcnt<0>();
          // a repaired score changes the row's maximum and exponentials: recompute the row
          // (the exchange is a wave-wide operation: evaluate it outside any per-lane short circuit)
          const float partner_fixed = xchg32(lin_fixed ? 1.f : 0.f, half);
          bool redo = lin_fixed | (partner_fixed != 0.f);
          if (wave_any(redo)) {
            float mx2 = -__builtin_inff();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                bool ok = valid(kb, v);
                mx2 = fmax2(mx2, ok ? s[kb][v] : -__builtin_inff());
              }
            mx2 = max32(mx2);
            if (redo) {
              mx = mx2;
              m_new = renewed(mx);
              negm = -m_new * sl2;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                bool ok = valid(kb, v);
                float pe = ok ? ex2(__builtin_fmaf(s[kb][v], sl2, negm)) : 0.f;
                if (redo) p[kb][v] = pe;
              }
          }
        }
      }

      // ============ rescale factor, lower bound of the row-sum (carried with the same rescale as the
      // row-sum itself, which is completed in the matrix phase), first quarter of P in fp16
      if (LAZY) m_true = fmax2(m_true, mx);
      // e^{m_old - m_new}, formed from the difference so that an unchanged maximum gives exactly one (the
      // product m_old * sl2 against the rounded m_new * sl2 would leave a rounding residue, and with it a
      // rescale of the whole output by 1 + 2^-23)
      al = ex2((m_run - m_new) * sl2);
      if (FT) l_low = l_low * al + ex2(__builtin_fmaf(mx, sl2, negm));
      m_run = m_new;
      convert_quarter(0);

      // ============ rescale of the running output (Algorithm 1: diag(e^{m_old - m_new}) O)
      if (wave_any(al != 1.f)) {
#pragma unroll
        for (int fb = 0; fb < NFB; ++fb) o[fb] *= al;
        if (FT) oc *= al;
      }
    }
    if (ALT) {
      if (grp == 0) wait_vmcnt<U::NLOAD>();       // unit i (unit i+1 may still be in flight)
    } else {
      wait_vmcnt<0>();                            // unit i (nothing younger has been requested)
    }
    phase_barrier();                              // ... everyone's pieces; and everyone is past the reads of the stage refilled next

    // =========================================================== matrix phase
    __builtin_amdgcn_s_setprio(1);
    // (after a wave's last key tile GEMM I runs on a tile it does not need: same code, result unused)
    if (DMR) l_prev = l_part;
    if (on) matrix_stream(stage + (uint32_t)U::KBYTES, stage, yes{}, yes{}, std::conditional_t<SELF, no, yes>{});
    else if (!SELF) {
#pragma unroll
      for (int n = 0; n < U::NLOAD; ++n) issue_piece(n);
    }
    if (!SELF) next_unit();
    __builtin_amdgcn_s_setprio(0);

    // ---- injection point: row-sum (right after the update of this iteration)
    if (tile_has_fault) {
      if (on) {
        for (int fi = fcur; fi < fend && F[fi].kv_tile == i; ++fi) {
          if (F[fi].stage != FTATTN_ST_ROWSUM) continue;
          int lr = F[fi].row - row0_w;
          bool mine = lr >= 0 && lr < 32 && lq == lr;
          float full = sum32(l_part);
          float flipped = flip_if(full, true, F[fi].bit);
          if (mine) l_part = hi ? 0.f : flipped;
        }
      }
    }
    // ---- injection point: output accumulator
    if (tile_has_fault) {
      if (on) {
        for (int fi = fcur; fi < fend && F[fi].kv_tile == i; ++fi) {
          if (F[fi].stage != FTATTN_ST_OACC) continue;
          int lr = F[fi].row - row0_w, col = F[fi].col, bit = F[fi].bit;
          bool mine = lr >= 0 && lr < 32 && lane == lr + 32 * ((col & 7) >> 2);
          int tfb = col >> 5, tv = 4 * ((col & 31) >> 3) + (col & 3);
#pragma unroll
          for (int fb = 0; fb < NFB; ++fb)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[fb][v] = flip_if(o[fb][v], mine && tfb == fb && tv == v, bit);
        }
      }
      while (fcur < fend && F[fcur].kv_tile == i) ++fcur;
    }
    if (STEP && on) {
      // ---- verification of this iteration's reduce-sum (range so far, Section 3.4 case 3) and of
      // GEMM II with the rescale (sum-form check on the unnormalised accumulator)
      const bool real = row < N;
      float l = sum32(l_part), rmax_step = 0.f;
      const int seen = k0 + BN < N ? k0 + BN : N;
      const float Ub = (float)(CAUSAL && row + 1 < seen ? row + 1 : seen);
      if (DMR) {
        // the two evaluations of the reduce-sum; a third one, from the fp16 P still in registers,
        // settles a difference
        const bool dl = as_u(l_part) != as_u(l2_part);
        if (wave_any(real && dl)) {
          float q3[2][2];
          const half2v ones = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
              q3[kb][n] = 0.f;
#pragma unroll
              for (int x = 0; x < 8; x += 2) {
                half2v pr2 = {ph[kb][n][x], ph[kb][n][x + 1]};
                q3[kb][n] = __builtin_amdgcn_fdot2(opaque(pr2), ones, q3[kb][n], false);
              }
            }
          const float l3 = rowsum_update(opaque(l_prev), q3);
          const bool row_dl = dl | (xchg32(dl ? 1.f : 0.f, hi) != 0.f);
          if (real && row_dl && hi == 0) log_event(a, bh, FTATTN_CHECK_L, i, row, 0, l, a.correct ? 1 : 0);
          if (a.correct && dl) {
            if (as_u(l3) == as_u(l2_part)) l_part = l2_part; else if (as_u(l3) == as_u(l_part)) l2_part = l_part;
          }
          l = sum32(l_part);
          wait_vmcnt<0>();    // the event log's stores complete out of order with loads: drain before the counted waits
        }
      }
      const bool detl = !DMR && real && !(l_low * (1.f - a.delta_l) <= l && l <= Ub * (1.f + a.delta_l));
      if (wave_any(detl)) {
        if (detl) {
          if (hi == 0) log_event(a, bh, FTATTN_CHECK_L, i, row, 0, l, a.correct ? 1 : 0);
          if (a.correct) { l = l_low; l_part = hi ? 0.f : l_low; }
        }
        wait_vmcnt<0>();      // the event log's stores complete out of order with loads: drain before the counted waits
      }
      if (sum_check<D, EW>(a, o, oc, bh, row, hi, a.tau_o * l, i, real, false, 0.f, false, rmax_step)) wait_vmcnt<0>();
    }
    if (ALT) {
      if (grp == 1) wait_vmcnt<U::NLOAD>();       // unit i+1 (unit i+2 may still be in flight)
      phase_barrier();
    }
  }
  if (ALT && grp == 0) phase_barrier();
  wait_vmcnt<0>();          // (the units after the last key tile: LDS is given back at the end)

  const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));      // (not kept through the loop)
  if constexpr (SELF) {
    // the statistics of the row tile are those of this workgroup's waves: written whole, through LDS (nobody reads the ring any more)
    __syncthreads();
    uint32_t* of_waves = reinterpret_cast<uint32_t*>(smem);
    finish_rows<D, FT, CAUSAL, PS>(a, o, oc, bh, ti, row0_w + (lane_e & 31), lane_e, l_part, l_low, m_run, m_true, dev_max, [&](const float (&vals)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const uint32_t v = wave_max_u32(as_u(vals[x]));
        if (lane_e == 63) of_waves[x * NWAVE + wave] = v;
      }
      if (lane_e == 0 && rechecks) atomicAdd(a.recheck, (unsigned long long)rechecks);
    });
    wait_vmcnt<0>();          // (this wave's counts and events are in memory)
    __syncthreads();
    if (wave == 0) {
      if (lane_e < 4) {
        uint32_t v = 0u;
        if (FT)
          for (int w = 0; w < NWAVE; ++w) v = of_waves[lane_e * NWAVE + w] > v ? of_waves[lane_e * NWAVE + w] : v;
        a.resmax[(size_t)bh * 4 + lane_e] = v;
      }
      if (lane_e == 0 && (gridDim.x == 1 || atomicInc(a.last.done, gridDim.x - 1) == gridDim.x - 1)) {      // (and is zero again)
        const int32_t events = atomicExch(a.ev_count, 0);
        const unsigned long long rechecked = atomicExch(a.recheck, 0ull);
        const uint32_t bits = atomicExch(a.range, 0u);
        __builtin_amdgcn_sched_barrier(0);
        *a.last.ev_count = events;
        *a.last.recheck = rechecked;
        *a.last.range = bits;
        *a.last.range_next = 0u;
      }
    }
    return;
  }
  if (!SPLIT || sh.nparts == 1)
    finish_rows<D, FT, CAUSAL, PS>(a, o, oc, bh, ti, row0_w + (lane_e & 31), lane_e, l_part, l_low, m_run, m_true, dev_max,
                                   [&](const float (&vals)[4]) __attribute__((always_inline)) { note_statistics(a, bh, ti, lane_e, vals, rechecks); });
  else
    store_part<D, FT>(a, o, oc, sh, wave, lane_e, l_part, l_low, m_run, dev_max, rechecks);
}

// A head of one row tile whose tiles the ring holds all at once: unit u stands in stage (u + 1) mod NSTAGE, and with
// at most NSTAGE key tiles none takes the place of another.
inline bool self_encodes(int D, int Ti, int Tj) { return Ti == 1 && Tj <= nstage_of(D); }

}  // namespace ftattn
