// gfx950 kernels for Y = alpha*A*X + beta*Y over Z/mZ on the tile table.
//
// One launch covers the whole matrix: workgroup g takes tile g, whatever the
// format of its row block. Three tile shapes:
//   STREAM  up to 256 consecutive rows whose entries are read with fully
//           coalesced 64-entry chunks; for one vector the terms (value times
//           gathered x) go to LDS and each row is summed from LDS by a group
//           of lanes sized to the tile (the CSR-Stream scheme of Greathouse
//           and Daga, SC'14, designed for AMD GPUs); for s > 1 vectors the
//           chunk stages words and values in LDS and the lanes take equal runs
//           of entries.
//   LONG    one row too long for a STREAM tile: all 256 lanes sweep it and
//           the partial sums meet through shuffles and LDS.
//   SELL    up to 4 slices of 64 rows stored column-major (ELL on a GPU is
//           column-major for coalescing, paper Section 2.4 "Basic formats"),
//           one lane per row, no LDS.
// Every tile may carry a band part: dense diagonals with one value per row,
// applied by one lane per row (the DIA idea of Section 2.1).
//
// Latency: a lane issues the loads of U chunks (entry words, then values and
// gathers) before it uses any of them, and the band part and row pointers,
// which do not depend on the entry stream, are loaded before it.
//
// Arithmetic (Section 2.2): each lane sums its terms in a wide accumulator
// and reduces modulo m only when the next term could overflow what the type
// represents exactly (CHUNK variants; the host sets reduce_every from the
// bound), otherwise once per row. Entries of residue 1 and m-1 carry no value
// (Section 2.4, "Taking into account the +-1"); a term multiplies by 1 or m - 1.
//
// Tx is the element type read from X (int32, int64, or a 16-bit copy of x
// when m <= 65536), Tv the element type of Y.
#pragma once

#include <algorithm>

#include "ffx_impl.h"
#include "launch.h"

namespace ffx {

// ------------------------------- arithmetic --------------------------------
// m <= 65536: values in 16 bits, one term (m-1)^2 < 2^32, and no row can have
// enough terms to reach 2^63, so a row is reduced once.
struct ArSmall {
  using ValT = uint16_t;
  using Acc = uint64_t;
  using Prod = uint32_t;
  static constexpr bool CHUNK = false;
  static constexpr bool CENTERED = false;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) { return v * x; }
  __device__ static inline uint32_t reduce(Acc a, const DevMat& A) { return mod_u64(a, A.m, A.mu); }
  __device__ static inline Acc from_residue(uint32_t r) { return r; }
};
// m > 65536 on 64-bit integers: a term is below 2^62.
template <bool CH>
struct ArBig {
  using ValT = uint32_t;
  using Acc = uint64_t;
  using Prod = uint64_t;
  static constexpr bool CHUNK = CH;
  static constexpr bool CENTERED = false;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) { return (uint64_t)v * x; }
  __device__ static inline uint32_t reduce(Acc a, const DevMat& A) { return mod_u64(a, A.m, A.mu); }
  __device__ static inline Acc from_residue(uint32_t r) { return r; }
};
// m = 2^31 - 1: since 2^31 = 1 (mod m), a product below 2^62 folds below
// 2^32 with one shift and one add, so a row needs no reduction inside it (a
// row of at most 2^30 + 64 folded terms stays below 2^63).
struct ArM31 {
  using ValT = uint32_t;
  using Acc = uint64_t;
  using Prod = uint64_t;
  static constexpr bool CHUNK = false;
  static constexpr bool CENTERED = false;
  static constexpr uint64_t M = 0x7FFFFFFFull;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) {
    uint64_t p = (uint64_t)v * x;
    return (p & M) + (p >> 31);
  }
  __device__ static inline uint32_t reduce(Acc a, const DevMat&) {
    a = (a & M) + (a >> 31);  // below 2^32 + 2^31 for a < 2^63
    a = (a & M) + (a >> 31);  // at most M + 2
    return (uint32_t)(a >= M ? a - M : a);
  }
  __device__ static inline Acc from_residue(uint32_t r) { return r; }
};
// GF(2) with bit-packed blocks: every 32-bit word of X holds bit j of 32
// vectors, an entry of A is 1 (m = 2 keeps only residue 1), and a sum over GF(2)
// is an exclusive or, so one word operation adds 32 products. The accumulator
// type makes + an exclusive or, so the tile code runs unchanged.
struct Gf2 {
  uint32_t v;
  Gf2() = default;
  __host__ __device__ Gf2(uint32_t x) : v(x) {}
  __device__ Gf2& operator+=(Gf2 o) {
    v ^= o.v;
    return *this;
  }
  __device__ Gf2 operator+(Gf2 o) const { return Gf2(v ^ o.v); }
};
using ::atomicAdd;  // the overload below must not hide the runtime's
__device__ inline void atomicAdd(Gf2* p, Gf2 x) { atomicXor(&p->v, x.v); }
struct ArGF2 {
  using ValT = uint16_t;
  using Acc = Gf2;
  using Prod = Gf2;
  static constexpr bool CHUNK = false;
  static constexpr bool CENTERED = false;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) { return Gf2((v & 1u) ? x : 0u); }
  __device__ static inline uint32_t reduce(Acc a, const DevMat&) { return a.v; }
  __device__ static inline Acc from_residue(uint32_t r) { return Gf2(r); }
};
// exact doubles: integers up to 2^53 add exactly.
template <typename V, bool CH>
struct ArF64 {
  using ValT = V;
  using Acc = double;
  using Prod = double;
  static constexpr bool CHUNK = CH;
  static constexpr bool CENTERED = false;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) { return (double)v * (double)x; }
  __device__ static inline uint32_t reduce(Acc a, const DevMat& A) { return mod_f64(a, A.m, A.inv_m); }
  __device__ static inline Acc from_residue(uint32_t r) { return (double)r; }
};

// exact floats: integers up to 2^24 add exactly (m <= 4096, values in 16 bits).
template <bool CH>
struct ArF32 {
  using ValT = uint16_t;
  using Acc = float;
  using Prod = float;
  static constexpr bool CHUNK = CH;
  static constexpr bool CENTERED = false;
  __device__ static inline Prod mul(uint32_t v, uint32_t x) { return (float)v * (float)x; }
  __device__ static inline uint32_t reduce(Acc a, const DevMat& A) { return mod_f32(a, A.m, A.inv_mf); }
  __device__ static inline Acc from_residue(uint32_t r) { return (float)r; }
};
// Centered residues (Section 2.2): a residue r is used as r - m when r > m/2,
// so every operand lies in [-h, h], h = floor(m/2), a product is at most h^2
// (about a quarter of (m-1)^2) in magnitude, and sums of both signs use the
// whole symmetric range of the floating type: about four times as many
// terms between reductions, and fp32 holds one product up to m = 8191. The
// stored entries and x stay canonical; operands are centered as they are
// used, partial reductions keep accumulators centered, and the final one
// returns the canonical residue.
template <typename F, typename V, bool CH>
struct ArCentered {
  using ValT = V;
  using Acc = F;
  using Prod = F;
  static constexpr bool CHUNK = CH;
  static constexpr bool CENTERED = true;
  __device__ static inline F lift(uint32_t r, uint32_t m) { return (F)(int32_t)(r > (m >> 1) ? r - m : r); }
  __device__ static inline F crem(F a, const DevMat& A) {
    if constexpr (sizeof(F) == 4) return crem_f32(a, A.m, A.inv_mf);
    else return crem_f64(a, A.m, A.inv_m);
  }
  __device__ static inline uint32_t reduce(Acc a, const DevMat& A) {
    F r = crem(a, A);
    return (uint32_t)(int32_t)(r < 0 ? r + (F)A.m : r);
  }
};

// one term v*x (the +-1 entries pass x or m - x), and a partial reduction
// that keeps an accumulator in the class's representation
template <class AR>
__device__ inline typename AR::Prod lift(uint32_t r, uint32_t m) {
  if constexpr (AR::CENTERED) return AR::lift(r, m);
  else return (typename AR::Prod)r;
}
template <class AR>
__device__ inline typename AR::Prod mul_term(uint32_t v, uint32_t x, uint32_t m) {
  if constexpr (AR::CENTERED) return AR::lift(v, m) * AR::lift(x, m);
  else return AR::mul(v, x);
}
template <class AR>
__device__ inline typename AR::Acc renorm(typename AR::Acc a, const DevMat& A) {
  if constexpr (AR::CENTERED) return AR::crem(a, A);
  else return AR::from_residue(AR::reduce(a, A));
}
template <class AR>
__device__ inline typename AR::Prod term(uint32_t tag, uint32_t v, uint32_t x, uint32_t m) {
  if (tag == TAG_GEN) return mul_term<AR>(v, x, m);
  if (tag == TAG_PLUS) return lift<AR>(x, m);
  if (tag == TAG_MINUS) return lift<AR>(m - x, m);
  return (typename AR::Prod)0;
}

// The value of an entry word, +-1 as 1 and m - 1 and 0 for padding: a term is then
// one product without a branch on the tag (whose lanes differ), and with several
// vectors the words of an entry are looked at once, not per vector.
__device__ inline uint32_t entry_value(uint32_t w, uint32_t v, uint32_t m) {
  const uint32_t tag = w >> TAG_SHIFT;
  return tag == TAG_GEN ? v : tag == TAG_PLUS ? 1u : tag == TAG_MINUS ? m - 1 : 0u;
}

// S accumulators of one lane with a shared countdown to the next reduction.
template <class AR, int S>
struct LaneAcc {
  typename AR::Acc a[S];
  int64_t left;
  __device__ inline void init(const DevMat& A) {
#pragma unroll
    for (int c = 0; c < S; ++c) a[c] = 0;
    left = A.reduce_every;
  }
  // called once per term position, after the S terms of that position were added
  __device__ inline void tick(const DevMat& A) {
    if (AR::CHUNK) {
      if (--left == 0) {
#pragma unroll
        for (int c = 0; c < S; ++c) a[c] = renorm<AR>(a[c], A);
        left = A.reduce_every;
      }
    }
  }
  // before partial sums of several lanes are added together
  __device__ inline void to_residues(const DevMat& A) {
    if (AR::CHUNK) {
#pragma unroll
      for (int c = 0; c < S; ++c) a[c] = renorm<AR>(a[c], A);
    }
  }
};

// ------------------------------- wave helpers ------------------------------
__device__ inline uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ inline uint64_t shfl_xor_u64(uint64_t v, int mask, int width) {
  uint32_t lo = __shfl_xor((int)(uint32_t)v, mask, width);
  uint32_t hi = __shfl_xor((int)(uint32_t)(v >> 32), mask, width);
  return ((uint64_t)hi << 32) | lo;
}
__device__ inline double shfl_xor_acc(double v, int mask, int width) { return __shfl_xor(v, mask, width); }
__device__ inline float shfl_xor_acc(float v, int mask, int width) { return __shfl_xor(v, mask, width); }
__device__ inline uint64_t shfl_xor_acc(uint64_t v, int mask, int width) { return shfl_xor_u64(v, mask, width); }
__device__ inline Gf2 shfl_xor_acc(Gf2 v, int mask, int width) { return Gf2((uint32_t)__shfl_xor((int)v.v, mask, width)); }

// stored values are streamed once: non-temporal loads keep them out of the way of x in L2
template <typename V>
__device__ inline uint32_t ldval(const void* p, uint32_t i) {
  return (uint32_t)__builtin_nontemporal_load((const V*)p + i);
}

// Writes row `row` of Y from the residues r[0..s).
template <typename Tv, int S>
__device__ inline void write_row(const DevMat& A, Tv* Y, int64_t ldy, uint32_t row, const uint32_t* r, int s,
                                 uint32_t alpha, uint32_t beta) {
  Tv* yr = Y + (int64_t)(A.rowmap ? A.rowmap[row] : row) * ldy;
#pragma unroll
  for (int c = 0; c < S; ++c) {
    if (c < s) {
      uint32_t yo = beta ? (uint32_t)yr[c] : 0u;
      uint32_t out = (alpha == 1 && beta == 0) ? r[c] : axpby(alpha, r[c], beta, yo, A.m, A.mu);
      yr[c] = (Tv)out;
    }
  }
}

// Adds the band terms of one row (diagonals d = first, first+step, ...). The
// x address depends only on the row and the offset, never on the stored value
// (absent entries hold 0), so all loads of a batch are issued together.
// Diagonals per batch: 16 gathers in flight per lane whatever S (more would
// only cost registers).
template <int S>
constexpr int band_batch() { return S >= 16 ? 1 : 16 / S > 8 ? 8 : 16 / S; }
template <class AR, typename Tx, int S>
__device__ inline void band_terms(const DevMat& A, const Tile& T, LaneAcc<AR, S>& acc, uint32_t row, uint32_t slot,
                                  uint32_t rows_in_tile, uint32_t first, uint32_t step, const Tx* X, int64_t ldx,
                                  int s) {
  constexpr int BAND_BATCH = band_batch<S>();
  const uint32_t nd = tile_nd(T.kind);
  for (uint32_t d0 = first; d0 < nd; d0 += BAND_BATCH * step) {
    uint32_t v[BAND_BATCH];
    uint32_t xv[BAND_BATCH][S];
#pragma unroll
    for (int q = 0; q < BAND_BATCH; ++q) {
      uint32_t d = d0 + q * step;
      bool in = d < nd;
      v[q] = in ? ldval<typename AR::ValT>(A.bval, T.b0 + d * rows_in_tile + slot) : 0u;
      int64_t col = in ? (int64_t)row + A.boffs[T.boff + d] : -1;
      bool ok = col >= 0 && col < (int64_t)A.ncols;
      const Tx* xr = X + (ok ? col : 0) * ldx;
#pragma unroll
      for (int c = 0; c < S; ++c) xv[q][c] = (ok && c < s) ? (uint32_t)xr[c] : 0u;
    }
#pragma unroll
    for (int q = 0; q < BAND_BATCH; ++q) {
      if (d0 + q * step < nd) {
#pragma unroll
        for (int c = 0; c < S; ++c) acc.a[c] += mul_term<AR>(v[q], xv[q][c], A.m);
        acc.tick(A);
      }
    }
  }
}

// Index of the first general value of this lane's four entry words w
// (entries 4*lane .. 4*lane+3 of a chunk whose value offset is vo). Values
// follow the entry order, so the lane's general values are consecutive, after
// those of lower lanes (four ballots over the wave).
__device__ inline uint32_t value_index4(const uint32_t* w, uint32_t vo) {
  uint32_t idx = vo;
#pragma unroll
  for (int k = 0; k < WIDE; ++k) idx += lanes_below(__ballot((w[k] >> TAG_SHIFT) == TAG_GEN));
  return idx;
}

// The general values of four entry words w whose first value is at index idx:
// one 12-byte (16-bit values) or 16-byte load fetches them all. Per lane: any
// lane may load the values of any row once it holds that row's words and index.
template <class AR>
__device__ inline void load_values_at(const DevMat& A, const uint32_t* w, uint32_t idx, uint32_t* v) {
  uint32_t g = 0;
#pragma unroll
  for (int k = 0; k < WIDE; ++k) g += (w[k] >> TAG_SHIFT) == TAG_GEN ? 1u : 0u;
  uint32_t q0 = 0, q1 = 0, q2 = 0, q3 = 0, j = 0;
  if constexpr (sizeof(typename AR::ValT) == 2) {
    if (g) {
      const uint32_t* p = (const uint32_t*)A.val + (idx >> 1);
      q0 = __builtin_nontemporal_load(p);
      q1 = __builtin_nontemporal_load(p + 1);
      q2 = __builtin_nontemporal_load(p + 2);
    }
    j = idx & 1u;
  } else {
    if (g) {
      const uint32_t* p = (const uint32_t*)A.val + idx;
      q0 = __builtin_nontemporal_load(p);
      q1 = __builtin_nontemporal_load(p + 1);
      q2 = __builtin_nontemporal_load(p + 2);
      q3 = __builtin_nontemporal_load(p + 3);
    }
  }
#pragma unroll
  for (int k = 0; k < WIDE; ++k) {
    bool gen = (w[k] >> TAG_SHIFT) == TAG_GEN;
    uint32_t val;
    if constexpr (sizeof(typename AR::ValT) == 2) {
      uint32_t d = j < 2 ? q0 : j < 4 ? q1 : q2;
      val = (d >> ((j & 1u) * 16)) & 0xffffu;
    } else {
      val = j == 0 ? q0 : j == 1 ? q1 : j == 2 ? q2 : q3;
    }
    v[k] = gen ? val : 0u;
    j += gen ? 1u : 0u;
  }
}

// Values of the four entry words w of this lane (entries 4*lane .. 4*lane+3
// of a chunk whose value offset is vo).
template <class AR>
__device__ inline void load_values4(const DevMat& A, const uint32_t* w, uint32_t vo, uint32_t* v) {
  load_values_at<AR>(A, w, value_index4(w, vo), v);
}

// U chunks of 256 entries, 4 words (16 bytes) per lane: the chunks of STREAM
// and LONG tiles, and the 4-column groups of SELL slices (where the 4 words of
// a lane are 4 consecutive entries of its row).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <class AR, typename Tx, int S, int U>
struct Chunk4 {
  uint32_t w[U][WIDE];
  uint32_t vo[U];
  uint32_t v[U][WIDE];
  uint32_t xv[U][WIDE][S];
  // step 1: at(u): this lane's 16-byte word group in chunk u, or null
  template <class At, class ChOff>
  __device__ inline void load_words(At at, ChOff choff_at) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u32x4* p = at(u);
      u32x4 q = p ? __builtin_nontemporal_load(p) : (u32x4)(PAD_WORD);
      w[u][0] = q.x;
      w[u][1] = q.y;
      w[u][2] = q.z;
      w[u][3] = q.w;
      vo[u] = choff_at(u);
    }
  }
  // step 2: values (1 and m - 1 for +-1 entries, 0 for padding) and gathered x. A term is then one
  // multiplication for every kind of entry; SKIP: padding is left out, for slices that are mostly padding
  // (the entries beside a band), otherwise it gathers row 0 like any entry. Without branches 20,001 rows of
  // about 60 entries modulo 2^31 - 1 take 28.0 us (40.1 with a branch per kind of entry, 34.2 with SKIP),
  // but 1,000,000 banded rows of 20 take 32.4 us (27.9, 27.5).
  template <bool SKIP>
  __device__ inline void load_gathers(const DevMat& A, const Tx* X, int64_t ldx, int s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load_values4<AR>(A, w[u], vo[u], v[u]);
#pragma unroll
      for (int k = 0; k < WIDE; ++k) {
        v[u][k] = entry_value(w[u][k], v[u][k], A.m);
        const bool on = !SKIP || (w[u][k] >> TAG_SHIFT) != TAG_PAD;
        const Tx* xr = X + (int64_t)(w[u][k] & COL_MASK) * ldx;
#pragma unroll
        for (int c = 0; c < S; ++c) xv[u][k][c] = on && c < s ? (uint32_t)xr[c] : 0u;
      }
    }
  }
  template <bool SKIP>
  __device__ inline void accumulate(const DevMat& A, LaneAcc<AR, S>& acc) const {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < WIDE; ++k)
        if (!SKIP || (w[u][k] >> TAG_SHIFT) != TAG_PAD) {
#pragma unroll
          for (int c = 0; c < S; ++c) acc.a[c] += mul_term<AR>(v[u][k], xv[u][k][c], A.m);
          acc.tick(A);
        }
  }
};

// The components of a row of X that one lane gathers: 16 bytes, so a row of
// eight int32 is two lanes. (Two loads of one row by the same lane, for four
// int64, are two requests to the L2: 72 us against 58 on 300,000 rows, s = 3.)
template <typename Tx, int S>
constexpr int lane_comps() { return sizeof(Tx) == 8 ? (S >= 2 ? 2 : 1) : S >= 4 ? 4 : S; }

// A lane's piece of rows: C components from c0 on, of which [lo, hi) are the
// lane's own. The last piece of a row ends where the row ends and then overlaps
// the one before it, so that every piece is one wide load without a condition;
// a lane with no component of its own (lo >= hi) loads that piece too. Only
// rows shorter than a piece are loaded element by element (SHORT: s = C - 1,
// three vectors of four, or one where a step always takes two); the tile code
// is built for either, since a choice at every gather makes the compiler split
// the wide loads into what the choices have in common (8 vectors of 32 bits on
// the 1M power law: 356 us with such a choice, 207 without).
template <int C>
struct RowPiece {
  int c0, lo, hi;
  __device__ inline RowPiece(uint32_t piece, int s) {
    c0 = max(0, min((int)piece * C, s - C));
    lo = (int)piece * C - c0;
    hi = min(C, s - c0);
  }
  __device__ inline bool used() const { return lo < hi; }
};

// Where lane slots (C to a piece) hold component c of a row of s.
template <int C>
__device__ inline int piece_slot(int c, int s) {
  const int p = c / C * C;
  return p + c - max(0, min(p, s - C));
}

typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));  // an element's alignment is enough
typedef uint32_t u32x4a8 __attribute__((ext_vector_type(4), aligned(8)));  // for a wide load or store
typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));

// The piece's residues of the row of X whose first element is at p. There is no
// condition on the entry: padding gathers row 0 with the value 0.
template <bool SHORT, typename Tx, int C>
__device__ inline void gather_comps(const Tx* p, const RowPiece<C>& rp, uint32_t* out) {
  if constexpr (SHORT) {
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = c + 1 < C ? (uint32_t)p[c] : 0u;
    return;
  }
  p += rp.c0;
  if constexpr (sizeof(Tx) == 4 && C == 4) {
    const u32x4a4 q = *(const u32x4a4*)p;
    out[0] = q.x, out[1] = q.y, out[2] = q.z, out[3] = q.w;
  } else if constexpr (sizeof(Tx) == 4 && C == 2) {
    const u32x2a4 q = *(const u32x2a4*)p;
    out[0] = q.x, out[1] = q.y;
  } else if constexpr (sizeof(Tx) == 8 && C == 2) {  // residues: the low words
    const u32x4a8 q = *(const u32x4a8*)p;
    out[0] = q.x, out[1] = q.z;
  } else {
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = (uint32_t)p[c];
  }
}

// The piece of row `row` of Y from the residues r.
template <typename Tv, int C>
__device__ inline void write_comps(const DevMat& A, Tv* Y, int64_t ldy, uint32_t row, const RowPiece<C>& rp, uint32_t* r,
                                   uint32_t alpha, uint32_t beta) {
  if (!rp.used()) return;
  Tv* y = Y + (int64_t)(A.rowmap ? A.rowmap[row] : row) * ldy;
  if (alpha != 1 || beta != 0) {
    uint32_t yo[C];
#pragma unroll
    for (int c = 0; c < C; ++c) yo[c] = 0u;
    if (beta) {
      if (rp.hi == C) gather_comps<false, Tv, C>(y, rp, yo);
      else gather_comps<true, Tv, C>(y, rp, yo);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = axpby(alpha, r[c], beta, yo[c], A.m, A.mu);
  }
  y += rp.c0;
  if constexpr (C >= 2) {
    if (rp.lo == 0 && rp.hi == C) {
      if constexpr (sizeof(Tv) == 4 && C == 4) {
        *(u32x4a4*)y = (u32x4a4){r[0], r[1], r[2], r[3]};
      } else if constexpr (sizeof(Tv) == 4) {
        *(u32x2a4*)y = (u32x2a4){r[0], r[1]};
      } else {
#pragma unroll
        for (int c = 0; c < C; c += 2) *(u32x4a8*)(y + c) = (u32x4a8){r[c], 0u, r[c + 1], 0u};
      }
      return;
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (c >= rp.lo && c < rp.hi) y[c] = (Tv)r[c];
}

// ------------------------------- SELL tile ---------------------------------
// A slice stores its rows in groups of 4 columns: group g is 256 words, word
// 4*lane + k being entry 4g + k of the slice's row `lane`; swidth holds the
// number of groups of each slice.
template <class AR, typename Tx, typename Tv, int S, int U, bool SKIP>
__device__ inline void sell_tile_1(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                 Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta) {
  const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  const uint32_t nsl = T.ne;
  if (wave >= nsl) return;
  uint32_t off = 0;
  for (uint32_t k = 0; k < wave; ++k) off += A.swidth[T.aux + k];
  const uint32_t groups = A.swidth[T.aux + wave];
  const uint32_t slot = wave * WAVE + lane;
  uint32_t row = (T.kind & TF_SORTED) ? A.perm[T.row0 + slot] : T.row0 + slot;
  const bool valid = row < A.nrows;
  const uint32_t* ent = A.ent + T.e0 + (size_t)off * SELL_GROUP + lane * WIDE;
  const uint32_t* choff = A.choff + T.c0 + off;
  auto words = [&](Chunk4<AR, Tx, S, U>& b, uint32_t g0) {
    b.load_words(
        [&](int u) -> const u32x4* {
          return g0 + u < groups ? (const u32x4*)(ent + (size_t)(g0 + u) * SELL_GROUP) : nullptr;
        },
        [&](int u) -> uint32_t { return g0 + u < groups ? choff[g0 + u] : 0u; });
  };
  // the first batch of entry words is requested before the band part, whose
  // loads then overlap its latency
  Chunk4<AR, Tx, S, U> first;
  words(first, 0);
  LaneAcc<AR, S> acc;
  acc.init(A);
  if (valid) band_terms<AR, Tx, S>(A, T, acc, row, slot, tile_rows(T.kind), 0, 1, X, ldx, s);
  first.template load_gathers<SKIP>(A, X, ldx, s);  // groups past the last hold padding words and add nothing
  first.template accumulate<SKIP>(A, acc);
  for (uint32_t g0 = U; g0 < groups; g0 += U) {
    Chunk4<AR, Tx, S, U> b;
    words(b, g0);
    b.template load_gathers<SKIP>(A, X, ldx, s);
    b.template accumulate<SKIP>(A, acc);
  }
  if (!valid) return;
  uint32_t r[S];
#pragma unroll
  for (int c = 0; c < S; ++c) r[c] = AR::reduce(acc.a[c], A);
  write_row<Tv, S>(A, Y, ldy, row, r, s, alpha, beta);
}

template <class AR, typename Tx, typename Tv, int S, int U>
__device__ inline void sell_tile(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                 Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta) {
  if (tile_nd(T.kind)) sell_tile_1<AR, Tx, Tv, S, U, true>(A, T, X, ldx, Y, ldy, s, alpha, beta);
  else sell_tile_1<AR, Tx, Tv, S, U, false>(A, T, X, ldx, Y, ldy, s, alpha, beta);
}

// SELL with s > 1 vectors: CL = S / C lanes share a row, each with C of its
// components, so a pass covers 64 / CL rows and a gather is one 16-byte load per
// lane (a vector-cache lane costs about a cycle whatever its width: with a lane
// per component a row of eight cost eight). The entry words and values of each
// row are loaded once per 4-column group with lane = row and handed to the
// lanes of its pass by shuffles. 300,000 rows of 20 entries, m = 65521: 102 ->
// 49 us with 8 vectors, 230 -> 69 with 16, unchanged (44, 43) with 4, where a
// lane held the whole row before too. Bound by the gathers: 64-byte rows at 8.
template <class AR, typename Tx, typename Tv, int S, bool SHORT>
__device__ inline void sell_tile_m(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                   Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta) {
  constexpr int C = lane_comps<Tx, S>(), CL = S / C, RPP = WAVE / CL;
  constexpr int KB = CL >= 4 ? 1 : CL == 2 ? 2 : WIDE;  // group columns per batch
  constexpr int DB = CL >= 4 ? 1 : 4 / CL;                   // diagonals per batch
  const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  const uint32_t nsl = T.ne;
  if (wave >= nsl) return;
  uint32_t off = 0;
  for (uint32_t k = 0; k < wave; ++k) off += A.swidth[T.aux + k];
  const uint32_t groups = A.swidth[T.aux + wave];
  const uint32_t sub = lane / CL;
  const RowPiece<C> piece(lane % CL, s);
  const uint32_t* ent = A.ent + T.e0 + (size_t)off * SELL_GROUP + lane * WIDE;
  const uint32_t* choff = A.choff + T.c0 + off;
  uint32_t prow[CL];  // row of each pass
#pragma unroll
  for (int p = 0; p < CL; ++p) {
    const uint32_t slot = wave * WAVE + p * RPP + sub;
    prow[p] = (T.kind & TF_SORTED) ? A.perm[T.row0 + slot] : T.row0 + slot;
  }
  LaneAcc<AR, CL * C> acc;  // acc.a[p * C + c]: component c0 + c of pass p
  acc.init(A);
  // band part
  const uint32_t nd = tile_nd(T.kind), rows_in_tile = tile_rows(T.kind);
  for (uint32_t d0 = 0; d0 < nd; d0 += DB) {
    uint32_t v[DB][CL], xv[DB][CL][C];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int p = 0; p < CL; ++p) {
        const uint32_t slot = wave * WAVE + p * RPP + sub;
        const int64_t col = d0 + d < nd ? (int64_t)prow[p] + A.boffs[T.boff + d0 + d] : -1;
        const bool ok = prow[p] < A.nrows && col >= 0 && col < (int64_t)A.ncols;
        v[d][p] = ok ? ldval<typename AR::ValT>(A.bval, T.b0 + (d0 + d) * rows_in_tile + slot) : 0u;
        gather_comps<SHORT, Tx, C>(X + (ok ? col : 0) * ldx, piece, xv[d][p]);
      }
#pragma unroll
    for (int d = 0; d < DB; ++d)
      if (d0 + d < nd) {
#pragma unroll
        for (int p = 0; p < CL; ++p)
#pragma unroll
          for (int c = 0; c < C; ++c) acc.a[p * C + c] += mul_term<AR>(v[d][p], xv[d][p][c], A.m);
        acc.tick(A);
      }
  }
  u32x4 next = groups ? __builtin_nontemporal_load((const u32x4*)ent) : (u32x4)(PAD_WORD);
  for (uint32_t g = 0; g < groups; ++g) {
    const uint32_t w[WIDE] = {next.x, next.y, next.z, next.w};
    uint32_t v[WIDE];
    load_values4<AR>(A, w, choff[g], v);
#pragma unroll
    for (int k = 0; k < WIDE; ++k) v[k] = entry_value(w[k], v[k], A.m);
    // the next group's words are requested before this one's gathers
    if (g + 1 < groups) next = __builtin_nontemporal_load((const u32x4*)(ent + (size_t)(g + 1) * SELL_GROUP));
    // (with two or more batches a real loop: unrolled, the next batch's shuffles and gathers are hoisted
    // over this one's terms, which cost 156 registers at S = 16 against 100)
#pragma unroll 1
    for (int k0 = 0; k0 < WIDE; k0 += KB) {
      uint32_t wk[KB], vk[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        wk[k] = KB == WIDE ? w[k] : KB == 2 ? (k0 ? w[2 + k] : w[k]) : k0 < 2 ? (k0 ? w[1] : w[0]) : k0 == 2 ? w[2] : w[3];
        vk[k] = KB == WIDE ? v[k] : KB == 2 ? (k0 ? v[2 + k] : v[k]) : k0 < 2 ? (k0 ? v[1] : v[0]) : k0 == 2 ? v[2] : v[3];
      }
      // every gather of the batch is issued before the first term is added
      uint32_t xv[KB][CL][C];
#pragma unroll
      for (int k = 0; k < KB; ++k)
#pragma unroll
        for (int p = 0; p < CL; ++p) {
          const uint32_t wp = CL == 1 ? wk[k] : (uint32_t)__shfl((int)wk[k], p * RPP + (int)sub);
          gather_comps<SHORT, Tx, C>(X + (int64_t)(wp & COL_MASK) * ldx, piece, xv[k][p]);
        }
#pragma unroll
      for (int k = 0; k < KB; ++k) {
#pragma unroll
        for (int p = 0; p < CL; ++p) {
          const uint32_t vp = CL == 1 ? vk[k] : (uint32_t)__shfl((int)vk[k], p * RPP + (int)sub);
#pragma unroll
          for (int c = 0; c < C; ++c) acc.a[p * C + c] += mul_term<AR>(vp, xv[k][p][c], A.m);
        }
        acc.tick(A);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < CL; ++p)
    if (prow[p] < A.nrows) {
      uint32_t r[C];
#pragma unroll
      for (int c = 0; c < C; ++c) r[c] = AR::reduce(acc.a[p * C + c], A);
      write_comps<Tv, C>(A, Y, ldy, prow[p], piece, r, alpha, beta);
    }
}

template <class AR, typename Tx, typename Tv, int S>
__device__ inline void sell_tile_q(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                   Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta) {
  constexpr int C = lane_comps<Tx, S>();
  if constexpr (S <= C)  // fewer vectors than a piece holds: only here
    if (s < C) return sell_tile_m<AR, Tx, Tv, S, true>(A, T, X, ldx, Y, ldy, s, alpha, beta);
  sell_tile_m<AR, Tx, Tv, S, false>(A, T, X, ldx, Y, ldy, s, alpha, beta);
}

// ------------------------------- LONG tile ---------------------------------
// Every wave sweeps every fourth chunk of the row, CL lanes to an entry as in
// sell_tile_q (one vector: a lane to an entry); the lanes' sums of a component
// meet through shuffles, the waves' in LDS.
template <class AR, typename Tx, typename Tv, int S, int U, bool SHORT>
__device__ inline void long_tile_m(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                 Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta,
                                 unsigned char* lds) {
  using Acc = typename AR::Acc;
  constexpr uint32_t NW = TILE_THREADS / WAVE;
  constexpr int C = lane_comps<Tx, S>(), CL = S / C, EPP = WAVE / CL;
  const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
  const uint32_t nchunks = (T.ne + WCHUNK - 1) / WCHUNK;
  const uint32_t sub = lane / CL;
  const RowPiece<C> piece(lane % CL, s);
  LaneAcc<AR, C> acc;
  acc.init(A);
  auto words = [&](auto& b, uint32_t ch0) {
    b.load_words(
        [&](int u) -> const u32x4* {
          uint32_t ch = ch0 + u * NW, k = ch * WCHUNK + lane * WIDE;
          return (ch < nchunks && k < T.ne) ? (const u32x4*)(A.ent + T.e0 + k) : nullptr;
        },
        [&](int u) -> uint32_t {
          uint32_t ch = ch0 + u * NW;
          return ch < nchunks ? A.choff[T.c0 + ch] : 0u;
        });
  };
  if constexpr (S == 1) {
    band_terms<AR, Tx, 1>(A, T, acc, T.row0, 0, 1, threadIdx.x, TILE_THREADS, X, ldx, s);
    for (uint32_t ch0 = wave; ch0 < nchunks; ch0 += NW * U) {
      Chunk4<AR, Tx, 1, U> b;
      words(b, ch0);
      b.template load_gathers<false>(A, X, ldx, s);
      b.template accumulate<false>(A, acc);
    }
  } else {
    const uint32_t nd = tile_nd(T.kind);
    for (uint32_t d = threadIdx.x / CL; d < nd; d += TILE_THREADS / CL) {
      const int64_t col = (int64_t)T.row0 + A.boffs[T.boff + d];
      const bool ok = col >= 0 && col < (int64_t)A.ncols;
      const uint32_t v = ok ? ldval<typename AR::ValT>(A.bval, T.b0 + d) : 0u;
      uint32_t xv[C];
      gather_comps<SHORT, Tx, C>(X + (ok ? col : 0) * ldx, piece, xv);
#pragma unroll
      for (int c = 0; c < C; ++c) acc.a[c] += mul_term<AR>(v, xv[c], A.m);
      acc.tick(A);
    }
    for (uint32_t ch = wave; ch < nchunks; ch += NW) {
      Chunk4<AR, Tx, 1, 1> b;
      words(b, ch);
      load_values4<AR>(A, b.w[0], b.vo[0], b.v[0]);
#pragma unroll
      for (int k = 0; k < WIDE; ++k) b.v[0][k] = entry_value(b.w[0][k], b.v[0][k], A.m);
      for (int p = 0; p < CL; ++p) {  // entries 4*(p * EPP + sub) + k of the chunk
        uint32_t w[WIDE], xv[WIDE][C];
        const int src = p * EPP + (int)sub;
#pragma unroll
        for (int k = 0; k < WIDE; ++k) {
          w[k] = CL == 1 ? b.w[0][k] : (uint32_t)__shfl((int)b.w[0][k], src);
          gather_comps<SHORT, Tx, C>(X + (int64_t)(w[k] & COL_MASK) * ldx, piece, xv[k]);
        }
#pragma unroll
        for (int k = 0; k < WIDE; ++k) {
          const uint32_t v = CL == 1 ? b.v[0][k] : (uint32_t)__shfl((int)b.v[0][k], src);
          if ((w[k] >> TAG_SHIFT) == TAG_PAD) continue;
#pragma unroll
          for (int c = 0; c < C; ++c) acc.a[c] += mul_term<AR>(v, xv[k][c], A.m);
          acc.tick(A);
        }
      }
    }
  }
  acc.to_residues(A);
  Acc* red = (Acc*)lds;  // [4 waves][S]
#pragma unroll
  for (int c = 0; c < C; ++c) {
    Acc v = acc.a[c];
    for (int o = WAVE / 2; o >= CL; o >>= 1) v += shfl_xor_acc(v, o, WAVE);
    if (lane < (uint32_t)CL) red[wave * S + lane * C + c] = v;
  }
  __syncthreads();
  if (threadIdx.x < (uint32_t)S && (int)threadIdx.x < s) {
    Acc t = 0;
    for (uint32_t q = 0; q < NW; ++q) t += red[q * S + piece_slot<C>(threadIdx.x, s)];
    uint32_t r = AR::reduce(t, A);
    write_comps<Tv, 1>(A, Y, ldy, T.row0, RowPiece<1>(threadIdx.x, s), &r, alpha, beta);
  }
}

template <class AR, typename Tx, typename Tv, int S, int U>
__device__ inline void long_tile(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                 Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta,
                                 unsigned char* lds) {
  constexpr int C = lane_comps<Tx, S>();
  if constexpr (S > 1 && S <= C)
    if (s < C) return long_tile_m<AR, Tx, Tv, S, U, true>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds);
  long_tile_m<AR, Tx, Tv, S, U, false>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds);
}

// ------------------------------- STREAM tile -------------------------------
// One vector. The tile's terms (value times gathered x) go to LDS; then every
// thread sums an equal run of consecutive terms and adds each row's piece to
// that row's LDS sum with an LDS atomic (exact in any order: integers, or
// integer-valued doubles below 2^53), so one long row inside a tile does not
// serialize on one lane. Row pointers and the band part are loaded first.
template <class AR, typename Tx, typename Tv, int U>
__device__ inline void stream_tile_1(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                     Tv* __restrict__ Y, int64_t ldy, uint32_t alpha, uint32_t beta,
                                     unsigned char* lds) {
  using Prod = typename AR::Prod;
  using Acc = typename AR::Acc;
  constexpr uint32_t NW = TILE_THREADS / WAVE;
  Acc* rowsum = (Acc*)lds;                                 // [256]
  uint32_t* rps = (uint32_t*)(rowsum + TILE_THREADS);     // [257] tile-relative row starts
  Prod* prod = (Prod*)(rps + TILE_THREADS + 4);            // [ne]
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const uint32_t ne = T.ne;
  const uint32_t nchunks = (ne + WCHUNK - 1) / WCHUNK;
  const uint32_t nr = tile_rows(T.kind);
  auto words = [&](Chunk4<AR, Tx, 1, U>& b, uint32_t ch0) {
    b.load_words(
        [&](int u) -> const u32x4* {
          uint32_t ch = ch0 + u * NW, k = ch * WCHUNK + lane * WIDE;
          return (ch < nchunks && k < ne) ? (const u32x4*)(A.ent + T.e0 + k) : nullptr;
        },
        [&](int u) -> uint32_t {
          uint32_t ch = ch0 + u * NW;
          return ch < nchunks ? A.choff[T.c0 + ch] : 0u;
        });
  };
  auto terms = [&](Chunk4<AR, Tx, 1, U>& b, uint32_t ch0) {
    b.template load_gathers<false>(A, X, ldx, 1);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < WIDE; ++k) {
        uint32_t e = (ch0 + u * NW) * WCHUNK + lane * WIDE + k;
        if (e < ne) prod[e] = mul_term<AR>(b.v[u][k], b.xv[u][k][0], A.m);
      }
  };
  // the first batch of entry words is requested before the row pointers and
  // the band part, whose loads then overlap its latency
  Chunk4<AR, Tx, 1, U> first;
  words(first, wave);
  if (tid < nr) rps[tid] = A.rowp[T.aux + tid] - T.e0;
  if (tid == 0) rps[nr] = ne;  // nr may be 256: the sentinel needs its own writer
  if (tid < nr) {
    LaneAcc<AR, 1> band;
    band.init(A);
    band_terms<AR, Tx, 1>(A, T, band, T.row0 + tid, tid, nr, 0, 1, X, ldx, 1);
    band.to_residues(A);
    rowsum[tid] = band.a[0];
  }
  terms(first, wave);  // chunks past the end hold padding words and store nothing
  for (uint32_t ch0 = wave + NW * U; ch0 < nchunks; ch0 += NW * U) {
    Chunk4<AR, Tx, 1, U> b;
    words(b, ch0);
    terms(b, ch0);
  }
  __syncthreads();
  // entry-balanced segmented sum
  const uint32_t per = (ne + TILE_THREADS - 1) / TILE_THREADS;
  const uint32_t p0 = tid * per, p1 = min(ne, p0 + per);
  if (p0 < p1) {
    uint32_t lo = 0, hi = nr;  // last row r with rps[r] <= p0
    while (hi - lo > 1) {
      uint32_t mid = (lo + hi) >> 1;
      if (rps[mid] <= p0) lo = mid;
      else hi = mid;
    }
    uint32_t r = lo, next = rps[r + 1];
    LaneAcc<AR, 1> acc;
    acc.init(A);
    for (uint32_t p = p0; p < p1; ++p) {
      while (p >= next) {
        acc.to_residues(A);
        atomicAdd(&rowsum[r], acc.a[0]);
        acc.init(A);
        next = rps[++r + 1];
      }
      acc.a[0] += prod[p];
      acc.tick(A);
    }
    acc.to_residues(A);
    atomicAdd(&rowsum[r], acc.a[0]);
  }
  __syncthreads();
  if (tid < nr) {
    uint32_t res = AR::reduce(rowsum[tid], A);
    write_row<Tv, 1>(A, Y, ldy, T.row0 + tid, &res, 1, alpha, beta);
  }
}

// LDS of stream_tile_b for a tile of nr rows and ne entries: the rows' sums at 0, then the byte offsets of the row
// starts, the words and the values, which are accessed in sixteens, and the end.
struct StreamLds {
  uint32_t rps, words, values, bytes;
};
template <class AR, int S>
__host__ __device__ inline StreamLds stream_b_lds(uint32_t nr, uint32_t ne) {
  StreamLds l;
  l.rps = (nr * S * (uint32_t)sizeof(typename AR::Acc) + 15u) & ~15u;
  l.words = l.rps + (nr + 4) / 4 * 16;
  l.values = l.words + (ne + 3) / 4 * 16;
  l.bytes = l.values + (ne + 3) / 4 * 16;
  return l;
}

// s > 1 vectors: words and values are staged in LDS, then each group of S / C
// lanes (C components to a lane) takes an equal run of consecutive entries, adds
// up the terms of a row in registers and adds them to the row's sums in LDS
// where the row ends. A tile's time then depends on its entries alone: with a
// lane per row and a kernel of its own for tiles with rows above 64 entries, the
// power-law matrix (1,000,000 rows, s = 8) took 481 us, its longest lanes
// walking 64 entries while most were done after three; now 207 us (17.2 M
// gathers of 32 bytes from all over a 32 MB X: 2.7 TB/s of them, L2 misses).
template <class AR, typename Tx, typename Tv, int S, bool SHORT>
__device__ inline void stream_tile_m(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                     Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta,
                                     unsigned char* lds) {
  using Acc = typename AR::Acc;
  constexpr uint32_t NW = TILE_THREADS / WAVE;
  constexpr int C = lane_comps<Tx, S>(), CL = S / C;
  constexpr uint32_t NG = TILE_THREADS / CL;
  constexpr int EU = C >= 4 || sizeof(Tx) == 8 ? 4 : 8;  // entries of a run whose gathers are in flight together
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const uint32_t ne = T.ne, nr = tile_rows(T.kind);
  const uint32_t nchunks = (ne + WCHUNK - 1) / WCHUNK;
  const StreamLds at = stream_b_lds<AR, S>(nr, ne);
  Acc* rowsum = (Acc*)lds;                        // [nr][S]
  uint32_t* rps = (uint32_t*)(lds + at.rps);      // [nr + 1] tile-relative row starts
  u32x4* sw = (u32x4*)(lds + at.words);           // [ne] words, in fours
  u32x4* sv = (u32x4*)(lds + at.values);          // [ne] values
  const uint32_t grp = tid / CL, slot = tid % CL * C;
  const RowPiece<C> piece(tid % CL, s);
  for (uint32_t ch = wave; ch < nchunks; ch += NW) {
    const uint32_t k = ch * WCHUNK + lane * WIDE;
    const u32x4 q = k < ne ? __builtin_nontemporal_load((const u32x4*)(A.ent + T.e0 + k)) : (u32x4)(PAD_WORD);
    const uint32_t w[WIDE] = {q.x, q.y, q.z, q.w};
    uint32_t v[WIDE];
    load_values4<AR>(A, w, A.choff[T.c0 + ch], v);
    if (k < ne) {
      sw[k / WIDE] = q;
      sv[k / WIDE] = (u32x4){entry_value(w[0], v[0], A.m), entry_value(w[1], v[1], A.m), entry_value(w[2], v[2], A.m),
                             entry_value(w[3], v[3], A.m)};
    }
  }
  if (tid < nr) rps[tid] = A.rowp[T.aux + tid] - T.e0;
  if (tid == 0) rps[nr] = ne;  // nr may be 256: the sentinel needs its own writer
  // the rows' sums start from their band parts
  const uint32_t nd = tile_nd(T.kind);
  for (uint32_t r = grp; r < nr; r += NG) {
    LaneAcc<AR, C> acc;
    acc.init(A);
    constexpr int DB = 4;
    for (uint32_t d0 = 0; d0 < nd; d0 += DB) {
      uint32_t v[DB], xv[DB][C];
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        const bool in = d0 + d < nd;
        const int64_t col = in ? (int64_t)(T.row0 + r) + A.boffs[T.boff + d0 + d] : -1;
        const bool ok = col >= 0 && col < (int64_t)A.ncols;
        v[d] = ok ? ldval<typename AR::ValT>(A.bval, T.b0 + (d0 + d) * nr + r) : 0u;
        gather_comps<SHORT, Tx, C>(X + (ok ? col : 0) * ldx, piece, xv[d]);
      }
#pragma unroll
      for (int d = 0; d < DB; ++d)
        if (d0 + d < nd) {
#pragma unroll
          for (int c = 0; c < C; ++c) acc.a[c] += mul_term<AR>(v[d], xv[d][c], A.m);
          acc.tick(A);
        }
    }
    acc.to_residues(A);
#pragma unroll
    for (int c = 0; c < C; ++c) rowsum[r * S + slot + c] = acc.a[c];
  }
  __syncthreads();
  const uint32_t per = ((ne + NG - 1) / NG + WIDE - 1) / WIDE * WIDE;
  const uint32_t p0 = grp * per, p1 = min(ne, p0 + per);
  auto row_of = [&](uint32_t p, uint32_t lo) {  // last row r >= lo with rps[r] <= p
    uint32_t hi = nr;
#pragma unroll 1
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (rps[mid] <= p) lo = mid;
      else hi = mid;
    }
    return lo;
  };
  // A tile of few entries, in mostly empty rows: an entry to each group, whose walk from row to row would be all of
  // its time (1,000,000 rows with an entry in every fiftieth, m = 65521: 16.5 -> 9.5 us with 2 vectors, 19.1 -> 11.9
  // with 4; ten times as many entries are above this line and take 18.4 and 21.9).
  if (ne <= NG) {
    if (grp < ne && piece.used()) {
      uint32_t xv[C];
      gather_comps<SHORT, Tx, C>(X + (int64_t)(((const uint32_t*)sw)[grp] & COL_MASK) * ldx, piece, xv);
      const uint32_t r = row_of(grp, 0), v = ((const uint32_t*)sv)[grp];
      LaneAcc<AR, C> acc;
      acc.init(A);
#pragma unroll
      for (int c = 0; c < C; ++c) acc.a[c] += mul_term<AR>(v, xv[c], A.m);
      acc.to_residues(A);
#pragma unroll
      for (int c = 0; c < C; ++c) atomicAdd(&rowsum[r * S + slot + c], acc.a[c]);
    }
  } else if (p0 < p1 && piece.used()) {
    uint32_t r = row_of(p0, 0), next = rps[r + 1];
    LaneAcc<AR, C> acc;
    acc.init(A);
    auto flush = [&] {
      acc.to_residues(A);
#pragma unroll
      for (int c = 0; c < C; ++c) atomicAdd(&rowsum[r * S + slot + c], acc.a[c]);
    };
    for (uint32_t p = p0; p < p1; p += EU) {
      uint32_t w[EU], v[EU], xv[EU][C];
#pragma unroll
      for (int e = 0; e < EU; e += WIDE) {
        const bool in = p + e < p1;
        const u32x4 q = in ? sw[(p + e) / WIDE] : (u32x4)(PAD_WORD), z = in ? sv[(p + e) / WIDE] : (u32x4)(0u);
        w[e] = q.x, w[e + 1] = q.y, w[e + 2] = q.z, w[e + 3] = q.w;
        v[e] = z.x, v[e + 1] = z.y, v[e + 2] = z.z, v[e + 3] = z.w;
      }
#pragma unroll
      for (int e = 0; e < EU; ++e) gather_comps<SHORT, Tx, C>(X + (int64_t)(w[e] & COL_MASK) * ldx, piece, xv[e]);
#pragma unroll
      for (int e = 0; e < EU; ++e) {
        if (p + e >= p1) break;
        if (p + e >= next) {
          flush();
          acc.init(A);
          next = rps[++r + 1];
          // past rows without entries, sixteen at a time where there are as many: each row walked is an LDS read that
          // the next one waits for (tiles of 300 and 1 entries in their first and last rows, 256,000 rows, 8 vectors:
          // 37.0 -> 11.7 us; by bisection 9.6, but that cost products over GF(2) without such rows 3%)
          while (p + e >= next) {
            r += r + 16 < nr && rps[r + 16] <= p + e ? 16 : 1;
            next = rps[r + 1];
          }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) acc.a[c] += mul_term<AR>(v[e], xv[e][c], A.m);
        acc.tick(A);
      }
    }
    flush();
  }
  __syncthreads();
  for (uint32_t i = tid; i < nr * S; i += TILE_THREADS) {
    const uint32_t r = i / S, c = i % S;
    if ((int)c >= s) continue;
    const uint32_t row = T.row0 + r, res = AR::reduce(rowsum[r * S + piece_slot<C>(c, s)], A);
    Tv* y = Y + (int64_t)(A.rowmap ? A.rowmap[row] : row) * ldy + c;
    *y = (Tv)((alpha == 1 && beta == 0) ? res : axpby(alpha, res, beta, beta ? (uint32_t)*y : 0u, A.m, A.mu));
  }
}

template <class AR, typename Tx, typename Tv, int S>
__device__ inline void stream_tile_b(const DevMat& A, const Tile& T, const Tx* __restrict__ X, int64_t ldx,
                                     Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta,
                                     unsigned char* lds) {
  constexpr int C = lane_comps<Tx, S>();
  if constexpr (S <= C)  // fewer vectors than a piece holds: only here
    if (s < C) return stream_tile_m<AR, Tx, Tv, S, true>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds);
  stream_tile_m<AR, Tx, Tv, S, false>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds);
}

// ------------------------------- the launch --------------------------------
template <class AR, typename Tx, typename Tv, int S, int U>
__global__ __launch_bounds__(TILE_THREADS) void k_tiles(DevMat A, const Tx* __restrict__ X, int64_t ldx,
                                                        Tv* __restrict__ Y, int64_t ldy, int s, uint32_t alpha,
                                                        uint32_t beta) {
  extern __shared__ __align__(16) unsigned char lds[];
  // a grid larger than the tile table repeats it (per-block timing)
  const Tile T = A.tiles[blockIdx.x % A.ntiles];
  switch (tile_kind(T.kind)) {
    case TK_SELL:
      if constexpr (S == 1) sell_tile<AR, Tx, Tv, 1, 4>(A, T, X, ldx, Y, ldy, s, alpha, beta);
      else sell_tile_q<AR, Tx, Tv, S>(A, T, X, ldx, Y, ldy, s, alpha, beta);
      break;
    case TK_LONG: long_tile<AR, Tx, Tv, S, (S == 1 ? U : 1)>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds); break;
    default:
      if constexpr (S == 1) stream_tile_1<AR, Tx, Tv, U>(A, T, X, ldx, Y, ldy, alpha, beta, lds);
      else stream_tile_b<AR, Tx, Tv, S>(A, T, X, ldx, Y, ldy, s, alpha, beta, lds);
  }
}

template <typename Tv>
__global__ void k_to_u16(const Tv* __restrict__ x, int64_t ldx, uint16_t* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (uint16_t)x[i * ldx];
}

// Contiguous x with 16-byte alignment: eight residues per thread, read with
// 16-byte loads and written with one 16-byte store.
template <typename Tv>
__global__ void k_to_u16_x8(const Tv* __restrict__ x, uint16_t* __restrict__ out, int64_t n) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, base = t * 8;
  if (base + 8 <= n) {
    constexpr int NV = (int)(8 * sizeof(Tv) / 16);  // 16-byte loads per thread
    constexpr int PER = 16 / (int)sizeof(Tv);       // residues per load
    uint32_t r[8];
    const u32x4_t* src = (const u32x4_t*)(x + base);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      u32x4_t q = __builtin_nontemporal_load(src + k);
      if constexpr (PER == 4) {
        r[4 * k] = q.x; r[4 * k + 1] = q.y; r[4 * k + 2] = q.z; r[4 * k + 3] = q.w;
      } else {  // two int64 residues: their low words
        r[2 * k] = q.x; r[2 * k + 1] = q.z;
      }
    }
    u32x4_t o;
    o.x = (r[0] & 0xffffu) | (r[1] << 16);
    o.y = (r[2] & 0xffffu) | (r[3] << 16);
    o.z = (r[4] & 0xffffu) | (r[5] << 16);
    o.w = (r[6] & 0xffffu) | (r[7] << 16);
    *(u32x4_t*)(out + base) = o;
  } else {
    for (int64_t i = base; i < n; ++i) out[i] = (uint16_t)x[i];
  }
}

// Dynamic LDS of one launch over tiles of which the STREAM ones have at most
// max_tile_rows rows and max_tile_entries entries.
template <class AR>
inline size_t tiles_lds_bytes(int64_t max_tile_rows, int64_t max_tile_entries, int S) {
  size_t stream = S == 1 ? TILE_THREADS * sizeof(typename AR::Acc) + (TILE_THREADS + 4) * 4 +
                               (size_t)max_tile_entries * sizeof(typename AR::Prod)
                  : S == 2  ? stream_b_lds<AR, 2>((uint32_t)max_tile_rows, (uint32_t)max_tile_entries).bytes
                  : S == 4  ? stream_b_lds<AR, 4>((uint32_t)max_tile_rows, (uint32_t)max_tile_entries).bytes
                  : S == 8  ? stream_b_lds<AR, 8>((uint32_t)max_tile_rows, (uint32_t)max_tile_entries).bytes
                            : stream_b_lds<AR, 16>((uint32_t)max_tile_rows, (uint32_t)max_tile_entries).bytes;
  size_t red = (size_t)(TILE_THREADS / WAVE) * S * sizeof(typename AR::Acc);
  size_t b = stream > red ? stream : red;
  return b < 16 ? 16 : b;
}

// Unroll of the one-vector STREAM/LONG paths: every chunk of a tile in one batch.
inline int unroll_for(int64_t max_tile_entries) {
  int64_t per_wave = (max_tile_entries + (int64_t)WCHUNK * (TILE_THREADS / WAVE) - 1) / ((int64_t)WCHUNK * (TILE_THREADS / WAVE));
  return per_wave <= 1 ? 1 : per_wave <= 2 ? 2 : 4;
}

template <class AR, typename Tx, typename Tv, int U>
static void launch_s1(const DevMat& A, dim3 grid, size_t lds, const Tx* x, int64_t ldx, Tv* y, int64_t ldy,
                      uint32_t alpha, uint32_t beta, hipStream_t st) {
  hipLaunchKernelGGL((k_tiles<AR, Tx, Tv, 1, U>), grid, dim3(TILE_THREADS), lds, st, A, x, ldx, y, ldy, 1, alpha,
                     beta);
}

// The most dynamic LDS of a multi-vector launch: 256 rows and 4,096 entries of 16 vectors.
template <class AR, typename Tv>
hipError_t raise_tiles_lds(int S) {
  const int most = (int)tiles_lds_bytes<AR>(TILE_THREADS, 4096, S);
  switch (S) {
    case 2: return raise_lds_limit((const void*)k_tiles<AR, Tv, Tv, 2, 4>, most);
    case 4: return raise_lds_limit((const void*)k_tiles<AR, Tv, Tv, 4, 4>, most);
    case 8: return raise_lds_limit((const void*)k_tiles<AR, Tv, Tv, 8, 4>, most);
    default: return raise_lds_limit((const void*)k_tiles<AR, Tv, Tv, 16, 4>, most);
  }
}

// What the tiles read as X. A one-vector tile's padding gathers element 0 with the value 0, and a matrix without
// columns has tiles (its rows are all padding) but no such element: X is empty and may be null, so the tile table
// stands in for it.
inline const void* readable_x(const DevMat& A, const void* X) { return A.ncols ? X : (const void*)A.tiles; }

// x16: when not null, a 16-bit copy of the one vector (s must be 1)
template <class AR, typename Tv>
hipError_t launch_tiles_t(const DevMat& A, int64_t max_tile_entries, const void* X, int64_t ldx, void* Y, int64_t ldy,
                          int s, uint32_t alpha, uint32_t beta, hipStream_t st, const uint16_t* x16,
                          uint32_t nblocks = 0) {
  if (A.ntiles == 0) return hipSuccess;
  const int S = s <= 1 ? 1 : s <= 2 ? 2 : s <= 4 ? 4 : s <= 8 ? 8 : 16;
  size_t lds = tiles_lds_bytes<AR>(A.max_tile_rows, max_tile_entries, S);
  if (lds > 64 * 1024) {
    hipError_t e = raise_tiles_lds<AR, Tv>(S);
    if (e != hipSuccess) return e;
  }
  dim3 grid(nblocks ? nblocks : A.ntiles), block(TILE_THREADS);
  const Tv* x = (const Tv*)readable_x(A, X);
  Tv* y = (Tv*)Y;
  if (S == 1) {
    const int U = unroll_for(max_tile_entries);
    if (x16) {
      if (U == 1) launch_s1<AR, uint16_t, Tv, 1>(A, grid, lds, x16, 1, y, ldy, alpha, beta, st);
      else if (U == 2) launch_s1<AR, uint16_t, Tv, 2>(A, grid, lds, x16, 1, y, ldy, alpha, beta, st);
      else launch_s1<AR, uint16_t, Tv, 4>(A, grid, lds, x16, 1, y, ldy, alpha, beta, st);
    } else {
      if (U == 1) launch_s1<AR, Tv, Tv, 1>(A, grid, lds, x, ldx, y, ldy, alpha, beta, st);
      else if (U == 2) launch_s1<AR, Tv, Tv, 2>(A, grid, lds, x, ldx, y, ldy, alpha, beta, st);
      else launch_s1<AR, Tv, Tv, 4>(A, grid, lds, x, ldx, y, ldy, alpha, beta, st);
    }
    return hipGetLastError();
  }
  switch (S) {
    case 2: hipLaunchKernelGGL((k_tiles<AR, Tv, Tv, 2, 4>), grid, block, lds, st, A, x, ldx, y, ldy, s, alpha, beta); break;
    case 4: hipLaunchKernelGGL((k_tiles<AR, Tv, Tv, 4, 4>), grid, block, lds, st, A, x, ldx, y, ldy, s, alpha, beta); break;
    case 8: hipLaunchKernelGGL((k_tiles<AR, Tv, Tv, 8, 4>), grid, block, lds, st, A, x, ldx, y, ldy, s, alpha, beta); break;
    default: hipLaunchKernelGGL((k_tiles<AR, Tv, Tv, 16, 4>), grid, block, lds, st, A, x, ldx, y, ldy, s, alpha, beta); break;
  }
  return hipGetLastError();
}

// 16-bit copy of one vector (residues < 65536), for the compact-x path.
template <typename Tv>
hipError_t launch_to_u16(const void* X, int64_t ldx, uint16_t* out, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (ldx == 1 && ((uintptr_t)X & 15) == 0 && ((uintptr_t)out & 15) == 0) {
    int64_t threads = (n + 7) / 8;
    hipLaunchKernelGGL((k_to_u16_x8<Tv>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, (const Tv*)X,
                       out, n);
    return hipGetLastError();
  }
  int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL((k_to_u16<Tv>), dim3(blocks), dim3(256), 0, st, (const Tv*)X, ldx, out, n);
  return hipGetLastError();
}

}  // namespace ffx
