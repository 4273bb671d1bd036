// Tile kernels over GF(2) with bit-packed blocks of 32-bit words.
#include "launch.h"
#include "tiles.h"

namespace ffx {
hipError_t launch_tiles_gf2(const DevMat& A, int64_t mte, const void* X, int64_t ldx, void* Y, int64_t ldy, int w,
                            hipStream_t st) {
  // words are moved as int32 bit patterns: conversions to and from uint32 keep every bit
  return launch_tiles_t<ArGF2, int32_t>(A, mte, X, ldx, Y, ldy, w, 1, 0, st, nullptr, 0);
}
}  // namespace ffx

// ------------------------------------------------------------------------
// Block-Wiedemann sequence over GF(2) with packed blocks (Section 3, step 1,
// with the GF(2) compression of Section 4): S_i = U^T A^i V for 32w vectors.
// S_i is a 32w x 32w bit matrix; its row a is w words, bit b of word c being
// entry (a, 32c + b), the parity of the rows j where bit a of U[j] and bit b of
// word c of (A^i V)[j] are both set.
//
// One launch per iteration i: workgroup t < ntiles computes its tile's rows of
// W_{i+1} = A W_i (the product's tile code); one workgroup per 256 rows computes
// their XOR share of U^T W_i, a partial of 32w*w words; GF2_NMID workgroups fold
// the partials of W_{i-1} (written by the previous launch) into GF2_NMID words
// per pair, and one workgroup folds those of iteration i-2 into S_{i-2}. Partials
// and folds are double-buffered by parity.
//
// The product waits for the L2's answers to its gathers and the projection keeps
// the vector ALU and LDS busy, so they run in workgroups of their own, side by
// side: 200,000 rows of 15 entries, w = 2: 30.3 us per iteration with each
// workgroup doing the projection of its tile after its product, 23.8 us now.
namespace ffx {

constexpr uint32_t GF2_NMID = 64;

struct Gf2SeqArgs {
  const uint32_t* U;   // n x w words
  uint32_t* W[2];      // W_i in W[i & 1]; n x w words
  uint32_t* part[2];   // [ntiles][npairs], by parity
  uint32_t* mid[2];    // [GF2_NMID][npairs], by parity
  uint32_t* S;         // L x npairs
  uint32_t* Wlast;     // W_L (or null)
  int64_t L;
  int32_t w;
};

// out[a*w + c]: XOR over the nr <= 256 rows from r0 on of (bit a of U[row]) * W[row][c]. The rows of U and
// W are staged in LDS (su: w words to a row, sw: S, those past w zero); a lane takes one bit a and all of
// W's words, so a row costs two reads, one bit extraction and an and-xor per word, and where there are
// fewer than 256 bits, groups of lanes take every ngrp-th row each.
template <int S>
__device__ inline void rows_projection_gf2(const uint32_t* __restrict__ U, const uint32_t* __restrict__ W, int64_t r0,
                                           int nr, int w, uint32_t* sh, uint32_t* __restrict__ out) {
  struct alignas(S >= 4 ? 16 : 8) Words { uint32_t x[S]; };
  const int tid = threadIdx.x, nbits = 32 * w;
  uint32_t* su = sh;
  Words* sw = (Words*)(sh + TILE_THREADS * w);
  for (int k = tid; k < nr * w; k += TILE_THREADS) su[k] = U[r0 * w + k];
  for (int k = tid; k < nr * S; k += TILE_THREADS) {
    const int c = k % S;
    ((uint32_t*)sw)[k] = c < w ? W[(r0 + k / S) * w + c] : 0u;
  }
  __syncthreads();
  const int ngrp = nbits < TILE_THREADS ? TILE_THREADS / nbits : 1, grp = nbits < TILE_THREADS ? tid / nbits : 0;
  auto bit_words = [&](int a, uint32_t* acc) {
    const int ua = a >> 5, ub = a & 31;
#pragma unroll
    for (int c = 0; c < S; ++c) acc[c] = 0u;
#pragma unroll 4
    for (int q = grp; q < nr; q += ngrp) {
      const uint32_t on = (uint32_t)((int32_t)(su[q * w + ua] << (31 - ub)) >> 31);  // all ones where the bit is set
      const Words x = sw[q];
#pragma unroll
      for (int c = 0; c < S; ++c) acc[c] ^= on & x.x[c];
    }
  };
  if (nbits >= TILE_THREADS) {
    for (int a = tid; a < nbits; a += TILE_THREADS) {
      uint32_t acc[S];
      bit_words(a, acc);
#pragma unroll
      for (int c = 0; c < S; ++c)
        if (c < w) out[a * w + c] = acc[c];
    }
    return;
  }
  uint32_t acc[S];
  const int a = tid - grp * nbits;
  if (grp < ngrp) bit_words(a, acc);
  __syncthreads();  // the sums take the place of the rows of W
  if (grp < ngrp) {
    Words v;
#pragma unroll
    for (int c = 0; c < S; ++c) v.x[c] = acc[c];
    sw[tid] = v;
  }
  __syncthreads();
  for (int p = tid; p < nbits * w; p += TILE_THREADS) {
    uint32_t x = 0;
    for (int g = 0; g < ngrp; ++g) x ^= sw[g * nbits + p / w].x[p % w];
    out[p] = x;
  }
}

// LDS of rows_projection_gf2.
inline size_t gf2_projection_lds(int w, int S) { return (size_t)TILE_THREADS * (w + S) * sizeof(uint32_t); }
// Workgroups of the projection.
inline uint32_t gf2_projection_blocks(const DevMat& A) { return (A.nrows + TILE_THREADS - 1) / TILE_THREADS; }

// XOR of part[g][p] over g = first, first + stride, ... < nparts, for every pair p.
__device__ inline void fold_xor(const uint32_t* __restrict__ part, uint32_t first, uint32_t stride, uint32_t nparts,
                                int npairs, uint32_t* __restrict__ out) {
  for (int p = threadIdx.x; p < npairs; p += TILE_THREADS) {
    uint32_t x = 0;
    for (uint32_t g = first; g < nparts; g += stride) x ^= part[(int64_t)g * npairs + p];
    out[p] = x;
  }
}

// Iteration i < L, and i = L for the folds that are left.
template <int S>
__global__ __launch_bounds__(TILE_THREADS) void k_seq_step_gf2(DevMat A, Gf2SeqArgs q, int64_t i) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int w = q.w, npairs = 32 * w * w;
  const uint32_t nt = A.ntiles, np = (A.nrows + TILE_THREADS - 1) / TILE_THREADS;
  const bool last = i + 1 == q.L;
  if (blockIdx.x >= nt + np) {
    const uint32_t r = blockIdx.x - nt - np;
    if (r < GF2_NMID) {
      if (i > 0) fold_xor(q.part[(i - 1) & 1], r, GF2_NMID, np, npairs, q.mid[(i - 1) & 1] + (int64_t)r * npairs);
    } else if (i > 1) {
      fold_xor(q.mid[i & 1], 0, 1, GF2_NMID, npairs, q.S + (i - 2) * (int64_t)npairs);
    }
  } else if (i == q.L) {
    return;
  } else if (blockIdx.x >= nt) {
    const uint32_t r = blockIdx.x - nt, r0 = r * TILE_THREADS;
    rows_projection_gf2<S>(q.U, q.W[i & 1], r0, (int)min((uint32_t)TILE_THREADS, A.nrows - r0), w, (uint32_t*)lds,
                           q.part[i & 1] + (int64_t)r * npairs);
  } else if (!last || q.Wlast) {
    const int32_t* X = (const int32_t*)q.W[i & 1];
    int32_t* Y = (int32_t*)(last ? q.Wlast : q.W[(i + 1) & 1]);
    const Tile T = A.tiles[blockIdx.x];
    switch (tile_kind(T.kind)) {
      case TK_SELL: sell_tile_q<ArGF2, int32_t, int32_t, S>(A, T, X, w, Y, w, w, 1, 0); break;
      case TK_LONG: long_tile<ArGF2, int32_t, int32_t, S, 1>(A, T, X, w, Y, w, w, 1, 0, lds); break;
      default: stream_tile_b<ArGF2, int32_t, int32_t, S>(A, T, X, w, Y, w, w, 1, 0, lds);
    }
  }
}

// S_{L-1} from the folds of the last iteration.
__global__ __launch_bounds__(TILE_THREADS) void k_seq_finish_gf2(Gf2SeqArgs q) {
  const int npairs = 32 * q.w * q.w;
  fold_xor(q.mid[(q.L - 1) & 1], 0, 1, GF2_NMID, npairs, q.S + (q.L - 1) * (int64_t)npairs);
}

size_t gf2_sequence_part_words(const DevMat& A, int w) {
  return 2 * ((size_t)gf2_projection_blocks(A) + GF2_NMID) * 32 * w * w;
}

hipError_t launch_sequence_gf2(const DevMat& A, int64_t mte, int w, const uint32_t* U, const uint32_t* W0, int64_t L,
                               uint32_t* S, uint32_t* w1, uint32_t* part, uint32_t* Wlast, hipStream_t st) {
  if (L <= 0) return hipSuccess;
  if (A.ntiles == 0) return hipErrorInvalidValue;  // every row lies in a tile, so n > 0 means tiles
  const int npairs = 32 * w * w;
  const size_t pw = (size_t)gf2_projection_blocks(A) * npairs, mw = (size_t)GF2_NMID * npairs;
  Gf2SeqArgs q;
  q.U = U;
  q.W[0] = const_cast<uint32_t*>(W0);
  q.W[1] = w1;
  q.part[0] = part;
  q.part[1] = part + pw;
  q.mid[0] = part + 2 * pw;
  q.mid[1] = part + 2 * pw + mw;
  q.S = S;
  q.Wlast = Wlast;
  q.L = L;
  q.w = w;
  const int S_ = w <= 2 ? 2 : w <= 4 ? 4 : w <= 8 ? 8 : 16;  // the multi-vector tiles, as for residues
  size_t lds = tiles_lds_bytes<ArGF2>(A.max_tile_rows, mte, S_);
  const size_t plds = gf2_projection_lds(w, S_);
  if (lds < plds) lds = plds;
  const dim3 g(A.ntiles + gf2_projection_blocks(A) + GF2_NMID + 1), b(TILE_THREADS);
  for (int64_t i = 0; i <= L; ++i) {
    switch (S_) {
      case 2: hipLaunchKernelGGL((k_seq_step_gf2<2>), g, b, lds, st, A, q, i); break;
      case 4: hipLaunchKernelGGL((k_seq_step_gf2<4>), g, b, lds, st, A, q, i); break;
      case 8: hipLaunchKernelGGL((k_seq_step_gf2<8>), g, b, lds, st, A, q, i); break;
      default: hipLaunchKernelGGL((k_seq_step_gf2<16>), g, b, lds, st, A, q, i); break;
    }
  }
  hipLaunchKernelGGL(k_seq_finish_gf2, dim3(1), dim3(TILE_THREADS), 0, st, q);
  return hipGetLastError();
}

}  // namespace ffx
