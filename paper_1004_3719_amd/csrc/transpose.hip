// Y = alpha*A^T*X + beta*Y without a stored A^T (paper Section 4 notes that A
// and A^T may not fit together): every entry A[i,j] adds its terms
// A[i,j]*X[i][c] to the sum of output row j. Sums are 64-bit integers, exact in
// any order: for m <= 65536 a term is below 2^32 and there are at most 2^32
// entries; for m = 2^31 - 1 a product folds below 2^32; for other m each term
// is reduced mod m first.
//
// What bounds it: a global atomic. MI355X takes about 23 G atomic
// transactions/s whatever the table (80 KB to 16 MB), the scope or the width,
// a transaction being the lanes of one instruction that fall in one 64-byte
// piece of memory. Two forms:
//  - binned (launch_binned): no global atomics. The entries of a batch of at
//    most 2,048 are sorted in LDS by output panel, and a second kernel, one
//    workgroup per panel and part of the batches, adds the records of its
//    panel to sums in LDS. An entry costs 8 bytes written and 8 bytes read.
//    One vector, 1,000,000 power-law rows (17.2 M entries): 577 us scattered,
//    167 us binned; four vectors, 100,000 rows of 15: 276 us with an atomic per
//    entry and vector, 44 us binned.
//  - scattered (k_scatter_t): one 64-bit atomic per entry and vector, with the
//    s sums of an output row side by side in adjacent lanes, so an entry costs
//    ceil(s/8) transactions and not s. For small products, very wide ones, few
//    diagonals and batches that leave few records to a panel (t_plan).
#include <algorithm>

#include "launch.h"
#include "tiles.h"

namespace ffx {

// the value type of the stored entries (all that load_values4 needs to know)
template <typename V>
struct ValsOf {
  using ValT = V;
};

// arithmetic of one term
enum TKind { TM_SMALL, TM_BIG, TM_M31 };
template <int K>
using TVal = typename std::conditional<K == TM_SMALL, uint16_t, uint32_t>::type;

// v*x as a term below 2^32
template <int K>
__device__ inline uint32_t tterm(uint32_t v, uint32_t x, const DevMat& A) {
  if constexpr (K == TM_SMALL) return v * x;
  else if constexpr (K == TM_M31) return (uint32_t)ArM31::mul(v, x);
  else return mod_u64((uint64_t)v * x, A.m, A.mu);
}
// the value of an entry word (its stored value v when the entry is general)
__device__ inline uint32_t tvalue(uint32_t w, uint32_t v, uint32_t m) {
  const uint32_t tag = w >> TAG_SHIFT;
  return tag == TAG_GEN ? v : tag == TAG_PLUS ? 1u : m - 1;
}

// Four consecutive entry words of one wave's chunk of 256 and their values and
// row slots: chunk ch of a tile of any format (a STREAM or LONG tile's runs of
// 256 entries; a SELL tile's 4-column groups, slice after slice). rps: the
// tile-relative row starts of a STREAM tile, in LDS. Called by whole waves.
template <typename V>
__device__ inline void load_chunk(const DevMat& A, const Tile& T, uint32_t ch, uint32_t lane, const uint32_t* rps,
                                  uint32_t* w, uint32_t* v, uint32_t* slot) {
  const uint32_t kind = tile_kind(T.kind);
  const uint32_t e = ch * WCHUNK + lane * WIDE;
  u32x4 q = (u32x4)(PAD_WORD);
  if (kind == TK_SELL || e < T.ne) q = __builtin_nontemporal_load((const u32x4*)(A.ent + T.e0 + e));
  w[0] = q.x;
  w[1] = q.y;
  w[2] = q.z;
  w[3] = q.w;
  load_values4<ValsOf<V>>(A, w, A.choff[T.c0 + ch], v);
  if (kind == TK_SELL) {
    uint32_t slice = 0, off = 0;
    for (uint32_t k = 0; k + 1 < T.ne; ++k) {
      off += A.swidth[T.aux + k];
      slice += ch >= off ? 1u : 0u;
    }
#pragma unroll
    for (int k = 0; k < WIDE; ++k) slot[k] = slice * WAVE + lane;
  } else if (kind == TK_LONG) {
#pragma unroll
    for (int k = 0; k < WIDE; ++k) slot[k] = 0;
  } else {
    // the last row whose start is <= e + k, by bisection also from one entry to the next: a walk over empty rows
    // is a chain of LDS reads (a band with a few entries beside it: 25 us for 255 rows)
    const uint32_t nr = tile_rows(T.kind);
    uint32_t lo = 0;
#pragma unroll
    for (int k = 0; k < WIDE; ++k) {
      if (e + k < T.ne && (k == 0 || (lo + 1 < nr && rps[lo + 1] <= e + k))) {
        uint32_t hi = nr;
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (rps[mid] <= e + k) lo = mid;
          else hi = mid;
        }
      }
      slot[k] = lo;
    }
  }
}

__device__ inline void load_rps(const DevMat& A, const Tile& T, uint32_t* rps) {
  if (tile_kind(T.kind) == TK_STREAM)
    for (uint32_t r = threadIdx.x; r < tile_rows(T.kind); r += blockDim.x) rps[r] = A.rowp[T.aux + r] - T.e0;
}

// Row of a slot (>= nrows for a padding slot of a SELL tile).
__device__ inline uint32_t slot_row(const DevMat& A, const Tile& T, uint32_t slot) {
  return (tile_kind(T.kind) == TK_SELL && (T.kind & TF_SORTED)) ? A.perm[T.row0 + slot] : T.row0 + slot;
}

// ------------------------------------------------------------- scattered ---
// Lane (e, c) of a wave adds component c of entry e, SP lanes per entry (SP a
// power of two >= s); the sums of output row j are acc[j*st .. j*st + s), with
// st = SP so that the SP lanes of an entry make one transaction (SP <= 8). Random rows of
// four 64-bit sums take 92 G additions/s this way and 23 G/s when one lane
// adds the four in turn.
template <int K, typename Tv, int SP>
__global__ __launch_bounds__(TILE_THREADS) void k_scatter_t(DevMat A, const Tv* __restrict__ X, int64_t ldx, int s, int st,
                                                            unsigned long long* __restrict__ acc) {
  __shared__ uint32_t rps[TILE_THREADS];
  const Tile T = A.tiles[blockIdx.x];
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const uint32_t kind = tile_kind(T.kind);
  const uint32_t comp = lane % SP, sub = lane / SP;
  load_rps(A, T, rps);
  __syncthreads();
  uint32_t nchunks = 0;
  if (kind == TK_SELL)
    for (uint32_t k = 0; k < T.ne; ++k) nchunks += A.swidth[T.aux + k];
  else nchunks = (T.ne + WCHUNK - 1) / WCHUNK;
  for (uint32_t ch = wave; ch < nchunks; ch += TILE_THREADS / WAVE) {
    uint32_t w[WIDE], v[WIDE], slot[WIDE];
    load_chunk<TVal<K>>(A, T, ch, lane, rps, w, v, slot);
#pragma unroll
    for (int k = 0; k < WIDE; ++k) {
      const uint32_t row = slot_row(A, T, slot[k]);
      auto pass = [&](int p, uint32_t& wp, uint32_t& vp, uint32_t& rp) {  // entry, value and row of pass p
        const int src = p * (WAVE / SP) + (int)sub;
        wp = SP == 1 ? w[k] : (uint32_t)__shfl((int)w[k], src);
        vp = SP == 1 ? v[k] : (uint32_t)__shfl((int)v[k], src);
        rp = SP == 1 ? row : (uint32_t)__shfl((int)row, src);
        return (wp >> TAG_SHIFT) != TAG_PAD && rp < A.nrows && (int)comp < s;
      };
      auto term = [&](uint32_t wp, uint32_t vp, uint32_t rp) {
        return tterm<K>(tvalue(wp, vp, A.m), (uint32_t)X[(int64_t)rp * ldx + comp], A);
      };
      auto add = [&](uint32_t wp, uint32_t t) {
        atomicAdd(&acc[(int64_t)(wp & COL_MASK) * st + comp], (unsigned long long)t);
      };
      if constexpr (SP <= 4) {
        // every pass's load of x before the first atomic, which would keep it behind (300 rows of 10, 3 vectors: 27 us,
        // now 21); with 16 lanes to an entry that is slower (1,000,000 rows with three entries in every tenth, 12
        // vectors: 139 us and 107)
        uint32_t wp[SP], t[SP];
        bool on[SP];
#pragma unroll
        for (int p = 0; p < SP; ++p) {
          uint32_t vp, rp;
          on[p] = pass(p, wp[p], vp, rp);
          t[p] = on[p] ? term(wp[p], vp, rp) : 0u;
        }
#pragma unroll
        for (int p = 0; p < SP; ++p)
          if (on[p]) add(wp[p], t[p]);
      } else {
#pragma unroll
        for (int p = 0; p < SP; ++p) {
          uint32_t wp, vp, rp;
          if (pass(p, wp, vp, rp)) add(wp, term(wp, vp, rp));
        }
      }
    }
  }
  // band part: SP lanes per row, whose x stays in a register, and the values of DB diagonals in flight together
  constexpr uint32_t DB = 8;
  const uint32_t nd = tile_nd(T.kind), rows = tile_rows(T.kind);
  for (uint32_t slot = tid / SP; nd && slot < rows; slot += TILE_THREADS / SP) {
    const uint32_t row = slot_row(A, T, slot);
    if (row >= A.nrows || (int)comp >= s) continue;
    const uint32_t x = (uint32_t)X[(int64_t)row * ldx + comp];
    for (uint32_t d0 = 0; d0 < nd; d0 += DB) {
      uint32_t v[DB];
#pragma unroll
      for (uint32_t d = 0; d < DB; ++d)
        v[d] = d0 + d < nd ? ldval<TVal<K>>(A.bval, T.b0 + (d0 + d) * rows + slot) : 0u;
#pragma unroll
      for (uint32_t d = 0; d < DB; ++d)
        if (v[d])  // an absent entry may lie outside the matrix
          atomicAdd(&acc[((int64_t)row + A.boffs[T.boff + d0 + d]) * st + comp], (unsigned long long)tterm<K>(v[d], x, A));
    }
  }
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

template <typename Tv>
__device__ inline void finish_row(uint32_t m, uint64_t mu, uint64_t sum, uint32_t alpha, uint32_t beta, Tv* y) {
  const uint32_t r = mod_u64(sum, m, mu);
  const uint32_t yo = beta ? (uint32_t)*y : 0u;
  *y = (Tv)((alpha == 1 && beta == 0) ? r : axpby(alpha, r, beta, yo, m, mu));
}

template <typename Tv>
__global__ void k_finish_t(DevMat A, const unsigned long long* __restrict__ acc, int64_t n, int s, int sp,
                           uint32_t alpha, uint32_t beta, Tv* __restrict__ Y, int64_t ldy) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n * s; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = i / s;
    const int c = (int)(i - j * s);
    finish_row(A.m, A.mu, acc[j * sp + c], alpha, beta, Y + j * ldy + c);
  }
}

// ---------------------------------------------------------------- binned ---
// First kernel: one workgroup per batch (at most TB_MAX entries of one tile,
// TBatch). Each entry takes its place behind the entries of its panel seen so
// far (an LDS counter per panel of 2^sh output rows), the counts are summed,
// and the records leave through LDS in panel order, so the batch is written
// coalesced; off[b][p] is where panel p starts in it. A record is (term,
// column in the panel) for one vector and (value, row slot << 16 | column in
// the panel) for several.
constexpr int TB_EPT = TB_MAX / TILE_THREADS;  // entries per thread
constexpr int TB_MAXP = 256;                   // panels

template <int K, typename Tv, bool TERM>
__global__ __launch_bounds__(TILE_THREADS) void k_t_bin(DevMat A, const Tv* __restrict__ X, int64_t ldx, uint32_t sh,
                                                        uint32_t P, uint2* __restrict__ rec,
                                                        uint16_t* __restrict__ off) {
  __shared__ __align__(16) uint2 srec[TB_MAX];  // leaves two records to a 16-byte store
  __shared__ uint32_t rps[TILE_THREADS];
  __shared__ uint32_t cnt[TB_MAXP];
  __shared__ uint32_t wsum[TILE_THREADS / WAVE];
  const TBatch B = A.tbatch[blockIdx.x];
  const Tile T = A.tiles[B.tile];
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  cnt[tid] = 0;
  load_rps(A, T, rps);
  __syncthreads();
  uint32_t col[TB_EPT], r0[TB_EPT], r1[TB_EPT];  // column (or ~0), record word 0, row slot and place in the panel
  const uint32_t cmask = (1u << sh) - 1;
  if (!(B.n & TB_BAND)) {
#pragma unroll
    for (int u = 0; u < TB_EPT / WIDE; ++u) {
      const uint32_t ch = u * (TILE_THREADS / WAVE) + wave;
      uint32_t w[WIDE], v[WIDE], slot[WIDE];
      const bool on = ch < B.n;  // the same in the whole wave
      if (on) load_chunk<TVal<K>>(A, T, B.first + ch, lane, rps, w, v, slot);
#pragma unroll
      for (int k = 0; k < WIDE; ++k) {
        const int e = u * WIDE + k;
        col[e] = 0xFFFFFFFFu;
        if (!on || (w[k] >> TAG_SHIFT) == TAG_PAD) continue;
        col[e] = w[k] & COL_MASK;
        r0[e] = tvalue(w[k], v[k], A.m);
        if constexpr (TERM) r0[e] = tterm<K>(r0[e], (uint32_t)X[(int64_t)slot_row(A, T, slot[k]) * ldx], A);
        r1[e] = slot[k] << 16;
      }
    }
  } else {
    const uint32_t nd = B.n & ~TB_BAND, rows = tile_rows(T.kind);
#pragma unroll
    for (int e = 0; e < TB_EPT; ++e) {
      const uint32_t q = e * TILE_THREADS + tid;
      col[e] = 0xFFFFFFFFu;
      if (q >= rows * nd) continue;
      const uint32_t d = B.first + q / rows, slot = q % rows;
      const uint32_t row = slot_row(A, T, slot);
      const uint32_t v = ldval<TVal<K>>(A.bval, T.b0 + d * rows + slot);
      if (!v || row >= A.nrows) continue;
      col[e] = (uint32_t)((int64_t)row + A.boffs[T.boff + d]);
      r0[e] = v;
      if constexpr (TERM) r0[e] = tterm<K>(v, (uint32_t)X[(int64_t)row * ldx], A);
      r1[e] = slot << 16;
    }
  }
#pragma unroll
  for (int e = 0; e < TB_EPT; ++e)
    if (col[e] != 0xFFFFFFFFu) r1[e] |= atomicAdd(&cnt[col[e] >> sh], 1u);  // place < TB_MAX
  __syncthreads();
  // panel starts: an exclusive scan of the counts, one panel per thread
  uint32_t c = cnt[tid], x = c;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, o);
    if ((int)lane >= o) x += y;
  }
  if (lane == WAVE - 1) wsum[wave] = x;
  __syncthreads();
  uint32_t total = 0;
#pragma unroll
  for (uint32_t k = 0; k < TILE_THREADS / WAVE; ++k) {
    if (k < wave) x += wsum[k];
    total += wsum[k];
  }
  cnt[tid] = x - c;
  if (tid < P) off[(size_t)blockIdx.x * (P + 1) + tid] = (uint16_t)(x - c);
  if (tid == 0) off[(size_t)blockIdx.x * (P + 1) + P] = (uint16_t)total;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < TB_EPT; ++e)
    if (col[e] != 0xFFFFFFFFu) {
      const uint32_t at = cnt[col[e] >> sh] + (r1[e] & 0xFFFFu);
      srec[at] = make_uint2(r0[e], (TERM ? 0u : r1[e] & 0xFFFF0000u) | (col[e] & cmask));
    }
  __syncthreads();
  // rec0 is even: two records per 16-byte store (the last may write one past the batch's records,
  // inside its room, which is rounded up to even)
  for (uint32_t i = 2 * tid; i < total; i += 2 * TILE_THREADS)
    *(u32x4*)(rec + B.rec0 + i) = *(const u32x4*)(srec + i);
}

// Second kernel: workgroup (p, q) adds the records of panel p of the batches of
// part q to its sums in LDS, SP sums per output row, and writes them as
// residues to part[q]. A batch's run of records of one panel is anything from
// none (a banded or blocked matrix) to all of its records, so the runs of up to
// 1,024 batches are cut into pieces of at most TA_PIECE records, listed in LDS,
// and the groups of lanes take pieces in turn (with one run per group of lanes
// a band of 33 diagonals, 8 vectors, took 391 us).
constexpr int TA_THREADS = 1024;
constexpr int TA_LIST = 4096;  // pieces listed at a time
template <int SP>
constexpr int ta_lanes() { return SP == 1 ? 16 : SP == 2 ? 32 : 64; }  // lanes that share a piece
template <int SP>
constexpr int ta_unroll() { return SP >= 8 ? 8 : 4; }                  // records in flight per lane
template <int SP>
constexpr int ta_piece() { return ta_lanes<SP>() / SP * ta_unroll<SP>(); }
// dynamic LDS: the sums, then per batch its first record, its row base and its number of records, the list of
// pieces and the wave sums of the scan
constexpr size_t TA_LDS_FIXED = (size_t)TA_THREADS * 12 + TA_LIST * 4 + 64;

template <int K, typename Tv, int SP>
__global__ __launch_bounds__(TA_THREADS) void k_t_acc(DevMat A, const Tv* __restrict__ X, int64_t ldx, int s,
                                                      uint32_t nb, uint32_t sh, uint32_t P, uint32_t Q,
                                                      const uint2* __restrict__ rec, const uint16_t* __restrict__ off,
                                                      uint32_t* __restrict__ part) {
  extern __shared__ __align__(16) unsigned long long sums[];
  uint32_t* first = (uint32_t*)(sums + ((size_t)SP << sh));
  uint32_t* rbase = first + TA_THREADS;  // first row (bit 31 clear), or first slot in perm with bit 31 set
  uint32_t* count = rbase + TA_THREADS;
  uint32_t* list = count + TA_THREADS;
  uint32_t* wsum = list + TA_LIST;
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const uint32_t p = blockIdx.x % P, q = blockIdx.x / P;
  const uint32_t j0 = p << sh, nj = min(1u << sh, A.ncols - j0);
  for (uint32_t i = tid; i < nj * SP; i += TA_THREADS) sums[i] = 0;
  constexpr uint32_t GL = ta_lanes<SP>(), EPI = GL / SP, NG = TA_THREADS / GL, PS = ta_piece<SP>();
  constexpr int U = ta_unroll<SP>();
  const uint32_t grp = tid / GL, sub = tid % GL / SP, comp = tid % SP;
  // part q takes the batches b = q (mod Q): the batches of a narrow band meet few panels each, and
  // this way a panel's batches fall in all of its parts
  for (uint32_t base = q; base < nb; base += TA_THREADS * Q) {
    const uint32_t b = base + Q * tid;
    uint32_t np = 0;
    if (b < nb) {
      const uint16_t* o = off + (size_t)b * (P + 1) + p;
      const uint32_t i0 = o[0], n = o[1] - i0;
      const TBatch B = A.tbatch[b];
      first[tid] = B.rec0 + i0;
      count[tid] = n;
      np = (n + PS - 1) / PS;
      if constexpr (SP > 1) {
        const Tile T = A.tiles[B.tile];
        rbase[tid] = T.row0 | ((tile_kind(T.kind) == TK_SELL && (T.kind & TF_SORTED)) ? 0x80000000u : 0u);
      }
    }
    uint32_t x = np;  // inclusive scan of the piece counts
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)x, o);
      if ((int)lane >= o) x += y;
    }
    if (lane == WAVE - 1) wsum[wave] = x;
    __syncthreads();
    uint32_t total = 0;
    for (uint32_t k = 0; k < TA_THREADS / WAVE; ++k) {
      if (k < wave) x += wsum[k];
      total += wsum[k];
    }
    const uint32_t mine = x - np;
    for (uint32_t w0 = 0; w0 < total; w0 += TA_LIST) {
      __syncthreads();  // the last window's pieces are done with
      for (uint32_t k = 0; k < np; ++k) {
        const uint32_t at = mine + k - w0;
        if (at < (uint32_t)TA_LIST) list[at] = tid | (k << 10);
      }
      __syncthreads();
      const uint32_t wn = min(total - w0, (uint32_t)TA_LIST);
      for (uint32_t i = grp; i < wn; i += NG) {
        const uint32_t e = list[i], t = e & 1023u, k0 = (e >> 10) * PS;
        const uint2* r = rec + first[t] + k0;
        const uint32_t n = count[t] - k0;  // records from here to the end of the run
        uint2 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = sub + u * EPI < n ? r[sub + u * EPI] : make_uint2(0u, 0u);
        if constexpr (SP == 1) {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (sub + u * EPI < n) atomicAdd(&sums[a[u].y], (unsigned long long)a[u].x);
        } else {
          const uint32_t rb = rbase[t];
          uint32_t x[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            uint32_t row = (rb & 0x7FFFFFFFu) + (a[u].y >> 16);
            const bool on = sub + u * EPI < n && (int)comp < s;
            if (on && (rb >> 31)) row = A.perm[row];
            x[u] = on ? (uint32_t)X[(int64_t)row * ldx + comp] : 0u;
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (sub + u * EPI < n && (int)comp < s)
              atomicAdd(&sums[(a[u].y & 0xFFFFu) * SP + comp], (unsigned long long)tterm<K>(a[u].x, x[u], A));
        }
      }
    }
    __syncthreads();  // before the next round rewrites the batches' entries
  }
  __syncthreads();
  uint32_t* out = part + ((size_t)q * A.ncols + j0) * SP;
  for (uint32_t i = tid; i < nj * SP; i += TA_THREADS) out[i] = mod_u64(sums[i], A.m, A.mu);
}

// y from Q parts, each below 2^32 (residues, or the 32-bit sums of the column-sorted groups; Q <= 2^31)
template <typename Tv>
__global__ void k_t_parts(uint32_t m, uint64_t mu, int64_t n, const uint32_t* __restrict__ part, uint32_t Q, int s,
                          int sp, uint32_t alpha, uint32_t beta, Tv* __restrict__ Y, int64_t ldy) {
  const int64_t total = n * s, stride = n * sp;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = i / s;
    const int c = (int)(i - j * s);
    const uint32_t* a = part + j * sp + c;
    uint64_t sum = 0;
#pragma unroll 4
    for (uint32_t q = 0; q < Q; ++q) sum += a[q * stride];
    finish_row(m, mu, sum, alpha, beta, Y + j * ldy + c);
  }
}

// ------------------------------------------------------------------ host ---
hipError_t launch_t_parts(ffx_dtype dt, uint32_t m, uint64_t mu, int64_t n, const uint32_t* part, uint32_t Q, int s,
                          int sp, uint32_t alpha, uint32_t beta, void* Y, int64_t ldy, hipStream_t st) {
  const dim3 g((unsigned)std::min<int64_t>((n * s + 255) / 256, 8192)), b(256);
  if (dt == FFX_I32)
    hipLaunchKernelGGL(k_t_parts<int32_t>, g, b, 0, st, m, mu, n, part, Q, s, sp, alpha, beta, (int32_t*)Y, ldy);
  else
    hipLaunchKernelGGL(k_t_parts<int64_t>, g, b, 0, st, m, mu, n, part, Q, s, sp, alpha, beta, (int64_t*)Y, ldy);
  return hipGetLastError();
}

static int pow2_at_least(int s) { return s <= 1 ? 1 : s <= 2 ? 2 : s <= 4 ? 4 : s <= 8 ? 8 : 16; }

// Shape of the binned form, or ok = false for the scattered one.
//  - Panels: at most 16,384 sums (128 KB of LDS) each, and at least about 32 of
//    them where the outputs allow, so that panels and parts fill 256 compute
//    units with few parts to add up. More than TB_MAXP panels would leave a
//    batch only a few records per panel: scattered.
//  - Runs: a workgroup works on a batch's records of its panel as one piece or more,
//    each a chain of loads that takes as long for one record as for 64, so the
//    additions take as long as the runs to a workgroup, a scatter as long as its
//    transactions. Scattered where records by workgroups to a run are fewer than
//    min_records. Four vectors, 20,000 rows of 300 (each a batch) over 300,000
//    columns (900): 415 us binned, 271 scattered; over 150,000 (1,800): 249 and 269.
//    Eight: 200,000 rows of 6 over 300,000 (2,043): 96 and 78; 20,000 of 300 over
//    60,000 (2,400): 274 and 271, over 20,000 (3,600): 208 and 275. Sixteen: over
//    150,000 (300): 1,371 and 536, over 60,000 (1,200): 475 and 530. Two: over
//    1,000,000 (590): 342 and 272, over 300,000 (1,800): 169 and 269. One: over
//    4,000,000 (300): 256 and 275; 1,000,000 rows with 8 entries in every fiftieth
//    (163): 39 and 20. Not with fewer tiles than fill the GPU with a scatter's
//    workgroups (8 vectors, 50,000 rows of 30 over 300,000 columns, 196 tiles, 2,043:
//    98 and 117).
//  - Small products: few transactions are soon done, but few output rows take many
//    atomics each, and those to one address wait for one another, so the line is
//    low (600 rows of 10, one vector: 14 us scattered, 16 binned, four: 23 and 16; 1,000:
//    16 and 17, 25 and 16), with five vectors or more lower still (100 rows of 10: 32
//    and 17; 60: 13 and 11), and for one vector and short columns higher (30,000 rows
//    of 5 near the diagonal: 15 and 21, all over: 17 and 17; of 12: 20 and 21, 27 and
//    20; 20,000 rows of 12 over 1,000,000 columns: 24 and 29).
//  - Almost only diagonals: adjacent lanes add to adjacent sums, so a transaction
//    takes 8 / SP of them, and atomics to one address are few. Scattered up to
//    max_per_row transactions to an output row: one vector always (200,000 rows, 40
//    diagonals: 61 us scattered, 78 binned; 5: 16 and 31), two vectors up to 32
//    diagonals (100,000 rows, 21: 37 and 47; 40: 61 and 60), four up to 10 (200,000
//    rows, 5: 35 and 39; 9: 57 and 57; 21: 114 and 78), more never (eight, 400,000
//    rows, 3: 70 and 56; 5: 108 and 72).
//  - Scratch: the records of all entries, at most TB_MAX_SCRATCH.
struct TPlan {
  bool ok = false;
  uint32_t sh = 0, P = 0, Q = 0;
  size_t rec_bytes = 0, off_bytes = 0, part_bytes = 0;
};
constexpr size_t TB_MAX_SCRATCH = (size_t)1 << 30;
constexpr int64_t T_MIN_TRANSACTIONS = (int64_t)1 << 13, T_MIN_TRANSACTIONS_1 = (int64_t)1 << 18, T_MIN_TRANSACTIONS_8 = 512;
constexpr uint32_t T_MIN_TILES = 512;

static TPlan t_plan(const DevMat& A, const TransposeInfo& I, int s) {
  TPlan t;
  const int sp = pow2_at_least(s);
  const int64_t n = A.ncols;
  const int64_t transactions = I.nnz * ((s + 7) / 8);
  if (!I.nbatch || transactions < (sp >= 8 ? T_MIN_TRANSACTIONS_8 : T_MIN_TRANSACTIONS)) return t;
  if (s == 1 && I.nnz < T_MIN_TRANSACTIONS_1 && I.nnz <= 12 * n) return t;
  const int64_t max_per_row = sp <= 2 ? 8 : sp == 4 ? 5 : 0, rest = I.nnz - I.nband;
  if (rest < I.nnz / 10 && I.nband * sp / 8 + rest * ((s + 7) / 8) <= max_per_row * n) return t;
  uint32_t top = 14;
  for (int k = 1; k < sp; k *= 2) --top;
  t.sh = 6;
  while (t.sh < top && (n + ((int64_t)1 << t.sh) - 1) >> t.sh > 32) ++t.sh;
  const int64_t P = (n + ((int64_t)1 << t.sh) - 1) >> t.sh;
  if (P > TB_MAXP) return t;
  const int64_t Q = std::min<int64_t>({16, std::max<int64_t>(1, 256 / P), I.nbatch});
  const int64_t min_records = sp == 1 ? 250 : sp == 2 ? 1000 : sp == 4 ? 1700 : sp == 8 ? 2400 : 900;
  if (A.ntiles >= T_MIN_TILES && I.nnz * P * Q < min_records * I.runs[t.sh]) return t;
  t.P = (uint32_t)P;
  t.Q = (uint32_t)Q;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  t.rec_bytes = al((size_t)I.nrec * sizeof(uint2));
  t.off_bytes = al((size_t)I.nbatch * (t.P + 1) * sizeof(uint16_t));
  t.part_bytes = al((size_t)t.Q * n * sp * sizeof(uint32_t));
  t.ok = t.rec_bytes + t.off_bytes + t.part_bytes <= TB_MAX_SCRATCH;
  return t;
}

static int t_kind(const DevMat& A) { return A.m <= 65536u ? TM_SMALL : A.m == 2147483647u ? TM_M31 : TM_BIG; }

template <int K, typename Tv, int SP>
static hipError_t t_acc_go(const DevMat& A, const TransposeInfo& I, const TPlan& t, const Tv* X, int64_t ldx, int s,
                           const uint2* rec, const uint16_t* off, uint32_t* part, hipStream_t st) {
  auto k = k_t_acc<K, Tv, SP>;
  const size_t lds = ((size_t)8 << t.sh) * SP + TA_LDS_FIXED;
  hipError_t e = raise_lds_limit((const void*)k, (int)(128 * 1024 + TA_LDS_FIXED));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(t.P * t.Q), dim3(TA_THREADS), lds, st, A, X, ldx, s, I.nbatch, t.sh, t.P, t.Q, rec, off,
                     part);
  return hipGetLastError();
}

template <int K, typename Tv>
static hipError_t launch_binned(const DevMat& A, const TransposeInfo& I, const TPlan& t, const Tv* X, int64_t ldx,
                                Tv* Y, int64_t ldy, int s, uint32_t alpha, uint32_t beta, unsigned char* scratch,
                                hipStream_t st) {
  uint2* rec = (uint2*)scratch;
  uint16_t* off = (uint16_t*)(scratch + t.rec_bytes);
  uint32_t* part = (uint32_t*)(scratch + t.rec_bytes + t.off_bytes);
  const int sp = pow2_at_least(s);
  const dim3 g(I.nbatch), b(TILE_THREADS);
  if (s == 1) hipLaunchKernelGGL((k_t_bin<K, Tv, true>), g, b, 0, st, A, X, ldx, t.sh, t.P, rec, off);
  else hipLaunchKernelGGL((k_t_bin<K, Tv, false>), g, b, 0, st, A, X, ldx, t.sh, t.P, rec, off);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (sp) {
    case 1: e = t_acc_go<K, Tv, 1>(A, I, t, X, ldx, s, rec, off, part, st); break;
    case 2: e = t_acc_go<K, Tv, 2>(A, I, t, X, ldx, s, rec, off, part, st); break;
    case 4: e = t_acc_go<K, Tv, 4>(A, I, t, X, ldx, s, rec, off, part, st); break;
    case 8: e = t_acc_go<K, Tv, 8>(A, I, t, X, ldx, s, rec, off, part, st); break;
    default: e = t_acc_go<K, Tv, 16>(A, I, t, X, ldx, s, rec, off, part, st); break;
  }
  if (e != hipSuccess) return e;
  return launch_t_parts(sizeof(Tv) == 4 ? FFX_I32 : FFX_I64, A.m, A.mu, A.ncols, part, t.Q, s, sp, alpha, beta, Y, ldy,
                        st);
}

// Sums to an output row of the scatter: padded to SP, up to T_MAX_PADDED bytes of them; s in larger temporaries,
// where an output row's sums may lie in one 64-byte piece more (4,000,000 columns of 9 vectors: 288 MB and not 512).
constexpr size_t T_MAX_PADDED = (size_t)256 << 20;
static int sum_stride(const DevMat& A, int s) {
  return (size_t)A.ncols * pow2_at_least(s) * sizeof(uint64_t) <= T_MAX_PADDED ? pow2_at_least(s) : s;
}

template <int K, typename Tv>
static hipError_t launch_scattered(const DevMat& A, const Tv* X, int64_t ldx, Tv* Y, int64_t ldy, int s,
                                   uint32_t alpha, uint32_t beta, unsigned long long* acc, hipStream_t st) {
  const int sp = pow2_at_least(s), stride = sum_stride(A, s);
  const int64_t n = A.ncols, total = n * stride;
  const int zb = (int)std::min<int64_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_zero_u64, dim3(zb), dim3(256), 0, st, acc, total);
  const dim3 g(A.ntiles), b(TILE_THREADS);
  if (A.ntiles) switch (sp) {
    case 1: hipLaunchKernelGGL((k_scatter_t<K, Tv, 1>), g, b, 0, st, A, X, ldx, s, stride, acc); break;
    case 2: hipLaunchKernelGGL((k_scatter_t<K, Tv, 2>), g, b, 0, st, A, X, ldx, s, stride, acc); break;
    case 4: hipLaunchKernelGGL((k_scatter_t<K, Tv, 4>), g, b, 0, st, A, X, ldx, s, stride, acc); break;
    case 8: hipLaunchKernelGGL((k_scatter_t<K, Tv, 8>), g, b, 0, st, A, X, ldx, s, stride, acc); break;
    default: hipLaunchKernelGGL((k_scatter_t<K, Tv, 16>), g, b, 0, st, A, X, ldx, s, stride, acc); break;
  }
  hipLaunchKernelGGL(k_finish_t<Tv>, dim3(zb), dim3(256), 0, st, A, acc, n, s, stride, alpha, beta, Y, ldy);
  return hipGetLastError();
}

size_t transpose_scratch_bytes(const DevMat& A, const TransposeInfo& I, int s, bool binned) {
  if (!binned) return (size_t)A.ncols * sum_stride(A, s) * sizeof(uint64_t);
  const TPlan t = t_plan(A, I, s);
  return t.ok ? t.rec_bytes + t.off_bytes + t.part_bytes : 0;
}

hipError_t launch_transpose(const DevMat& A, const TransposeInfo& I, ffx_dtype dt, const void* X, int64_t ldx, void* Y,
                            int64_t ldy, int s, uint32_t alpha, uint32_t beta, void* scratch, bool binned,
                            hipStream_t st) {
  if (A.ncols == 0) return hipSuccess;
  const TPlan t = binned ? t_plan(A, I, s) : TPlan{};
  auto go = [&](auto tv, auto kind) -> hipError_t {
    using Tv = decltype(tv);
    constexpr int K = decltype(kind)::value;
    if (t.ok)
      return launch_binned<K, Tv>(A, I, t, (const Tv*)X, ldx, (Tv*)Y, ldy, s, alpha, beta, (unsigned char*)scratch, st);
    return launch_scattered<K, Tv>(A, (const Tv*)X, ldx, (Tv*)Y, ldy, s, alpha, beta, (unsigned long long*)scratch, st);
  };
  auto by_kind = [&](auto tv) -> hipError_t {
    switch (t_kind(A)) {
      case TM_SMALL: return go(tv, std::integral_constant<int, TM_SMALL>{});
      case TM_M31: return go(tv, std::integral_constant<int, TM_M31>{});
      default: return go(tv, std::integral_constant<int, TM_BIG>{});
    }
  };
  return dt == FFX_I32 ? by_kind(int32_t{}) : by_kind(int64_t{});
}

}  // namespace ffx
