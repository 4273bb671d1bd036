// Block Wiedemann steps 2 and 3 (Section 3) over a prime field F_p, p < 2^31:
// the order basis (sigma-basis) of a power series by PM-Basis (Giorgi,
// Jeannerod and Villard, ISSAC 2003; Section 3.2 "Parallelization of the
// sigma-basis computation"), the minimal matrix generator of the sequence, and
// rank = deg det F - codeg det F.
//
// PM-Basis splits the order in two halves: the basis M1 of the first half, the
// middle product R = [x^s1 .. x^(s-1)] (M1 G), the basis M2 of R with M1's
// degrees, and M = M2 M1. Orders up to LEAF are done by the one-order-at-a-time
// M-Basis in one launch, a column of the basis to a workgroup, in LDS. Because M-Basis only
// looks at the residual coefficient [x^k](M G) and the degrees, the
// divide-and-conquer result is the same basis, step for step, as M-Basis run
// over the whole order.
//
// Large polynomial matrix products go through number-theoretic transforms over
// three word-size primes and a CRT (the paper's DFT multiplication; see the
// NTT section below); smaller ones are schoolbook convolutions, on the matrix
// cores in bytes (see k_polymul_mx), or for the fewest rows on the vector ALU.
// There a workgroup computes 256 consecutive coefficients of one entry; for each
// inner index q and each 256-coefficient chunk of A it stages the chunk of A and
// the 511 coefficients of B that the tile needs in LDS, and every lane adds
// 256 products into a 96-bit accumulator (64-bit sum plus a carry count), so a
// coefficient is reduced once.
#include <algorithm>
#include <atomic>
#include <vector>

#include "host.h"
#include "launch.h"

namespace ffx {

constexpr int SB_LEAF = 32;    // orders done by one launch of the in-LDS M-Basis
constexpr int SB_MAXM = 16;    // rows of the basis
constexpr int SB_MAXN = 8;     // columns of the series
constexpr int PM_TILE = 256;   // coefficients per workgroup in the products

struct Field {
  uint32_t p;
  uint64_t mu;    // floor((2^64-1)/p)
  uint32_t r64;   // 2^64 mod p
  int mersenne;   // p = 2^31 - 1: products fold with shifts
};

__device__ inline uint32_t fmul(uint32_t a, uint32_t b, const Field& F) {
  uint64_t x = (uint64_t)a * b;
  if (F.mersenne) {  // x < 2^62: two folds bring it to at most p + 1
    x = (x & 0x7FFFFFFFull) + (x >> 31);
    x = (x & 0x7FFFFFFFull) + (x >> 31);
    return (uint32_t)(x >= 0x7FFFFFFFull ? x - 0x7FFFFFFFull : x);
  }
  return mod_u64(x, F.p, F.mu);
}

// (hi * 2^64 + lo) mod p, hi < 2^32
__device__ inline uint32_t fold96(uint64_t lo, uint32_t hi, const Field& F) {
  uint64_t h = (uint64_t)(hi % F.p) * F.r64;
  return mod_u64(h + mod_u64(lo, F.p, F.mu), F.p, F.mu);
}

__device__ inline uint32_t finv(uint32_t a, const Field& F) {  // a^(p-2), a != 0
  uint32_t r = 1, b = a, e = F.p - 2;
  while (e) {
    if (e & 1) r = fmul(r, b, F);
    b = fmul(b, b, F);
    e >>= 1;
  }
  return r;
}

// Sums of products of two residues: for p = 2^31 - 1 each product is folded
// below 2^32 and added to 64 bits (no reduction for 2^31 terms); otherwise the
// products are added to a 96-bit sum.
template <bool MERS>
struct Acc96 {
  uint64_t lo = 0;
  uint32_t hi = 0;
  __device__ inline void add(uint64_t prod) {
    if (MERS) {
      lo += (prod & 0x7FFFFFFFull) + (prod >> 31);
    } else {
      lo += prod;
      hi += lo < prod;
    }
  }
  __device__ inline uint32_t reduce(const Field& F) const {
    if (MERS) {
      uint64_t x = (lo & 0x7FFFFFFFull) + (lo >> 31);  // below 2^33
      x = (x & 0x7FFFFFFFull) + (x >> 31);             // at most p + 3
      return (uint32_t)(x >= 0x7FFFFFFFull ? x - 0x7FFFFFFFull : x);
    }
    return fold96(lo, hi, F);
  }
};

// C[r][c][t] = sum_q sum_j A[r][q][j] B[q][c][k0 + t - j] for t < len.
// A: R x Q entries of la coefficients (entry (r,q) at A + (r*Q+q)*sa); B: Q x NC
// entries of lb coefficients (stride sb); C: R x NC entries (stride sc).
__global__ void __launch_bounds__(PM_TILE) k_polymul(const uint32_t* __restrict__ A, int64_t sa, int64_t la,
                                                     const uint32_t* __restrict__ B, int64_t sb, int64_t lb,
                                                     uint32_t* __restrict__ C, int64_t sc, int64_t k0, int64_t len,
                                                     int Q, int NC, Field F) {
  __shared__ uint32_t As[PM_TILE];
  __shared__ uint32_t Bs[2 * PM_TILE];
  const int tid = threadIdx.x;
  const int r = blockIdx.y / NC, c = blockIdx.y % NC;
  const int64_t kbase = k0 + (int64_t)blockIdx.x * PM_TILE;
  uint64_t lo = 0;
  uint32_t hi = 0;
  const int64_t jlo = std::max<int64_t>(0, kbase - (lb - 1));
  const int64_t jhi = std::min<int64_t>(la - 1, kbase + PM_TILE - 1);
  for (int q = 0; q < Q; ++q) {
    const uint32_t* a = A + (int64_t)(r * Q + q) * sa;
    const uint32_t* b = B + (int64_t)(q * NC + c) * sb;
    for (int64_t j0 = jlo; j0 <= jhi; j0 += PM_TILE) {
      __syncthreads();
      As[tid] = (j0 + tid <= jhi) ? a[j0 + tid] : 0u;
      // Bs[u] = B[kbase - j0 - (PM_TILE-1) + u], u < 2*PM_TILE - 1
      const int64_t base = kbase - j0 - (PM_TILE - 1);
      for (int u = tid; u < 2 * PM_TILE - 1; u += PM_TILE) {
        const int64_t idx = base + u;
        Bs[u] = (idx >= 0 && idx < lb) ? b[idx] : 0u;
      }
      __syncthreads();
#pragma unroll 8
      for (int jj = 0; jj < PM_TILE; ++jj) {
        const uint64_t prod = (uint64_t)As[jj] * Bs[tid - jj + PM_TILE - 1];
        lo += prod;
        hi += lo < prod;
      }
    }
  }
  const int64_t t = (int64_t)blockIdx.x * PM_TILE + tid;
  if (t < len) C[(int64_t)blockIdx.y * sc + t] = fold96(lo, hi, F);
}

// The same product with PM_OUT = 4 * PM_TILE coefficients per workgroup, four
// consecutive ones per lane, for products large enough to fill the GPU with
// such tiles: a lane keeps the B values of its four outputs in registers and
// shifts them by one per j, reading the next four B values and four A values
// (the same in every lane) with one aligned 16-byte read each, so each LDS read
// serves eight multiply-adds. For p = 2^31 - 1 the four products an output
// gets per group of four j are added raw (below 2^64) and folded once.
constexpr int PM_OUT = 4 * PM_TILE;
template <bool MERS>
__global__ void __launch_bounds__(PM_TILE) k_polymul4(const uint32_t* __restrict__ A, int64_t sa, int64_t la,
                                                      const uint32_t* __restrict__ B, int64_t sb, int64_t lb,
                                                      uint32_t* __restrict__ C, int64_t sc, int64_t k0, int64_t len,
                                                      int Q, int NC, Field F) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) uint32_t As[PM_TILE];
  __shared__ __align__(16) uint32_t Bs[PM_OUT + PM_TILE];  // Bs[1 + u] = B[kbase - j0 - (PM_TILE - 1) + u]
  const int tid = threadIdx.x;
  const int r = blockIdx.y / NC, c = blockIdx.y % NC;
  const int64_t kbase = k0 + (int64_t)blockIdx.x * PM_OUT;
  Acc96<MERS> acc[4];
  const int64_t jlo = std::max<int64_t>(0, kbase - (lb - 1));
  const int64_t jhi = std::min<int64_t>(la - 1, kbase + PM_OUT - 1);
  for (int q = 0; q < Q; ++q) {
    const uint32_t* a = A + (int64_t)(r * Q + q) * sa;
    const uint32_t* b = B + (int64_t)(q * NC + c) * sb;
    for (int64_t j0 = jlo; j0 <= jhi; j0 += PM_TILE) {
      __syncthreads();
      As[tid] = (j0 + tid <= jhi) ? a[j0 + tid] : 0u;
      const int64_t base = kbase - j0 - (PM_TILE - 1);
      for (int u = tid; u < PM_OUT + PM_TILE - 1; u += PM_TILE) {
        const int64_t idx = base + u;
        Bs[1 + u] = (idx >= 0 && idx < lb) ? b[idx] : 0u;
      }
      if (tid == 0) Bs[0] = 0u;
      __syncthreads();
      // output t = 4 tid + v meets A[j0 + jj] and Bs[t - jj + PM_TILE]
      const int t0 = 4 * tid + PM_TILE;
      uint32_t bv0 = Bs[t0], bv1 = Bs[t0 + 1], bv2 = Bs[t0 + 2], bv3 = Bs[t0 + 3];
      for (int jj = 0; jj < PM_TILE; jj += 4) {
        const u32x4_t a4 = *(const u32x4_t*)&As[jj];
        const u32x4_t nb = *(const u32x4_t*)&Bs[t0 - jj - 4];  // index >= 4 tid >= 0
        uint64_t g0 = 0, g1 = 0, g2 = 0, g3 = 0;
        auto step = [&](uint32_t av, uint32_t next) {
          const uint64_t x = av;
          if (MERS) {
            g0 += x * bv0;
            g1 += x * bv1;
            g2 += x * bv2;
            g3 += x * bv3;
          } else {
            acc[0].add(x * bv0);
            acc[1].add(x * bv1);
            acc[2].add(x * bv2);
            acc[3].add(x * bv3);
          }
          bv3 = bv2;
          bv2 = bv1;
          bv1 = bv0;
          bv0 = next;
        };
        step(a4.x, nb.w);
        step(a4.y, nb.z);
        step(a4.z, nb.y);
        step(a4.w, nb.x);
        if (MERS) {
          acc[0].lo += (g0 & 0x7FFFFFFFull) + (g0 >> 31);
          acc[1].lo += (g1 & 0x7FFFFFFFull) + (g1 >> 31);
          acc[2].lo += (g2 & 0x7FFFFFFFull) + (g2 >> 31);
          acc[3].lo += (g3 & 0x7FFFFFFFull) + (g3 >> 31);
        }
      }
    }
  }
  const int64_t t = (int64_t)blockIdx.x * PM_OUT + 4 * tid;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (t + v < len) C[(int64_t)blockIdx.y * sc + t + v] = acc[v].reduce(F);
}

// Products whose A entries have at most PMS_MAXA coefficients and whose output
// entries at most PMS_MAX_TILES * PM_TILE: the lower levels of the recursion,
// where a product is a few thousand multiply-adds per entry and the tile
// kernel's time goes to a barrier and a round trip to memory per inner index.
// Here one workgroup per output entry and PM_TILE outputs stages every A and B
// coefficient it needs in LDS at once, and four groups of PM_TILE lanes each
// take every fourth inner index q; the four partial sums, reduced, meet in LDS.
constexpr int PMS_MAXA = PM_TILE + 1;
constexpr int PMS_NT = 4 * PM_TILE;
constexpr int PMS_MAX_TILES = 4;  // longer outputs go to the tile kernels
inline size_t polymul_small_lds(int Q, int64_t la) {
  return ((size_t)Q * la + (size_t)Q * (PM_TILE + la - 1) + 3 * PM_TILE) * sizeof(uint32_t);
}
template <bool MERS>
__global__ void __launch_bounds__(PMS_NT) k_polymul_small(const uint32_t* __restrict__ A, int64_t sa, int la,
                                                          const uint32_t* __restrict__ B, int64_t sb, int64_t lb,
                                                          uint32_t* __restrict__ C, int64_t sc, int64_t k0, int64_t len,
                                                          int Q, int NC, Field F) {
  extern __shared__ uint32_t pms[];
  const int tid = threadIdx.x;
  const int r = blockIdx.x / NC, c = blockIdx.x % NC;
  // this workgroup's PM_TILE outputs: coefficients t0 .. t0 + tl - 1 of the entry
  const int64_t t0 = (int64_t)blockIdx.y * PM_TILE;
  const int tl = (int)std::min<int64_t>(PM_TILE, len - t0);
  k0 += t0;
  C += t0;
  const int nb = tl + la - 1;  // B[k0 - (la - 1) .. k0 + tl - 1]
  uint32_t* As = pms;
  uint32_t* Bs = pms + Q * la;
  uint32_t* part_s = Bs + Q * nb;
  for (int i = tid; i < Q * la; i += PMS_NT) {
    const int q = i / la, j = i - q * la;
    As[i] = A[(int64_t)(r * Q + q) * sa + j];
  }
  const int64_t b0 = k0 - (la - 1);
  for (int i = tid; i < Q * nb; i += PMS_NT) {
    const int q = i / nb, u = i - q * nb;
    const int64_t idx = b0 + u;
    Bs[i] = (idx >= 0 && idx < lb) ? B[(int64_t)(q * NC + c) * sb + idx] : 0u;
  }
  __syncthreads();
  const int t = tid % PM_TILE, part = tid / PM_TILE;
  Acc96<MERS> acc;
  if (t < tl) {
    // output k0 + t meets A[j] and B[k0 + t - j] = Bs[t - j + la - 1], for j with 0 <= k0 + t - j < lb
    const int64_t kt = k0 + t;
    const int jlo = (int)std::max<int64_t>(0, kt - (lb - 1));
    const int jhi = (int)std::min<int64_t>(la - 1, kt);
    for (int q = part; q < Q; q += 4) {
      const uint32_t* a = As + q * la;
      const uint32_t* b = Bs + q * nb + t + la - 1;
      for (int j = jlo; j <= jhi; ++j) acc.add((uint64_t)a[j] * b[-j]);
    }
  }
  const uint32_t v = acc.reduce(F);
  if (part > 0) part_s[(part - 1) * PM_TILE + t] = v;
  __syncthreads();
  if (part == 0 && t < tl) {
    uint32_t sum = v;
#pragma unroll
    for (int k = 0; k < 3; ++k) {  // residues below p < 2^31: a sum of two stays below 2^32
      sum += part_s[k * PM_TILE + t];
      sum = sum >= F.p ? sum - F.p : sum;
    }
    C[(int64_t)blockIdx.x * sc + t] = sum;
  }
}

// One-order-at-a-time basis (M-Basis) of the m x n series G to order sg <= SB_LEAF
// with shifted degrees d_in, written to d_out by workgroup 0 (another buffer: the
// others may start when it has ended). M: m x m entries of sm >= sg + 1 coefficients.
//
// One order is a chain of at most n pivot steps that nothing else can hide, so
// the rest of the work is taken off that chain. Workgroup c holds column c of M
// and all of the residual series R = x^-k M G, and carries out the same row
// operations as the others, so the workgroups need nothing from one another. In
// a workgroup, waves 0 to 3 (one to a SIMD) eliminate order k: lane & 15 is a
// row, in the order in which rows become pivots, of two columns of the residual
// coefficient, the same in each wave, and of one of the 16 columns of the
// transformation T_k, so that a step is a few moves between lanes and three
// registers, without LDS or a barrier. The other twelve
// waves apply T_(k-1) to R and M meanwhile, and one barrier per order hands T_k
// over; the next residual coefficient is T_k times one coefficient of R.
//
// 31 orders of 16 x 8 at p = 2^31 - 1: 363 us as one workgroup that formed each
// residual from M and G and eliminated behind a barrier per pivot, 85 us now (of
// 2.6 us per order the pivot steps are 1.3, the update as much: all four SIMDs are
// busy with multiplications, each a quarter of the rate of an addition).
constexpr int LEAF_NT = 1024;
constexpr int LEAF_EW = 4;                                // waves of the elimination
constexpr int LEAF_AW = LEAF_NT / WAVE - LEAF_EW;         // waves of the update, four rows each
constexpr int LEAF_RJ = SB_MAXM * SB_MAXN + SB_MAXN;      // words from a coefficient of R to the next, [q][c] each
constexpr int LEAF_MJ = SB_MAXM + 1;                      // of M's column, [q] each
constexpr int LEAF_TD = SB_MAXN;                          // a row of T: its entries in the pivots' columns, then
constexpr int LEAF_TR = SB_MAXN + 4;                      // its diagonal entry (it has no others); to the next row
static_assert(SB_MAXM == 16 && SB_MAXN == 8 && LEAF_AW % 4 == 0, "lanes of the leaf");

// x mod p, x any sum of two products of residues (or four for p = 2^31 - 1)
template <bool MERS>
__device__ inline uint32_t fred(uint64_t x, const Field& F) {
  if (!MERS) return mod_u64(x, F.p, F.mu);
  x = (x & 0x7FFFFFFFull) + (x >> 31);  // below 2^34
  x = (x & 0x7FFFFFFFull) + (x >> 31);  // below p + 9
  return (uint32_t)(x >= 0x7FFFFFFFull ? x - 0x7FFFFFFFull : x);
}

// Lane I of each 16 lanes, in all of them (a move on the vector ALU: no trip through LDS).
template <int I>
__device__ inline uint32_t bcast16(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + I, 0xf, 0xf, false);
}

// The 16 lanes of group gr (uniform, 0..3), in all four groups.
__device__ inline uint32_t group16(uint32_t v, int gr) {
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);  // both halves as the lower one, as the upper
  const uint32_t u = (gr & 2) ? h[1] : h[0];
  const auto q = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return (gr & 1) ? q[1] : q[0];
}

// f(0), f(1), ... with the index a constant, until one returns false
template <int I, class Fn>
__device__ inline void pivot_steps(Fn& f) {
  if constexpr (I < SB_MAXM)
    if (f(std::integral_constant<int, I>{})) pivot_steps<I + 1>(f);
}

template <bool MERS>
__global__ void __launch_bounds__(LEAF_NT) k_mbasis_leaf(const uint32_t* __restrict__ G, int64_t ldg, int m, int n,
                                                         int sg, const int32_t* __restrict__ d_in,
                                                         int32_t* __restrict__ d_out, uint32_t* __restrict__ M,
                                                         int64_t sm, Field F) {
  __shared__ __align__(16) uint32_t Rs[2][SB_LEAF * LEAF_RJ];
  __shared__ uint32_t Ms[2][(SB_LEAF + 1) * LEAF_MJ];
  __shared__ __align__(16) uint32_t Ts[2][SB_MAXM * LEAF_TR];
  __shared__ uint32_t piv_s[2];
  __shared__ uint32_t sc[SB_MAXM];  // scale of each row from fraction-free elimination
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int mc = blockIdx.x;  // this workgroup's column of M
  for (int i = tid; i < SB_MAXM * SB_MAXN * SB_LEAF; i += LEAF_NT) {
    const int k = i % SB_LEAF, c = i / SB_LEAF % SB_MAXN, r = i / (SB_LEAF * SB_MAXN);
    Rs[0][k * LEAF_RJ + r * SB_MAXN + c] = (r < m && c < n && k < sg) ? G[(int64_t)(r * n + c) * ldg + k] : 0u;
  }
  for (int i = tid; i < (SB_LEAF + 1) * LEAF_MJ; i += LEAF_NT) {  // both: coefficients above the degree stay 0
    Ms[0][i] = i == mc ? 1u : 0u;
    Ms[1][i] = 0u;
  }
  __syncthreads();

  if (wave < LEAF_EW) {
    __builtin_amdgcn_s_setprio(3);
    // this lane: position pos of the order's sequence of rows, columns g and g + 4 of the residual, col of T
    const int pos = lane & 15, g = lane >> 4, col = 4 * wave + g;
    int32_t deg = pos < m ? d_in[pos] : 0;  // of row pos
    // the row at this lane's position: rows by increasing shifted degree, ties by index, those past m last
    auto row_order = [&] {
      int before = 0;  // rows 4g .. 4g + 3 that come before row pos
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        const int j = 4 * g + z, dj = __shfl(deg, j);
        before += j < m && (pos >= m || dj < deg || (dj == deg && j < pos));
      }
      const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)before, (uint32_t)before, false, false);
      const uint32_t u = h[0] + h[1];
      const auto q = __builtin_amdgcn_permlane16_swap(u, u, false, false);
      const int at = pos < m ? (int)(q[0] + q[1]) : pos;
      return __builtin_amdgcn_ds_permute((at + 16 * g) * 4, pos);  // row pos goes to lane `at`
    };
    int row = row_order();
    uint32_t D0 = Rs[0][row * SB_MAXN + g], D1 = Rs[0][row * SB_MAXN + g + 4];
    for (int k = 0;; ++k) {
      if (k < sg) {
        // Echelon form of the residual, right-looking: when a row keeps a nonzero residual it becomes a
        // pivot (column: its first nonzero entry) and every later row is reduced by it at once. Fraction
        // free: row_j <- pv row_j - x_j row_i is the oracle's row_j - (x_j / pv) row_i times pv. The rows
        // stay scaled by the product of these factors, which is T's diagonal, from order to order; the
        // scales are divided out once, when the leaf writes its basis.
        uint32_t t = row == col ? 1u : 0u, pivots = 0;
        uint64_t b0 = __ballot(D0 != 0u), b1 = __ballot(D1 != 0u);
        auto step = [&](auto index) {
          constexpr int oi = decltype(index)::value;
          constexpr uint64_t row_oi = 0x0001000100010001ull << oi, from_oi = 0x0001000100010001ull * (0x10000u - (1u << oi));
          if (((b0 | b1) & from_oi) == 0) return false;  // what is left is zero
          const uint64_t r0 = b0 & row_oi, r1 = b1 & row_oi, r = r0 ? r0 : r1;
          if (r == 0) return true;
          const uint32_t x = group16(r0 ? D0 : D1, __builtin_ctzll(r) >> 4);  // this row's entry in the pivot column
          const uint32_t pv = bcast16<oi>(x), p0 = bcast16<oi>(D0), p1 = bcast16<oi>(D1), pt = bcast16<oi>(t);
          if (pos > oi && x) {
            const uint32_t nx = F.p - x;
            D0 = fred<MERS>((uint64_t)pv * D0 + (uint64_t)nx * p0, F);
            D1 = fred<MERS>((uint64_t)pv * D1 + (uint64_t)nx * p1, F);
            t = fred<MERS>((uint64_t)pv * t + (uint64_t)nx * pt, F);
          }
          pivots |= 1u << __builtin_amdgcn_readlane(row, oi);
          b0 = __ballot(D0 != 0u);
          b1 = __ballot(D1 != 0u);
          return true;
        };
        pivot_steps<0>(step);
        const uint32_t below = __popc(pivots & ((1u << col) - 1u)), npiv = __popc(pivots);
        const bool pc = (pivots >> col) & 1u;
        const uint32_t slot = pc ? below : npiv + (uint32_t)col - below;  // the slots past the last pivot hold 0
        if (slot < (uint32_t)LEAF_TD) Ts[k & 1][row * LEAF_TR + slot] = pc && row != col ? t : 0u;
        if (row == col) Ts[k & 1][row * LEAF_TR + LEAF_TD] = t;
        if (tid == 0) piv_s[k & 1] = pivots;
        deg += (int)((pivots >> pos) & 1u);
        row = row_order();
      }
      __syncthreads();
      if (k >= sg) break;
      // the next residual coefficient: T's row times coefficient k + 1 of R, or coefficient k for a pivot row,
      // which is multiplied by x
      if (k + 1 < sg) {
        typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
        uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane((int)piv_s[k & 1]);
        const uint32_t* tr = &Ts[k & 1][row * LEAF_TR];
        const uint32_t* rc = &Rs[k & 1][(k + 1 - (int)((pm >> row) & 1u)) * LEAF_RJ + g];
        Acc96<MERS> a0, a1;
        const uint32_t td = tr[LEAF_TD];
        a0.add((uint64_t)td * rc[row * SB_MAXN]);
        a1.add((uint64_t)td * rc[row * SB_MAXN + 4]);
#pragma unroll
        for (int q0 = 0; q0 < SB_MAXN; q0 += 4) {
          const u32x4_t tv = *(const u32x4_t*)(tr + q0);
          const uint32_t tq[4] = {tv.x, tv.y, tv.z, tv.w};
          uint64_t s0 = 0, s1 = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t* rv = rc + (pm ? __builtin_ctz(pm) : 0) * SB_MAXN;
            pm &= pm - 1u;
            if (MERS) {  // four products of residues below 2^31 add below 2^64
              s0 += (uint64_t)tq[q] * rv[0];
              s1 += (uint64_t)tq[q] * rv[4];
            } else {
              a0.add((uint64_t)tq[q] * rv[0]);
              a1.add((uint64_t)tq[q] * rv[4]);
            }
          }
          if (MERS) {
            a0.add(s0);
            a1.add(s1);
          }
        }
        D0 = a0.reduce(F);
        D1 = a1.reduce(F);
      }
    }
    if (mc == 0 && wave == 0 && g == 0 && pos < m) d_out[pos] = deg;
  } else {
    // rows 4 rg .. 4 rg + 3 of columns u = part * 64 + lane, + 64 LEAF_AW / 4, ...: first the 8 columns of R's
    // coefficients from k on, then M's coefficients up to k
    const int rg = (wave - LEAF_EW) % 4, part = (wave - LEAF_EW) / 4;
    uint32_t scale = 1u;  // of row 4 rg + r in the lane of its diagonal entry
    for (int k = 0;; ++k) {
      if (k > 0) {
        const int o = k - 1, b = o & 1, nb = b ^ 1;  // T of order o: buffers b to nb
        const int tv = (int)Ts[b][rg * 4 * LEAF_TR + min(lane, 4 * LEAF_TR - 1)];  // four rows of T
        const uint32_t pivots = (uint32_t)__builtin_amdgcn_readfirstlane((int)piv_s[b]);
        scale = fred<MERS>((uint64_t)scale * (uint32_t)tv, F);
        const int nr = SB_MAXN * (sg - o), nu = nr + o + 1;
        // (every lane takes every turn, so that readlane finds all of T's rows; the lanes past the end write nothing)
        for (int u0 = part * WAVE; u0 < nu; u0 += WAVE * LEAF_AW / 4) {
          const bool on = u0 + lane < nu;
          const int u = on ? u0 + lane : u0;
          const bool inr = u < nr;
          const int j = inr ? o + u / SB_MAXN : u - nr, c = inr ? u % SB_MAXN : 0;
          const int at = inr ? j * LEAF_RJ + c : j * LEAF_MJ, qs = inr ? 3 : 0;  // log2 of the stride over rows
          const uint32_t* src = (inr ? Rs[b] : Ms[b]) + at;
          uint32_t* dst = (inr ? Rs[nb] : Ms[nb]) + at;
          uint32_t po[SB_MAXN], own[4], pm = pivots;
#pragma unroll
          for (int q = 0; q < SB_MAXN; ++q) {
            po[q] = src[(pm ? __builtin_ctz(pm) : 0) << qs];
            pm &= pm - 1u;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) own[r] = src[(rg * 4 + r) << qs];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = rg * 4 + r;
            auto tq = [&](int q) { return (uint64_t)(uint32_t)__builtin_amdgcn_readlane(tv, r * LEAF_TR + q); };
            Acc96<MERS> acc;
            acc.add(tq(LEAF_TD) * own[r]);
#pragma unroll
            for (int q = 0; q < SB_MAXN; q += 4) {
              if (MERS) {
                acc.add(tq(q) * po[q] + tq(q + 1) * po[q + 1] + tq(q + 2) * po[q + 2] + tq(q + 3) * po[q + 3]);
              } else {
#pragma unroll
                for (int z = q; z < q + 4; ++z) acc.add(tq(z) * po[z]);
              }
            }
            const uint32_t v = acc.reduce(F);
            if (!on) continue;
            if ((pivots >> i) & 1u) {  // times x
              if (!inr || j + 1 < sg) dst[(inr ? LEAF_RJ : LEAF_MJ) + (i << qs)] = v;
              if (!inr && j == 0) dst[i] = 0u;
            } else {
              dst[i << qs] = v;
            }
          }
        }
      }
      __syncthreads();
      if (k >= sg) break;
    }
    if (part == 0 && lane < 4 * LEAF_TR && lane % LEAF_TR == LEAF_TD) sc[rg * 4 + lane / LEAF_TR] = scale;
  }
  __syncthreads();
  if (tid < SB_MAXM) sc[tid] = finv(sc[tid], F);
  __syncthreads();
  for (int idx = tid; idx < m * (sg + 1); idx += LEAF_NT) {
    const int i = idx / (sg + 1), j = idx % (sg + 1);
    M[(int64_t)(i * m + mc) * sm + j] = fmul(Ms[sg & 1][j * LEAF_MJ + i], sc[i], F);
  }
}

// G = [S(x); -I] as 2s x s entries of L coefficients from S (L x s x s, dtype residues mod p).
template <typename T>
__global__ void k_sequence_series(const T* __restrict__ S, int64_t L, int s, uint32_t p, uint32_t* __restrict__ G) {
  const int64_t total = (int64_t)2 * s * s * L;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = t / L, k = t % L;
    const int r = (int)(e / s), c = (int)(e % s);
    uint32_t v;
    if (r < s) {
      const int64_t x = (int64_t)S[(k * s + r) * s + c] % (int64_t)p;
      v = (uint32_t)(x < 0 ? x + p : x);
    } else {
      v = (k == 0 && r - s == c) ? p - 1 : 0u;
    }
    G[t] = v;
  }
}

// ------------------------------------------------------------------ host ----
static Field make_field(uint32_t p) {
  Field F;
  F.p = p;
  F.mu = UINT64_MAX / p;
  F.r64 = (uint32_t)((((unsigned __int128)1) << 64) % p);
  F.mersenne = p == 0x7FFFFFFFu;
  return F;
}

// ------------------------------------------------------------ NTT products
// The paper multiplies the polynomial matrices of PM-Basis through a DFT
// (Section 3.2, "Parallel polynomial matrix multiplication": transform the
// entries, multiply the transformed matrices point by point, transform back).
// F_p with p = 2^31 - 1 has no roots of unity of large power-of-two order, so
// the product is taken over the integers: exactly modulo three primes below
// 2^31 that have roots of unity of order 2^25 and more, with the coefficients
// recovered by the Chinese remainder theorem (Garner's mixed-radix form) and
// reduced mod p. An integer coefficient of the product is below
// Q * min(la, lb) * (p-1)^2, checked on the host against the product of the
// three primes (about 2^92.6).
//
// Transforms of length N (a power of two) run as log2 N radix-2 passes over
// global memory, each pass one launch over every entry and prime: forward
// passes are decimation in frequency (natural order in, bit-reversed out), the
// pointwise products work in that order, and the inverse passes are
// decimation in time (bit-reversed in, natural out). Products are cyclic of
// length N; N covers the wanted coefficients k0 .. k0+len-1 and is large
// enough that no coefficient of the full product wraps onto them.
constexpr int NTT_NP = 3;
static const uint32_t NTT_PRIME[NTT_NP] = {2013265921u, 1811939329u, 2113929217u};  // 15*2^27+1, 27*2^26+1, 63*2^25+1
static const uint32_t NTT_GEN[NTT_NP] = {31u, 13u, 5u};                            // primitive roots

struct NttPrimes {
  uint32_t p[NTT_NP];
  uint64_t mu[NTT_NP];
};

__device__ inline uint32_t nmul(uint32_t a, uint32_t b, uint32_t p, uint64_t mu) { return mod_u64((uint64_t)a * b, p, mu); }

// dst[i][e][t] = t < len ? src[e][t] mod p_i : 0, for n entries (entry e of src at src + e*stride)
__global__ void k_ntt_load(const uint32_t* __restrict__ src, int64_t stride, int64_t len, int ne, uint32_t* __restrict__ dst,
                           int64_t N, int dst_ne, int e0, NttPrimes P) {
  const int64_t total = (int64_t)NTT_NP * ne * N;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = g % N;
    const int64_t e = (g / N) % ne;
    const int i = (int)(g / (N * ne));
    const uint32_t v = t < len ? src[e * stride + t] % P.p[i] : 0u;
    dst[((int64_t)i * dst_ne + e0 + e) * N + t] = v;
  }
}

// tw[i][k] = w_i^k and itw[i][k] = w_i^-k, k < N/2, w_i a root of unity of order N modulo p_i
__global__ void k_ntt_twiddles(uint32_t* __restrict__ tw, int64_t half, const uint32_t* __restrict__ roots,
                               NttPrimes P) {
  const int64_t total = (int64_t)2 * NTT_NP * half;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = g % half;
    const int q = (int)(g / half);  // 0..2: forward roots, 3..5: inverse roots
    const int i = q % NTT_NP;
    uint32_t r = 1, b = roots[q];
    for (int64_t e = k; e; e >>= 1) {
      if (e & 1) r = nmul(r, b, P.p[i], P.mu[i]);
      b = nmul(b, b, P.p[i], P.mu[i]);
    }
    tw[g] = r;
  }
}

// One radix-2 pass over ne entries of every prime, butterflies of span h: forward (decimation in
// frequency) a, b -> a + b, (a - b) w^(j N / 2h); inverse (decimation in time) a, b -> a + b w', a - b w'.
template <bool INV>
__global__ void k_ntt_pass(uint32_t* __restrict__ X, int64_t N, int64_t h, int ne, const uint32_t* __restrict__ tw,
                           NttPrimes P) {
  const int64_t half = N / 2, total = (int64_t)NTT_NP * ne * half;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = g % half;
    const int64_t row = g / half;  // prime * ne + entry
    const int i = (int)(row / ne);
    const uint32_t p = P.p[i];
    const int64_t j = b % h, blk = b / h;
    uint32_t* x = X + row * N + blk * 2 * h + j;
    const uint32_t w = tw[((INV ? NTT_NP : 0) + i) * half + j * (half / h)];
    const uint32_t u = x[0], v = x[h];
    if (INV) {
      const uint32_t t = nmul(v, w, p, P.mu[i]);
      const uint32_t s = u + t;
      x[0] = s >= p ? s - p : s;
      x[h] = u >= t ? u - t : u + p - t;
    } else {
      const uint32_t s = u + v;
      x[0] = s >= p ? s - p : s;
      x[h] = nmul(u >= v ? u - v : u + p - v, w, p, P.mu[i]);
    }
  }
}

// C^[i][r][c][f] = sum_q A^[i][r][q][f] B^[i][q][c][f] mod p_i; AB holds the R*Q entries of A, then the Q*NC of B
__global__ void k_ntt_pointwise(const uint32_t* __restrict__ AB, uint32_t* __restrict__ Cf, int64_t N, int R, int Q,
                                int NC, NttPrimes P) {
  const int nab = R * Q + Q * NC, nc = R * NC;
  const int64_t total = (int64_t)NTT_NP * nc * N;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t f = g % N;
    const int e = (int)((g / N) % nc);
    const int i = (int)(g / (N * nc));
    const int r = e / NC, c = e % NC;
    const uint32_t* base = AB + (int64_t)i * nab * N;
    uint64_t acc = 0;  // Q <= 16 reduced products: below 2^36
    for (int q = 0; q < Q; ++q)
      acc += nmul(base[(int64_t)(r * Q + q) * N + f], base[(int64_t)(R * Q + q * NC + c) * N + f], P.p[i], P.mu[i]);
    Cf[((int64_t)i * nc + e) * N + f] = (uint32_t)(acc % P.p[i]);
  }
}

struct Garner {
  NttPrimes P;
  uint32_t ninv[NTT_NP];  // N^-1 mod p_i
  uint32_t inv1_2;        // p1^-1 mod p2
  uint32_t inv12_3;       // (p1 p2)^-1 mod p3
  uint32_t p12_3;         // p1 p2 mod p3
  uint32_t p1_f, p12_f;   // p1 and p1 p2 mod the field prime
};

// C[e][t - k0] = the product's coefficient t mod the field prime, for k0 <= t < k0 + len
__global__ void k_ntt_crt(const uint32_t* __restrict__ Cf, int64_t N, int nc, uint32_t* __restrict__ C, int64_t sc,
                          int64_t k0, int64_t len, Garner G, Field F) {
  const int64_t total = (int64_t)nc * len;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = g % len;
    const int e = (int)(g / len);
    uint32_t r[NTT_NP];
#pragma unroll
    for (int i = 0; i < NTT_NP; ++i)
      r[i] = nmul(Cf[((int64_t)i * nc + e) * N + k0 + t], G.ninv[i], G.P.p[i], G.P.mu[i]);
    const uint32_t p1 = G.P.p[0], p2 = G.P.p[1], p3 = G.P.p[2];
    // x = r1 + p1 t1 + p1 p2 t2 with 0 <= t1 < p2, 0 <= t2 < p3
    const uint32_t r1m2 = r[0] % p2;
    const uint32_t t1 = nmul(r[1] >= r1m2 ? r[1] - r1m2 : r[1] + p2 - r1m2, G.inv1_2, p2, G.P.mu[1]);
    const uint64_t x12 = (uint64_t)r[0] + (uint64_t)p1 * t1;  // < p1 p2 < 2^62
    const uint32_t x12m3 = (uint32_t)(x12 % p3);
    const uint32_t t2 = nmul(r[2] >= x12m3 ? r[2] - x12m3 : r[2] + p3 - x12m3, G.inv12_3, p3, G.P.mu[2]);
    const uint64_t lo = (uint64_t)mod_u64(x12, F.p, F.mu) + mod_u64((uint64_t)G.p12_f * t2, F.p, F.mu);
    C[(int64_t)e * sc + t] = (uint32_t)(lo >= F.p ? lo - F.p : lo);
  }
}

static uint32_t host_pow(uint64_t b, uint64_t e, uint32_t p) {
  uint64_t r = 1;
  b %= p;
  while (e) {
    if (e & 1) r = r * b % p;
    b = b * b % p;
    e >>= 1;
  }
  return (uint32_t)r;
}

// process-wide: the smallest la and lb at which a product goes through the NTT (0: never)
static std::atomic<int64_t> g_ntt_min{1024};

static int ntt_grid(int64_t work) { return (int)std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, 8192)); }

// The NTT form of polymul; returns false (nothing enqueued) when the coefficient bound exceeds the
// three primes' product or the length exceeds the primes' roots of unity.
static bool polymul_ntt(const uint32_t* A, int64_t sa, int64_t la, const uint32_t* B, int64_t sb, int64_t lb,
                        uint32_t* C, int64_t sc, int64_t k0, int64_t len, int R, int Q, int NC, const Field& F,
                        hipStream_t st) {
  const long double bound = (long double)Q * (long double)std::min(la, lb) * (long double)(F.p - 1) * (long double)(F.p - 1);
  const long double prod = (long double)NTT_PRIME[0] * NTT_PRIME[1] * NTT_PRIME[2];
  if (!(bound < prod * 0.999L)) return false;
  // cyclic length: covers k0 + len, and full coefficients at index >= N land below k0
  const int64_t need = std::max<int64_t>(k0 + len, la + lb - 1 - k0);
  int64_t N = 2;
  while (N < need) N *= 2;
  if (N > ((int64_t)1 << 25)) return false;
  NttPrimes P;
  uint32_t roots[2 * NTT_NP];
  Garner G;
  for (int i = 0; i < NTT_NP; ++i) {
    P.p[i] = NTT_PRIME[i];
    P.mu[i] = UINT64_MAX / NTT_PRIME[i];
    const uint32_t w = host_pow(NTT_GEN[i], (NTT_PRIME[i] - 1) / (uint64_t)N, NTT_PRIME[i]);
    if (host_pow(w, N / 2, NTT_PRIME[i]) != NTT_PRIME[i] - 1) fail(FFX_EDEVICE, "NTT root of unity check failed");
    roots[i] = w;
    roots[NTT_NP + i] = host_pow(w, NTT_PRIME[i] - 2, NTT_PRIME[i]);
    G.ninv[i] = host_pow((uint64_t)N % NTT_PRIME[i], NTT_PRIME[i] - 2, NTT_PRIME[i]);
  }
  G.P = P;
  const uint64_t p1 = NTT_PRIME[0], p2 = NTT_PRIME[1], p3 = NTT_PRIME[2];
  G.inv1_2 = host_pow(p1 % p2, p2 - 2, (uint32_t)p2);
  G.p12_3 = (uint32_t)((p1 * p2) % p3);
  G.inv12_3 = host_pow(G.p12_3, p3 - 2, (uint32_t)p3);
  G.p1_f = (uint32_t)(p1 % F.p);
  G.p12_f = (uint32_t)((unsigned __int128)(p1 * p2) % F.p);
  const int nab = R * Q + Q * NC, nc = R * NC;
  const int64_t half = N / 2;
  uint32_t *AB = nullptr, *Cf = nullptr, *tw = nullptr;
  const size_t bab = (size_t)NTT_NP * nab * N * 4, bc = (size_t)NTT_NP * nc * N * 4,
               btw = (size_t)2 * NTT_NP * half * 4 + 2 * NTT_NP * 4;
  if (hipMallocAsync((void**)&AB, bab, st) != hipSuccess || hipMallocAsync((void**)&Cf, bc, st) != hipSuccess ||
      hipMallocAsync((void**)&tw, btw, st) != hipSuccess) {
    for (void* q : {(void*)AB, (void*)Cf, (void*)tw})
      if (q) (void)hipFreeAsync(q, st);
    fail(FFX_ENOMEM, "NTT workspace allocation failed (length %lld)", (long long)N);
  }
  uint32_t* d_roots = tw + 2 * NTT_NP * half;
  hipError_t e = hipMemcpyAsync(d_roots, roots, sizeof roots, hipMemcpyHostToDevice, st);
  // the roots are read by the next kernel before this function returns the host array
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_ntt_twiddles, dim3(ntt_grid(2 * NTT_NP * half)), dim3(256), 0, st, tw, half, d_roots, P);
    hipLaunchKernelGGL(k_ntt_load, dim3(ntt_grid((int64_t)NTT_NP * R * Q * N)), dim3(256), 0, st, A, sa, la, R * Q, AB,
                       N, nab, 0, P);
    hipLaunchKernelGGL(k_ntt_load, dim3(ntt_grid((int64_t)NTT_NP * Q * NC * N)), dim3(256), 0, st, B, sb, lb, Q * NC,
                       AB, N, nab, R * Q, P);
    for (int64_t h = half; h >= 1; h /= 2)
      hipLaunchKernelGGL((k_ntt_pass<false>), dim3(ntt_grid((int64_t)NTT_NP * nab * half)), dim3(256), 0, st, AB, N, h,
                         nab, tw, P);
    hipLaunchKernelGGL(k_ntt_pointwise, dim3(ntt_grid((int64_t)NTT_NP * nc * N)), dim3(256), 0, st, AB, Cf, N, R, Q,
                       NC, P);
    for (int64_t h = 1; h < N; h *= 2)
      hipLaunchKernelGGL((k_ntt_pass<true>), dim3(ntt_grid((int64_t)NTT_NP * nc * half)), dim3(256), 0, st, Cf, N, h,
                         nc, tw, P);
    hipLaunchKernelGGL(k_ntt_crt, dim3(ntt_grid((int64_t)nc * len)), dim3(256), 0, st, Cf, N, nc, C, sc, k0, len, G, F);
    e = hipGetLastError();
    // the host array `roots` must outlive its copy
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  (void)hipFreeAsync(AB, st);
  (void)hipFreeAsync(Cf, st);
  (void)hipFreeAsync(tw, st);
  FFX_HIP(e);
  return true;
}

// Matrix-core products. A residue, taken in (-p/2, p/2), is four signed bytes
// d_l, x = sum_l d_l 256^l, so a product of two polynomial matrices is sixteen
// convolutions of matrices of bytes, of which those of equal l + l' share an
// accumulator, and one 16 x 16 x 64 instruction takes four coefficients j of A
// against B's coefficients t - j: rows r, columns c, and for the inner index
// the pairs (j, q). A column count below 16 leaves room for several t.
//
// k_pm_bytes writes the operands as byte planes [l][coefficient][row or column][q]
// (q in 16 consecutive bytes: one lane's operand), B's with zeros around the
// coefficients it has, so that k_polymul_mx has no conditions in its loop. A
// wave computes T coefficients t four apart: as j advances by four, coefficient
// t + 4 needs the operand of B that t has just used, so a step loads one operand
// of A and one of B for 16 T instructions. The four waves of a workgroup split the
// range of j and add up their residues in LDS.
//
// The vector ALU does at most one 31-bit multiply-add per lane in 22 cycles
// (a product at a quarter of the rate and its folds), 3 per cycle and SIMD; the
// matrix cores take 64. The 508 products of a 16 x 8 order basis of 8,003 orders
// took 19.4 ms on the vector ALU and take 5.5 ms, 2.4 of them for the planes.
//
// The line is at four rows, below which most of an instruction is padding: a basis
// of 8,003 orders with m = 2 takes 21.5 ms this way and 20.5 on the vector ALU,
// with m = 4 22.7 and 23.0, one of 3,001 orders with m = 5 8.9 and 9.3.
constexpr int MX_MINQ = 4;
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));
constexpr int MX_FLUSH = 256;  // steps of 4 coefficients an accumulator takes: 4 * 16 * 1024 products of at most 2^14

struct MxField {
  Field F;
  uint64_t bias;  // a multiple of p, at least 2^55: makes sums of byte products positive
  uint32_t r32;   // 2^32 mod p
};

__device__ inline void mx_bytes(const uint32_t* x, uint32_t p, uint32_t* plane) {
  uint32_t d[4];  // the four signed bytes of each residue
#pragma unroll
  for (int k = 0; k < 4; ++k) d[k] = ((x[k] > p / 2 ? x[k] - p : x[k]) + 0x80808080u) ^ 0x80808080u;
#pragma unroll
  for (int l = 0; l < 4; ++l)
    plane[l] = (d[0] >> (8 * l) & 0xffu) | (d[1] >> (8 * l) & 0xffu) << 8 | (d[2] >> (8 * l) & 0xffu) << 16 |
               (d[3] >> (8 * l)) << 24;
}

// pa: 4 planes of na coefficients, [16 rows][16 q] bytes each; pb: 4 planes of nb coefficients from ub on,
// [1 << cl columns][16 q] bytes each
__global__ void __launch_bounds__(256) k_pm_bytes(const uint32_t* __restrict__ A, int64_t sa, int64_t la, int64_t na,
                                                  int R, const uint32_t* __restrict__ B, int64_t sb, int64_t lb,
                                                  int64_t ub, int64_t nb, int NC, int cl, int Q, uint32_t p,
                                                  uint32_t* __restrict__ pa, uint32_t* __restrict__ pb) {
  const int64_t ia = (na + 15) / 16 * 1024, ib = (nb + 15) / 16 << (cl + 6);  // items: four q of a row or column
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ia + ib; i += (int64_t)gridDim.x * 256) {
    // 16 coefficients by 4 groups of q to a wave: runs of 64 bytes in, of 16 bytes out
    const bool isa = i < ia;
    const int64_t k = isa ? i : i - ia, n = isa ? na : nb;
    const int l = isa ? 4 : cl;
    const int64_t blk = k >> (6 + l);              // block of 16 coefficients
    const int in = (int)(k & ((64 << l) - 1));     // within it: [row or column][q group][coefficient]
    const int rc = in >> 6, qg = in >> 4 & 3;
    const int64_t j = blk * 16 + (in & 15);
    if (j >= n) continue;
    const int64_t u = isa ? j : ub + j;
    const bool on = u >= 0 && u < (isa ? la : lb) && rc < (isa ? R : NC);
    uint32_t x[4], plane[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const int q = 4 * qg + z;
      x[z] = on && q < Q ? (isa ? A[(int64_t)(rc * Q + q) * sa + u] : B[(int64_t)(q * NC + rc) * sb + u]) : 0u;
    }
    mx_bytes(x, p, plane);
    uint32_t* out = isa ? pa : pb;
#pragma unroll
    for (int z = 0; z < 4; ++z) out[(((int64_t)z * n + j << l) + rc) * 4 + qg] = plane[z];
  }
}

template <bool MERS, int T>
__global__ void __launch_bounds__(256) k_polymul_mx(const i32x4_t* __restrict__ pa, int64_t la, int64_t na,
                                                    const i32x4_t* __restrict__ pb, int64_t lb, int64_t ub, int64_t nb,
                                                    uint32_t* __restrict__ C, int64_t sc, int64_t k0, int64_t len,
                                                    int R, int NC, int cl, MxField P) {
  __shared__ uint32_t sums[4][4 * T][WAVE];
  const int lane = threadIdx.x & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int row = lane & 15, jj = lane >> 4, c = row & ((1 << cl) - 1), tt = row >> cl;
  const int64_t tb = (int64_t)(blockIdx.x >> 2) * (4 * T << (4 - cl)) + (blockIdx.x & 3);  // the tile's first coefficient
  const int64_t t0 = tb + tt * 4 * T;  // this lane's column's
  const int64_t tlast = k0 + tb + 4 * T * ((16 >> cl) - 1) + 4 * (T - 1);
  // steps of four j that meet coefficients of B
  const int64_t s0 = std::max<int64_t>(0, k0 + tb - (lb - 1)) / 4, s1 = std::min<int64_t>(la - 1, tlast) / 4 + 1;
  const int64_t ns = std::max<int64_t>(0, s1 - s0), w0 = s0 + ns * wave / 4, w1 = s0 + ns * (wave + 1) / 4;
  uint32_t res[T][4];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) res[i][v] = 0u;
  auto load_a = [&](int64_t s, i32x4_t* a) {
#pragma unroll
    for (int l = 0; l < 4; ++l) a[l] = pa[(l * na + 4 * s + jj) * 16 + row];
  };
  auto load_b = [&](int64_t s, int i, i32x4_t* b) {
#pragma unroll
    for (int l = 0; l < 4; ++l) b[l] = pb[((l * nb + (k0 + t0 + 4 * i - 4 * s - jj - ub)) << cl) + c];
  };
  for (int64_t f0 = w0; f0 < w1; f0 += MX_FLUSH) {
    const int64_t f1 = std::min<int64_t>(w1, f0 + MX_FLUSH);
    i32x4_t acc[T][7], a[4], b[T][4], an[4], bn[4];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int w = 0; w < 7; ++w) acc[i][w] = (i32x4_t)(0);
    load_a(f0, a);
#pragma unroll
    for (int i = 0; i < T; ++i) load_b(f0, i, b[i]);
#pragma unroll T
    for (int64_t s = f0; s < f1; ++s) {
      const int64_t sn = std::min<int64_t>(s + 1, f1 - 1);
      load_a(sn, an);
      load_b(sn, 0, bn);
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int y = 0; y < 4; ++y)
            acc[i][x + y] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[x], b[i][y], acc[i][x + y], 0, 0, 0);
#pragma unroll
      for (int i = T - 1; i > 0; --i)
#pragma unroll
        for (int l = 0; l < 4; ++l) b[i][l] = b[i - 1][l];
#pragma unroll
      for (int l = 0; l < 4; ++l) a[l] = an[l], b[0][l] = bn[l];
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t lo = (int64_t)acc[i][0][v] + ((int64_t)acc[i][1][v] << 8) + ((int64_t)acc[i][2][v] << 16) +
                           ((int64_t)acc[i][3][v] << 24);  // below 2^55 in magnitude
        const int64_t hi = (int64_t)acc[i][4][v] + ((int64_t)acc[i][5][v] << 8) + ((int64_t)acc[i][6][v] << 16);
        uint32_t x;
        if (MERS) x = fred<true>((uint64_t)(lo + 2 * hi) + P.bias, P.F);  // 2^32 = 2 mod p
        else
          x = mod_u64((uint64_t)mod_u64((uint64_t)hi + P.bias, P.F.p, P.F.mu) * P.r32 +
                          mod_u64((uint64_t)lo + P.bias, P.F.p, P.F.mu),
                      P.F.p, P.F.mu);
        const uint32_t sum = res[i][v] + x;
        res[i][v] = sum >= P.F.p ? sum - P.F.p : sum;
      }
  }
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) sums[wave][4 * i + v][lane] = res[i][v];
  __syncthreads();
#pragma unroll
  for (int z = 0; z < T; ++z) {  // a quarter of the tile to each wave
    const int e = wave * T + z, i = e / 4, v = e % 4;
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      sum += sums[w][e][lane];
      sum = sum >= P.F.p ? sum - P.F.p : sum;
    }
    const int r = 4 * jj + v;
    const int64_t t = t0 + 4 * i;
    if (r < R && c < NC && t < len) C[(int64_t)(r * NC + c) * sc + t] = sum;
  }
}

template <int T>
static void launch_mx(unsigned tiles, const i32x4_t* pa, int64_t la, int64_t na, const i32x4_t* pb, int64_t lb, int64_t ub,
                      int64_t nb, uint32_t* C, int64_t sc, int64_t k0, int64_t len, int R, int NC, int cl,
                      const MxField& P, hipStream_t st) {
  if (P.F.mersenne)
    hipLaunchKernelGGL((k_polymul_mx<true, T>), dim3(tiles), dim3(256), 0, st, pa, la, na, pb, lb, ub, nb, C, sc, k0,
                       len, R, NC, cl, P);
  else
    hipLaunchKernelGGL((k_polymul_mx<false, T>), dim3(tiles), dim3(256), 0, st, pa, la, na, pb, lb, ub, nb, C, sc, k0,
                       len, R, NC, cl, P);
}

// The most bytes of planes that polymul_mx writes for la coefficients of A and len of the product.
static size_t mx_plane_bytes(int64_t la, int64_t len, int NC) {
  int cl = 0;
  while ((1 << cl) < NC) ++cl;
  return (size_t)(la + 3) * 1024 + ((size_t)(len + la + 3 + (16 << (4 - cl))) << (cl + 6));
}

// polymul on the matrix cores, any la, lb >= 1; planes: mx_plane_bytes of memory
static void polymul_mx(const uint32_t* A, int64_t sa, int64_t la, const uint32_t* B, int64_t sb, int64_t lb,
                       uint32_t* C, int64_t sc, int64_t k0, int64_t len, int R, int Q, int NC, const Field& F,
                       uint8_t* planes, hipStream_t st) {
  int cl = 0;
  while ((1 << cl) < NC) ++cl;
  MxField P{F, (((uint64_t)1 << 55) / F.p + 1) * F.p, (uint32_t)(((uint64_t)1 << 32) % F.p)};
  // more coefficients to a wave once there is a workgroup for every compute unit
  const int T = len > (int64_t)2048 << (4 - cl) ? 4 : len > (int64_t)512 << (4 - cl) ? 2 : 1;
  const int64_t per = (int64_t)4 * T << (4 - cl), blocks = (len + per - 1) / per;
  const int64_t na = (la + 3) / 4 * 4, ub = k0 - na + 1, nb = k0 + blocks * per - ub;
  const size_t ba = (size_t)na * 1024;
  const int64_t items = (na + 15) / 16 * 1024 + ((nb + 15) / 16 << (cl + 6));
  hipLaunchKernelGGL(k_pm_bytes, dim3((unsigned)std::min<int64_t>((items + 255) / 256, 4096)), dim3(256), 0, st, A, sa, la,
                     na, R, B, sb, lb, ub, nb, NC, cl, Q, F.p, (uint32_t*)planes, (uint32_t*)(planes + ba));
  FFX_HIP(hipGetLastError());
  const i32x4_t *pa = (const i32x4_t*)planes, *pb = (const i32x4_t*)(planes + ba);
  const unsigned tiles = (unsigned)(blocks * 4);
  if (T == 4) launch_mx<4>(tiles, pa, la, na, pb, lb, ub, nb, C, sc, k0, len, R, NC, cl, P, st);
  else if (T == 2) launch_mx<2>(tiles, pa, la, na, pb, lb, ub, nb, C, sc, k0, len, R, NC, cl, P, st);
  else launch_mx<1>(tiles, pa, la, na, pb, lb, ub, nb, C, sc, k0, len, R, NC, cl, P, st);
  FFX_HIP(hipGetLastError());
}

static void polymul(const uint32_t* A, int64_t sa, int64_t la, const uint32_t* B, int64_t sb, int64_t lb, uint32_t* C,
                    int64_t sc, int64_t k0, int64_t len, int R, int Q, int NC, const Field& F, uint8_t* planes,
                    hipStream_t st) {
  if (len <= 0) return;
  const int64_t nt = g_ntt_min.load();
  if (nt > 0 && la >= nt && lb >= nt && polymul_ntt(A, sa, la, B, sb, lb, C, sc, k0, len, R, Q, NC, F, st)) return;
  if (Q >= MX_MINQ) return polymul_mx(A, sa, std::max<int64_t>(la, 1), B, sb, lb, C, sc, k0, len, R, Q, NC, F, planes, st);
  const int64_t tiles = (len + PM_TILE - 1) / PM_TILE;
  if (tiles <= PMS_MAX_TILES && la <= PMS_MAXA && polymul_small_lds(Q, std::max<int64_t>(la, 1)) <= 64 * 1024) {
    const int la1 = (int)std::max<int64_t>(la, 1);
    const size_t lds = polymul_small_lds(Q, la1);
    const dim3 grid((unsigned)(R * NC), (unsigned)tiles);
    if (F.mersenne)
      hipLaunchKernelGGL((k_polymul_small<true>), grid, dim3(PMS_NT), lds, st, A, sa, la1, B, sb, lb, C, sc, k0, len,
                         Q, NC, F);
    else
      hipLaunchKernelGGL((k_polymul_small<false>), grid, dim3(PMS_NT), lds, st, A, sa, la1, B, sb, lb, C, sc, k0, len,
                         Q, NC, F);
    FFX_HIP(hipGetLastError());
    return;
  }
  const int64_t tiles4 = (len + PM_OUT - 1) / PM_OUT;
  if (tiles4 * R * NC >= 2048) {  // enough four-per-lane tiles to fill the GPU
    dim3 grid4((unsigned)tiles4, (unsigned)(R * NC));
    if (F.mersenne)
      hipLaunchKernelGGL((k_polymul4<true>), grid4, dim3(PM_TILE), 0, st, A, sa, std::max<int64_t>(la, 1), B, sb, lb,
                         C, sc, k0, len, Q, NC, F);
    else
      hipLaunchKernelGGL((k_polymul4<false>), grid4, dim3(PM_TILE), 0, st, A, sa, std::max<int64_t>(la, 1), B, sb, lb,
                         C, sc, k0, len, Q, NC, F);
    FFX_HIP(hipGetLastError());
    return;
  }
  dim3 grid((unsigned)((len + PM_TILE - 1) / PM_TILE), (unsigned)(R * NC));
  hipLaunchKernelGGL(k_polymul, grid, dim3(PM_TILE), 0, st, A, sa, std::max<int64_t>(la, 1), B, sb, lb, C, sc, k0, len,
                     Q, NC, F);
  FFX_HIP(hipGetLastError());
}

struct SbCtx {
  Field F;
  int m, n;
  hipStream_t st;
  int32_t* d_dev;       // m shifted degrees on the device: a leaf reads them here and writes the
  int32_t* d_next;      // new ones there, and the two change places
  uint8_t* top;         // free part of the workspace
  bool d_host = true;   // the host copy of the degrees is current
};

// Workspace of pmbasis: a node's M1, R and M2, and above them, in turn, its halves' and the planes
// of its products where they take the matrix cores. One allocation for a whole order basis: with four per node, their calls held up
// the launches (16 x 8, order 8,003: 35.8 ms, 29.2 with one).
struct SbNode {
  size_t m1, r, m2;
  SbNode(int m, int n, int64_t s1, int64_t s2) {
    auto pad = [](int64_t words) { return (size_t)(words * 4 + 255) / 256 * 256; };
    m1 = pad((int64_t)m * m * (s1 + 1)), r = pad((int64_t)m * n * s2), m2 = pad((int64_t)m * m * (s2 + 1));
  }
};
static size_t pmbasis_bytes(int m, int n, int64_t sigma) {
  if (sigma <= SB_LEAF) return 0;
  const int64_t s1 = sigma / 2, s2 = sigma - s1;
  const SbNode N(m, n, s1, s2);
  const size_t planes = m < MX_MINQ ? 0 : std::max(mx_plane_bytes(s1 + 1, s2, n), mx_plane_bytes(s2 + 1, sigma + 1, m));
  return N.m1 + N.r + N.m2 + std::max(planes, pmbasis_bytes(m, n, s2));
}

// Nodes of at most this order take no degrees from the device: their lengths are the bound
// sigma + 1 (the extra coefficients come out zero), so a subtree of such nodes is queued without
// waiting for the GPU; larger nodes read the degrees back to size their products exactly.
constexpr int64_t SB_EXACT_ABOVE = 256;

// The host copy of the degrees, read back when a leaf has run since the last read.
static void host_degrees(SbCtx& X, std::vector<int32_t>& d) {
  if (X.d_host) return;
  FFX_HIP(hipMemcpyAsync(d.data(), X.d_dev, X.m * sizeof(int32_t), hipMemcpyDeviceToHost, X.st));
  FFX_HIP(hipStreamSynchronize(X.st));
  X.d_host = true;
}

// Basis of G (m x n entries, stride sg, order sigma) into M (m x m entries, stride sm >= sigma + 1,
// zero beyond the returned length); the shifted degrees are updated in X.d_dev (and in d when it is
// read back). Returns a bound on the number of coefficients of M that can be nonzero.
static int64_t pmbasis(SbCtx& X, const uint32_t* G, int64_t sg, int64_t sigma, std::vector<int32_t>& d, uint32_t* M,
                       int64_t sm) {
  const int m = X.m, n = X.n;
  if (sigma <= SB_LEAF) {
    const dim3 grid((unsigned)m);
    if (X.F.mersenne)
      hipLaunchKernelGGL((k_mbasis_leaf<true>), grid, dim3(LEAF_NT), 0, X.st, G, sg, m, n, (int)sigma, X.d_dev,
                         X.d_next, M, sm, X.F);
    else
      hipLaunchKernelGGL((k_mbasis_leaf<false>), grid, dim3(LEAF_NT), 0, X.st, G, sg, m, n, (int)sigma, X.d_dev,
                         X.d_next, M, sm, X.F);
    std::swap(X.d_dev, X.d_next);
    FFX_HIP(hipGetLastError());
    X.d_host = false;
    return sigma + 1;
  }
  const bool exact = sigma > SB_EXACT_ABOVE;
  int32_t dmin = 0;
  if (exact) {
    host_degrees(X, d);
    dmin = *std::min_element(d.begin(), d.end());
  }
  const int64_t s1 = sigma / 2, s2 = sigma - s1;
  const SbNode N(m, n, s1, s2);
  uint8_t* const base = X.top;
  uint32_t *M1 = (uint32_t*)base, *R = (uint32_t*)(base + N.m1), *M2 = (uint32_t*)(base + N.m1 + N.r);
  X.top = base + N.m1 + N.r + N.m2;
  const int64_t l1 = pmbasis(X, G, sg, s1, d, M1, s1 + 1);
  // R = [x^s1 .. x^(sigma-1)] (M1 G)
  polymul(M1, s1 + 1, l1, G, sg, sigma, R, s2, s1, s2, m, m, n, X.F, X.top, X.st);
  const int64_t l2 = pmbasis(X, R, s2, s2, d, M2, s2 + 1);
  int64_t len = std::min<int64_t>(sigma + 1, l1 + l2 - 1);
  if (exact) {
    host_degrees(X, d);
    const int32_t dmax = *std::max_element(d.begin(), d.end());
    len = std::min<int64_t>(len, (int64_t)dmax - dmin + 1);
  }
  polymul(M2, s2 + 1, l2, M1, s1 + 1, l1, M, sm, 0, len, m, m, m, X.F, X.top, X.st);
  if (len < sm) FFX_HIP(hipMemset2DAsync(M + len, sm * 4, 0, (sm - len) * 4, (size_t)m * m, X.st));
  X.top = base;
  return len;
}

static bool is_prime(uint32_t p) {
  if (p < 2) return false;
  for (uint32_t q : {2u, 3u, 5u, 7u}) {
    if (p % q == 0) return p == q;
  }
  uint32_t dd = p - 1;
  int r = 0;
  while (!(dd & 1)) {
    dd >>= 1;
    ++r;
  }
  auto mulm = [&](uint64_t a, uint64_t b) { return a * b % p; };
  for (uint64_t a : {2ull, 3ull, 5ull, 7ull}) {  // deterministic below 3,215,031,751
    uint64_t x = 1, b = a, e = dd;
    while (e) {
      if (e & 1) x = mulm(x, b);
      b = mulm(b, b);
      e >>= 1;
    }
    if (x == 1 || x == p - 1) continue;
    bool comp = true;
    for (int i = 1; i < r && comp; ++i) {
      x = mulm(x, x);
      if (x == p - 1) comp = false;
    }
    if (comp) return false;
  }
  return true;
}

void sigma_basis(uint32_t p, int m, int n, int64_t sigma, const uint32_t* G, int64_t ldg, const int32_t* shift,
                 uint32_t* M, int64_t ldm, int32_t* d_out, hipStream_t st) {
  if (p > 2147483647u) fail(FFX_EINVAL, "the order basis needs a prime p < 2^31 (p = %u)", p);
  if (!is_prime(p)) fail(FFX_EINVAL, "the order basis needs a prime modulus (%u is not prime)", p);
  if (m < 1 || m > SB_MAXM || n < 1 || n > SB_MAXN || n > m)
    fail(FFX_EINVAL, "m = %d, n = %d: need 1 <= n <= m <= %d and n <= %d", m, n, SB_MAXM, SB_MAXN);
  if (sigma < 1) fail(FFX_EINVAL, "sigma = %lld < 1", (long long)sigma);
  if (ldg < sigma || ldm < sigma + 1) fail(FFX_EINVAL, "ldg < sigma or ldm < sigma + 1");
  if (!G || !M || !shift || !d_out) fail(FFX_EINVAL, "NULL argument");
  std::vector<int32_t> d(shift, shift + m);
  for (int32_t v : d)
    if (v < 0 || v > (1 << 28)) fail(FFX_EINVAL, "shift %d outside [0, 2^28]", v);
  int32_t* degrees = nullptr;  // two buffers of degrees, then the recursion's workspace
  if (hipMallocAsync((void**)&degrees, 256 + pmbasis_bytes(m, n, sigma), st) != hipSuccess)
    fail(FFX_ENOMEM, "order basis workspace allocation failed (order %lld)", (long long)sigma);
  SbCtx X{make_field(p), m, n, st, degrees, degrees + SB_MAXM, (uint8_t*)degrees + 256};
  try {
    FFX_HIP(hipMemcpyAsync(X.d_dev, d.data(), m * sizeof(int32_t), hipMemcpyHostToDevice, st));
    const int64_t len = pmbasis(X, G, ldg, sigma, d, M, ldm);
    if (len < ldm) FFX_HIP(hipMemset2DAsync(M + len, ldm * 4, 0, (ldm - len) * 4, (size_t)m * m, st));
    host_degrees(X, d);
  } catch (...) {
    (void)hipFreeAsync(degrees, st);
    throw;
  }
  (void)hipFreeAsync(degrees, st);
  FFX_HIP(hipStreamSynchronize(st));
  std::copy(d.begin(), d.end(), d_out);
}

// x-adic valuation of det F (s x s entries of K coefficients, row-major [r][c][k]) over F_p by
// elimination over F_p[[x]]/x^K; -1 when det F = 0 mod x^K.
static int64_t det_valuation(std::vector<uint64_t> A, int s, int64_t K, uint32_t p) {
  auto at = [&](int r, int c) { return &A[((size_t)r * s + c) * K]; };
  auto pw = [&](uint64_t a, uint64_t e) {
    uint64_t r = 1;
    a %= p;
    while (e) {
      if (e & 1) r = r * a % p;
      a = a * a % p;
      e >>= 1;
    }
    return r;
  };
  int64_t val = 0;
  std::vector<uint64_t> u(K), ui(K), f(K);
  for (int c = 0; c < s; ++c) {
    int best = -1;
    int64_t bv = K;
    for (int r = c; r < s; ++r) {
      const uint64_t* x = at(r, c);
      for (int64_t k = 0; k < bv; ++k)
        if (x[k]) {
          best = r;
          bv = k;
          break;
        }
    }
    if (best < 0) return -1;
    if (best != c)
      for (int cc = 0; cc < s; ++cc) std::swap_ranges(at(c, cc), at(c, cc) + K, at(best, cc));
    val += bv;
    if (val >= K) return -1;
    // u = A[c][c] / x^bv, ui = 1/u
    std::fill(u.begin(), u.end(), 0);
    for (int64_t k = bv; k < K; ++k) u[k - bv] = at(c, c)[k];
    const uint64_t i0 = pw(u[0], p - 2);
    for (int64_t k = 0; k < K; ++k) {
      uint64_t acc = 0;
      for (int64_t j = 1; j <= k; ++j) acc = (acc + u[j] * ui[k - j]) % p;
      ui[k] = k == 0 ? i0 : (p - acc) % p * i0 % p;
    }
    for (int r = c + 1; r < s; ++r) {
      // f = (A[r][c] / x^bv) * ui; row r -= f * row c
      std::fill(f.begin(), f.end(), 0);
      for (int64_t k = 0; k + bv < K; ++k) {
        const uint64_t q = at(r, c)[k + bv];
        if (!q) continue;
        for (int64_t j = 0; k + j < K; ++j) f[k + j] = (f[k + j] + q * ui[j]) % p;
      }
      for (int cc = c; cc < s; ++cc) {
        uint64_t* y = at(r, cc);
        const uint64_t* x = at(c, cc);
        for (int64_t k = 0; k < K; ++k) {
          if (!f[k]) continue;
          for (int64_t j = 0; k + j < K; ++j) y[k + j] = (y[k + j] + (p - f[k]) * x[j]) % p;
        }
      }
    }
  }
  return val;
}

void sequence_rank(uint32_t p, int s, int64_t L, const void* S, ffx_dtype dt, int32_t* deg_out, int64_t* rank,
                   int64_t* deg_det, int64_t* codeg_det, hipStream_t st) {
  if (s < 1 || s > SB_MAXN) fail(FFX_EINVAL, "s = %d outside [1, %d]", s, SB_MAXN);
  if (L < 1) fail(FFX_EINVAL, "L = %lld < 1", (long long)L);
  if (!S) fail(FFX_EINVAL, "S is NULL");
  if (p > 2147483647u) fail(FFX_EINVAL, "the rank needs a prime p < 2^31 (p = %u)", p);
  if (!is_prime(p)) fail(FFX_EINVAL, "the rank needs a prime modulus (%u is not prime)", p);
  const int m = 2 * s;
  uint32_t *G = nullptr, *M = nullptr;
  if (hipMallocAsync((void**)&G, (size_t)m * s * L * 4, st) != hipSuccess ||
      hipMallocAsync((void**)&M, (size_t)m * m * (L + 1) * 4, st) != hipSuccess) {
    if (G) (void)hipFreeAsync(G, st);
    if (M) (void)hipFreeAsync(M, st);
    fail(FFX_ENOMEM, "rank workspace allocation failed (L = %lld)", (long long)L);
  }
  std::vector<int32_t> d(m);
  std::vector<uint32_t> Mh;
  try {
    const int64_t total = (int64_t)m * s * L;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 16384);
    if (dt == FFX_I32)
      hipLaunchKernelGGL((k_sequence_series<int32_t>), dim3(blocks), dim3(256), 0, st, (const int32_t*)S, L, s, p, G);
    else
      hipLaunchKernelGGL((k_sequence_series<int64_t>), dim3(blocks), dim3(256), 0, st, (const int64_t*)S, L, s, p, G);
    FFX_HIP(hipGetLastError());
    std::vector<int32_t> shift(m, 0);
    for (int i = s; i < m; ++i) shift[i] = 1;
    sigma_basis(p, m, s, L, G, L, shift.data(), M, L + 1, d.data(), st);
    Mh.resize((size_t)m * m * (L + 1));
    FFX_HIP(hipMemcpyAsync(Mh.data(), M, Mh.size() * 4, hipMemcpyDeviceToHost, st));
    FFX_HIP(hipStreamSynchronize(st));
  } catch (...) {
    (void)hipFreeAsync(G, st);
    (void)hipFreeAsync(M, st);
    throw;
  }
  (void)hipFreeAsync(G, st);
  (void)hipFreeAsync(M, st);
  // the generator: the s rows of smallest shifted degree (ties by index), left s x s part
  std::vector<int> rows(m);
  for (int i = 0; i < m; ++i) rows[i] = i;
  std::stable_sort(rows.begin(), rows.end(), [&](int a, int b) { return d[a] < d[b]; });
  rows.resize(s);
  int64_t D = 0;
  for (int i = 0; i < s; ++i) {
    deg_out[i] = d[rows[i]];
    D += d[rows[i]];
    if (d[rows[i]] > L) fail(FFX_EUNSUPPORTED, "generator degree %d exceeds the sequence length", d[rows[i]]);
  }
  auto coef = [&](int r, int c, int64_t k) { return Mh[((size_t)rows[r] * m + c) * (L + 1) + k]; };
  // row reduced: the reversed form's constant coefficients must be nonsingular, else deg det F is
  // not the sum of the row degrees
  {
    std::vector<uint64_t> A0((size_t)s * s);
    for (int r = 0; r < s; ++r)
      for (int c = 0; c < s; ++c) A0[(size_t)r * s + c] = coef(r, c, 0);
    if (det_valuation(A0, s, 1, p) != 0)
      fail(FFX_EUNSUPPORTED, "the generator is not row reduced (sequence too short or degenerate projections)");
  }
  // codeg det F: F row i = lambda^deg_i Frev_i(1/lambda), so [lambda^k] F_i = [x^(deg_i - k)] Frev_i.
  // F is row reduced, so det F has degree D exactly and its valuation is at most D: a truncation
  // order K > D always finds it.
  int64_t e = -1;
  for (int64_t K = 16;; K *= 2) {
    std::vector<uint64_t> A((size_t)s * s * K, 0);
    for (int r = 0; r < s; ++r)
      for (int c = 0; c < s; ++c)
        for (int64_t k = 0; k < K && k <= deg_out[r]; ++k) A[((size_t)r * s + c) * K + k] = coef(r, c, deg_out[r] - k);
    e = det_valuation(A, s, K, p);
    if (e >= 0 || K > D) break;
  }
  if (e < 0) fail(FFX_EUNSUPPORTED, "det F vanishes: no rank from this sequence");
  *deg_det = D;
  *codeg_det = e;
  *rank = D - e;
}

}  // namespace ffx

extern "C" ffx_status ffx_set_ntt_threshold(int64_t min_length) {
  return ffx::guard([&] {
    if (min_length < 0) ffx::fail(FFX_EINVAL, "NTT threshold %lld < 0", (long long)min_length);
    ffx::g_ntt_min.store(min_length);
  });
}
