// The one-vector product on column-sorted row groups (layout in sg.h).
#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "sg.h"

namespace ffx {

constexpr int SG_THREADS = 1024;  // one workgroup per compute unit: 16 waves
constexpr int SG_U = 2;           // chunks per wave in flight
// Dynamic LDS of one group is at least this much, so that a compute unit never
// holds two groups (the groups are sized to be about one per compute unit, and
// two on one CU would leave another CU idle).
constexpr size_t SG_LDS_FLOOR = 96 * 1024;

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// This lane's four entry words of chunk ch, and their values two to a word (streamed once); without VALS a value is
// 1 or m - 1, by the tag
template <bool VALS>
struct SgLane {
  uint32_t w[4], p[2];
  __device__ inline void words(const SgMat& G, uint32_t ch, uint32_t lane) {
    const u32x4_t q = __builtin_nontemporal_load((const u32x4_t*)(G.ent + (size_t)ch * SG_CHUNK) + lane);
    w[0] = q.x;
    w[1] = q.y;
    w[2] = q.z;
    w[3] = q.w;
  }
  __device__ inline void values(const SgMat& G, uint32_t ch, uint32_t lane) {
    if constexpr (!VALS) return;
    const u32x2_t q = __builtin_nontemporal_load((const u32x2_t*)(G.val + (size_t)ch * SG_CHUNK) + lane);
    p[0] = q.x;
    p[1] = q.y;
  }
  __device__ inline bool pad(int k) const { return (w[k] >> TAG_SHIFT) == TAG_PAD; }
  __device__ inline uint32_t val(int k, uint32_t m) const {  // of an entry; 0 for padding with VALS
    if constexpr (VALS) return (k & 1) ? p[k / 2] >> 16 : p[k / 2] & 0xFFFFu;
    else return (w[k] >> TAG_SHIFT) == TAG_PLUS ? 1u : m - 1;
  }
  __device__ inline uint32_t col(int k) const { return w[k] & SG_COL_MASK; }
  __device__ inline uint32_t row(int k) const { return (w[k] >> SG_ROW_SHIFT) & (SG_MAX_ROWS - 1); }
};

// v*x below 2^32 for residues of at most 16 bits, in one full-rate instruction
__device__ inline uint32_t sg_mul(uint32_t v, uint32_t x) { return __umul24(v, x); }

template <typename Tv>
__device__ inline void sg_write(const SgMat& G, const SgGroup& g, const unsigned long long* acc, Tv* y, uint32_t alpha,
                                uint32_t beta, uint16_t* y16) {
  for (uint32_t r = threadIdx.x; r < g.nrows; r += SG_THREADS) {
    const uint32_t row = g.row0 + r, to = G.rowmap ? G.rowmap[row] : row;
    const uint32_t res = mod_u64(acc[r], G.m, G.mu);
    const uint32_t out = (alpha == 1 && beta == 0) ? res : axpby(alpha, res, beta, beta ? (uint32_t)y[to] : 0u, G.m, G.mu);
    y[to] = (Tv)out;
    if (y16) y16[to] = (uint16_t)out;  // the next product's 16-bit x
  }
}

// GF2: a matrix mod 2 times one bit-packed word per row (32 vectors over GF(2)):
// x and y are words (stride ldx, ldy), a row's sum is the exclusive or of its
// columns' words (32-bit LDS sums).
// Bound by the gathers' misses in the vector cache: the texture data path is busy
// 76% of the kernel and for 53% of it waits for the cache, which has about 73 reads
// of the L2 in flight, 384 cycles each; the vector ALU is busy 14%, the LDS 16%. (With
// compacted values the kernel took 50 us with all gathers in a 4 KB table and 86
// with x.) What would shorten the wait is not known: half as many lines per compute
// unit, or four chunks in flight instead of two, take the same time. On the
// 2,000,000-row power-law matrix a product took 85.6 us when the kernel decoded
// compacted values, 80.0 with each entry's loaded. A wave copying the columns its
// next 256 or 128 entries span to LDS and gathering from there, four windows ahead:
// 108 us. Chunks of +-1 entries marked, so that their values are not read: 96.7 (the
// mark has to be there before the loads, and splits the additions).
template <typename Tx, typename Tv, int U, bool GF2, bool VALS>
__global__ __launch_bounds__(SG_THREADS) void k_sg(SgMat G, const Tx* __restrict__ x, Tv* __restrict__ y,
                                                   uint32_t alpha, uint32_t beta, uint16_t* __restrict__ y16,
                                                   int64_t ldx, int64_t ldy) {
  extern __shared__ __align__(16) unsigned long long acc[];
  uint32_t* accx = (uint32_t*)acc;  // GF2
  constexpr uint32_t NW = SG_THREADS / WAVE;
  const SgGroup g = G.groups[blockIdx.x];
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  for (uint32_t r = tid; r < g.nrows; r += SG_THREADS) {
    if constexpr (GF2) accx[r] = 0u;
    else acc[r] = 0ull;
  }
  __syncthreads();
  // the entries of the next U chunks are requested before the gathers of the current ones, so each
  // pass waits on one round trip to memory instead of two
  using Lane = SgLane<VALS>;
  Lane e[U], en[U];
  uint32_t cb[U], cbn[U];
  auto load = [&](uint32_t ch0, Lane (&q)[U], uint32_t (&c)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t ch = ch0 + u * NW;
      c[u] = 0;
      if (ch < g.nchunks) {
        q[u].words(G, g.c0 + ch, lane);
        if constexpr (!GF2) q[u].values(G, g.c0 + ch, lane);
        c[u] = G.cbase[g.c0 + ch];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) q[u].w[k] = PAD_WORD;
      }
    }
  };
  load(wave, e, cb);
  for (uint32_t ch0 = wave; ch0 < g.nchunks; ch0 += NW * U) {
    load(ch0 + NW * U, en, cbn);
    uint32_t xv[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t col = cb[u] + e[u].col(k);
        xv[u][k] = !e[u].pad(k) ? (uint32_t)(GF2 ? x[col * ldx] : x[col]) : 0u;
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (!e[u].pad(k)) {
          if constexpr (GF2) atomicXor(&accx[e[u].row(k)], xv[u][k]);  // every entry is 1
          else atomicAdd(&acc[e[u].row(k)], (unsigned long long)sg_mul(e[u].val(k, G.m), xv[u][k]));
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      e[u] = en[u];
      cb[u] = cbn[u];
    }
  }
  __syncthreads();
  if constexpr (GF2) {
    for (uint32_t r = tid; r < g.nrows; r += SG_THREADS) {
      const uint32_t row = g.row0 + r;
      y[(int64_t)(G.rowmap ? G.rowmap[row] : row) * ldy] = (Tv)accx[r];
    }
  } else {
    sg_write(G, g, acc, y, alpha, beta, y16);
  }
}

// The largest dynamic LDS a group can ask for: SG_MAX_ROWS 64-bit sums.
constexpr size_t SG_LDS_MAX = (size_t)SG_MAX_ROWS * 8;

template <typename Tx, typename Tv, bool GF2, bool VALS>
static hipError_t sg_launch(const SgMat& G, const Tx* x, Tv* y, uint32_t alpha, uint32_t beta, uint16_t* y16,
                            hipStream_t st, int64_t ldx, int64_t ldy) {
  const size_t lds = std::max<size_t>((size_t)G.max_rows * 8, SG_LDS_FLOOR);
  auto k = k_sg<Tx, Tv, SG_U, GF2, VALS>;
  hipError_t e = raise_lds_limit((const void*)k, (int)SG_LDS_MAX);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(G.ngroups), dim3(SG_THREADS), lds, st, G, x, y, alpha, beta, y16, ldx, ldy);
  return hipGetLastError();
}

template <typename Tx, typename Tv, bool GF2 = false>
static hipError_t sg_go(const SgMat& G, const Tx* x, Tv* y, uint32_t alpha, uint32_t beta, uint16_t* y16,
                        hipStream_t st, int64_t ldx = 1, int64_t ldy = 1) {
  if constexpr (!GF2)
    if (G.val) return sg_launch<Tx, Tv, false, true>(G, x, y, alpha, beta, y16, st, ldx, ldy);
  return sg_launch<Tx, Tv, GF2, false>(G, x, y, alpha, beta, y16, st, ldx, ldy);
}

template <typename Tv>
static hipError_t sg_by_x(const SgMat& G, const void* x, const uint16_t* x16, Tv* y, uint32_t alpha, uint32_t beta,
                          uint16_t* y16, hipStream_t st) {
  if (!x16) return sg_go<Tv, Tv>(G, (const Tv*)x, y, alpha, beta, y16, st);
  return sg_go<uint16_t, Tv>(G, x16, y, alpha, beta, y16, st);
}

hipError_t launch_sg(const SgMat& G, ffx_dtype dt, const void* x, const uint16_t* x16, void* y, uint32_t alpha,
                     uint32_t beta, hipStream_t st, uint16_t* y16) {
  if (G.ngroups == 0) return hipSuccess;
  if (dt == FFX_I32) return sg_by_x<int32_t>(G, x, x16, (int32_t*)y, alpha, beta, y16, st);
  return sg_by_x<int64_t>(G, x, x16, (int64_t*)y, alpha, beta, y16, st);
}

hipError_t launch_sg_gf2(const SgMat& G, const uint32_t* X, int64_t ldx, uint32_t* Y, int64_t ldy, hipStream_t st) {
  if (G.ngroups == 0) return hipSuccess;
  return sg_go<uint32_t, uint32_t, true>(G, X, Y, 1, 0, nullptr, st, ldx, ldy);
}

// ---------------------------------------------------------- A^T x ---------
// The same entries read the other way: workgroup (p, q) sums the columns of
// panel p (2^14 of them) over the groups q, q + Q, .. in LDS. A group's entries
// are sorted by column, so those of a panel are a run of its chunks (tindex);
// chunks at the ends of the run are read by both panels they touch. x is the
// 16-bit copy, of which the rows of up to SGT_ROUND groups are staged in LDS at
// a time: a gather of x and the addition to a sum are then one LDS access
// each, and no atomic leaves the compute unit. The sums are 32 bits: a general
// term is reduced below 3m first (one multiplication by floor(2^32/m)), which
// halves the sums' LDS and leaves room to stage x for about eleven groups.
// Groups are dealt out to the parts in turn, since a band puts most of a
// panel's entries in neighbouring groups. Bound by the latency of a round
// (stage, then three or four chunks per wave): the texture data path is busy 55% of
// the kernel (waiting 32%), the vector ALU 31%, the LDS 15%. One vector, 1,000,000
// power-law rows (17.2 M entries): 167 us through binned records, 86 with compacted
// values, 75 now.
constexpr uint32_t SGT_XROWS = 44 * 1024;  // staged 16-bit x entries
constexpr uint32_t SGT_ROUND = 32;         // groups staged at a time, at most
constexpr int SGT_U = 2;                   // chunks per wave in flight (three or four: the same)
constexpr size_t SGT_LDS = (((size_t)1 << SGT_SHIFT) + WAVE) * 4 + SGT_XROWS * 2;  // the sums and 64 spare ones

template <bool VALS>
__global__ __launch_bounds__(SG_THREADS) void k_sg_t(SgMat G, const uint16_t* __restrict__ x16, uint32_t P, uint32_t Q,
                                                     uint32_t slots, uint32_t slot_rows, uint32_t mu32,
                                                     uint32_t* __restrict__ part) {
  extern __shared__ __align__(16) unsigned long long acc[];
  uint32_t* sums = (uint32_t*)acc;
  uint16_t* xs = (uint16_t*)(sums + (1u << SGT_SHIFT) + WAVE);
  constexpr uint32_t NW = SG_THREADS / WAVE;
  constexpr int U = SGT_U;
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  const uint32_t p = blockIdx.x % P, q = blockIdx.x / P;
  const uint32_t j0 = p << SGT_SHIFT, nj = min(1u << SGT_SHIFT, G.ncols - j0);
  for (uint32_t i = tid; i < nj; i += SG_THREADS) sums[i] = 0u;
  for (uint32_t g0 = q; g0 < G.ngroups; g0 += slots * Q) {
    const uint32_t ng = min(slots, (G.ngroups - g0 + Q - 1) / Q);  // groups g0 + i*Q, i < ng
    __syncthreads();  // the last round's x is done with
    uint32_t n = 0, c0 = 0, xoff = 0;
    if (lane < ng) {  // every wave: the chunk run of group `lane`
      const uint32_t g = g0 + lane * Q;
      const SgGroup gr = G.groups[g];
      const uint2 r = G.tindex[(size_t)p * G.ngroups + g];
      n = r.y - r.x;
      c0 = gr.c0 + r.x;
      xoff = lane * slot_rows + (gr.row0 & 7u);
    }
    uint32_t pre = n;
#pragma unroll
    for (int o = 1; o < (int)SGT_ROUND; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)pre, o);
      if ((int)lane >= o) pre += y;
    }
    const uint32_t total = (uint32_t)__shfl((int)pre, (int)SGT_ROUND - 1);
    pre -= n;  // chunks of the round before this group's
    // the entries of the wave's first chunks are requested before x is staged
    SgLane<VALS> e[U];
    uint32_t cb[U], xo[U];
    auto load = [&](uint32_t j) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t jj = j + u * NW;
        cb[u] = xo[u] = 0;
        if (jj < total) {  // the same in the whole wave
          const int k = __builtin_popcountll(__ballot(lane < ng && pre <= jj)) - 1;
          const uint32_t ch = (uint32_t)__builtin_amdgcn_readlane((int)c0, k) + jj -
                              (uint32_t)__builtin_amdgcn_readlane((int)pre, k);
          e[u].words(G, ch, lane);
          e[u].values(G, ch, lane);
          cb[u] = G.cbase[ch] - j0;
          xo[u] = (uint32_t)__builtin_amdgcn_readlane((int)xoff, k);
        }
      }
    };
    load(wave);
    // x of the groups, from the 16-byte boundary before their first row
    const uint32_t per = slot_rows / 8;
    for (uint32_t i = tid; i < ng * per; i += SG_THREADS) {
      const uint32_t k = i / per, o = (i - k * per) * 8;
      const SgGroup gr = G.groups[g0 + k * Q];
      const uint32_t r = (gr.row0 & ~7u) + o;
      if (r < gr.row0 + gr.nrows) *(u32x4_t*)(xs + k * slot_rows + o) = *(const u32x4_t*)(x16 + r);
    }
    __syncthreads();
    for (uint32_t j = wave; j < total; j += NW * U) {
      if (j != wave) load(j);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (j + u * NW >= total) break;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (!VALS && e[u].pad(k)) continue;
          uint32_t t = sg_mul(e[u].val(k, G.m), xs[xo[u] + e[u].row(k)]);  // below 2^32
          t -= __umul24(__umulhi(t, mu32), G.m);  // the quotient is below 2^16 and at most two low: below 3m
          // a column of another panel (below j0 it wraps) goes to the spare sums
          const uint32_t at = min(cb[u] + e[u].col(k), (1u << SGT_SHIFT) + lane);
          atomicAdd(&sums[at], t);
        }
      }
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < nj; i += SG_THREADS) part[(size_t)q * G.ncols + j0 + i] = sums[i];
}

struct SgtPlan {
  uint32_t P, Q, slots, slot_rows;
  size_t x_bytes, part_bytes;
};
static SgtPlan sgt_plan(const SgMat& G) {
  SgtPlan t;
  t.P = (G.ncols + (1u << SGT_SHIFT) - 1) >> SGT_SHIFT;
  // one workgroup per compute unit (its LDS fills one): as many parts as that leaves room for
  t.Q = std::max<uint32_t>(1, std::min<uint32_t>(256 / t.P, G.ngroups));
  t.slot_rows = (G.max_rows + 7 + 7) & ~7u;  // a group's rows from the 8-row boundary before them
  t.slots = std::min<uint32_t>(SGT_ROUND, SGT_XROWS / t.slot_rows);
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  t.x_bytes = al((size_t)G.nrows * 2 + 16);  // the last 16-byte read may pass the last row
  t.part_bytes = al((size_t)t.Q * G.ncols * 4);
  return t;
}

size_t sg_transpose_scratch(const SgMat& G) {
  if (!G.tindex || G.ncols == 0) return 0;
  const SgtPlan t = sgt_plan(G);
  return t.x_bytes + t.part_bytes;
}

hipError_t launch_sg_transpose(const SgMat& G, ffx_dtype dt, const void* x, int64_t ldx, void* y, int64_t ldy,
                               uint32_t alpha, uint32_t beta, void* scratch, hipStream_t st) {
  const SgtPlan t = sgt_plan(G);
  uint16_t* x16 = (uint16_t*)scratch;
  uint32_t* part = (uint32_t*)((unsigned char*)scratch + t.x_bytes);
  hipError_t e = launch_compact_x(dt, x, ldx, x16, G.nrows, st);
  auto k = G.val ? k_sg_t<true> : k_sg_t<false>;
  if (e == hipSuccess) e = raise_lds_limit((const void*)k, (int)SGT_LDS);
  if (e != hipSuccess) return e;
  const uint32_t mu32 = (uint32_t)(((uint64_t)1 << 32) / G.m);
  hipLaunchKernelGGL(k, dim3(t.P * t.Q), dim3(SG_THREADS), SGT_LDS, st, G, x16, t.P, t.Q, t.slots, t.slot_rows,
                     mu32, part);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_t_parts(dt, G.m, G.mu, G.ncols, part, t.Q, 1, 1, alpha, beta, y, ldy, st);
}

}  // namespace ffx
