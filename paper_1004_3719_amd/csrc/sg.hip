// The one-vector product on column-sorted row groups (layout in sg.h).
#include <algorithm>
#include <mutex>

#include "launch.h"
#include "sg.h"

namespace ffx {

constexpr int SG_THREADS = 1024;  // one workgroup per compute unit: 16 waves
constexpr int SG_U = 2;           // chunks per wave in flight
// Dynamic LDS of one group is at least this much, so that a compute unit never
// holds two groups (the groups are sized to be about one per compute unit, and
// two on one CU would leave another CU idle).
constexpr size_t SG_LDS_FLOOR = 96 * 1024;

__device__ inline uint32_t sg_lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// GF2: a matrix mod 2 times one bit-packed word per row (32 vectors over GF(2)): x and y are words
// (stride ldx, ldy), a row's sum is the exclusive or of its columns' words (32-bit LDS sums).
template <typename Tx, typename Tv, int NT, int U, bool GF2>
__global__ __launch_bounds__(NT) void k_sg(SgMat G, const Tx* __restrict__ x, Tv* __restrict__ y, uint32_t alpha,
                                           uint32_t beta, uint16_t* __restrict__ y16, int64_t ldx, int64_t ldy) {
  extern __shared__ __align__(16) unsigned long long acc[];
  uint32_t* accx = (uint32_t*)acc;  // GF2
  constexpr uint32_t NW = NT / WAVE;
  const SgGroup g = G.groups[blockIdx.x];
  const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
  for (uint32_t r = tid; r < g.nrows; r += NT) {
    if constexpr (GF2) accx[r] = 0u;
    else acc[r] = 0ull;
  }
  __syncthreads();
  // the entry words of the next U chunks are requested before the values and gathers of the
  // current ones, so each pass waits on one round trip to memory instead of two
  uint32_t w[U][4], vo[U], cb[U];
  auto load_words = [&](uint32_t ch0, uint32_t (&ww)[U][4], uint32_t (&vv)[U], uint32_t (&cc)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t ch = ch0 + u * NW;
      const bool ok = ch < g.nchunks;
      typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
      const u32x4_t q = ok ? __builtin_nontemporal_load((const u32x4_t*)(G.ent + (size_t)(g.c0 + ch) * SG_CHUNK) + lane)
                           : (u32x4_t)(PAD_WORD);
      ww[u][0] = q.x;
      ww[u][1] = q.y;
      ww[u][2] = q.z;
      ww[u][3] = q.w;
      vv[u] = ok ? G.choff[g.c0 + ch] : 0u;
      cc[u] = ok ? G.cbase[g.c0 + ch] : 0u;
    }
  };
  load_words(wave, w, vo, cb);
  for (uint32_t ch0 = wave; ch0 < g.nchunks; ch0 += NW * U) {
    uint32_t wn[U][4], von[U], cbn[U];
    load_words(ch0 + NW * U, wn, von, cbn);
    // values: a lane's general values are consecutive, after those of the lanes below it (four
    // ballots give their count), and one 12-byte load brings all of them; then x
    uint32_t v[U][4], xv[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint32_t idx = vo[u], ng = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool gen = (w[u][k] >> TAG_SHIFT) == TAG_GEN;
        idx += sg_lanes_below(__ballot(gen));
        ng += gen ? 1u : 0u;
      }
      uint32_t q0 = 0, q1 = 0, q2 = 0;
      if (ng) {
        typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
        const u32x3_t q = __builtin_nontemporal_load((const u32x3_t*)((const uint32_t*)G.val + (idx >> 1)));
        q0 = q.x;
        q1 = q.y;
        q2 = q.z;
      }
      uint32_t j = idx & 1u;  // position of the lane's first value in the 12 bytes (16-bit units)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t tag = w[u][k] >> TAG_SHIFT;
        const uint32_t d = j < 2 ? q0 : j < 4 ? q1 : q2;
        v[u][k] = tag == TAG_GEN ? (d >> ((j & 1u) * 16)) & 0xFFFFu : 0u;
        j += tag == TAG_GEN ? 1u : 0u;
        const uint32_t col = cb[u] + (w[u][k] & SG_COL_MASK);
        xv[u][k] = tag != TAG_PAD ? (uint32_t)(GF2 ? x[(int64_t)col * ldx] : x[col]) : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t tag = w[u][k] >> TAG_SHIFT;
        if (tag != TAG_PAD) {
          const uint32_t row = (w[u][k] >> SG_ROW_SHIFT) & (SG_MAX_ROWS - 1);
          if constexpr (GF2) {  // entries are 1 (with values off, a stored value is odd)
            atomicXor(&accx[row], (tag != TAG_GEN || (v[u][k] & 1u)) ? xv[u][k] : 0u);
          } else {
            // a term is below 2^32: (m-1)^2, x or m - x
            const uint32_t t = tag == TAG_GEN ? v[u][k] * xv[u][k] : tag == TAG_PLUS ? xv[u][k] : G.m - xv[u][k];
            atomicAdd(&acc[row], (unsigned long long)t);
          }
        }
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      vo[u] = von[u];
      cb[u] = cbn[u];
#pragma unroll
      for (int k = 0; k < 4; ++k) w[u][k] = wn[u][k];
    }
  }
  __syncthreads();
  if constexpr (GF2) {
    for (uint32_t r = tid; r < g.nrows; r += NT) {
      const uint32_t row = g.row0 + r;
      y[(int64_t)(G.rowmap ? G.rowmap[row] : row) * ldy] = (Tv)accx[r];
    }
    return;
  }
  for (uint32_t r = tid; r < g.nrows; r += NT) {
    const uint32_t row = g.row0 + r;
    Tv* yr = y + (G.rowmap ? G.rowmap[row] : row);
    const uint32_t res = mod_u64(acc[r], G.m, G.mu);
    const uint32_t out = (alpha == 1 && beta == 0) ? res : axpby(alpha, res, beta, beta ? (uint32_t)*yr : 0u, G.m, G.mu);
    *yr = (Tv)out;
    if (y16) y16[G.rowmap ? G.rowmap[row] : row] = (uint16_t)out;  // the next product's 16-bit x
  }
}

// The largest dynamic LDS a group can ask for: SG_MAX_ROWS 64-bit sums.
constexpr size_t SG_LDS_MAX = (size_t)SG_MAX_ROWS * 8;

template <typename Tx, typename Tv, bool GF2 = false>
static hipError_t sg_go(const SgMat& G, const Tx* x, Tv* y, uint32_t alpha, uint32_t beta, uint16_t* y16,
                        hipStream_t st, int64_t ldx = 1, int64_t ldy = 1) {
  const size_t lds = std::max<size_t>((size_t)G.max_rows * 8, SG_LDS_FLOOR);
  auto k = k_sg<Tx, Tv, SG_THREADS, SG_U, GF2>;
  // the kernel's LDS limit is raised once per device to the most any group can need (the
  // attribute is a host call that would otherwise cost a few microseconds per product)
  static std::mutex mu;
  static bool done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
      e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SG_LDS_MAX);
      if (e != hipSuccess) return e;
      done[dev] = true;
    }
  }
  hipLaunchKernelGGL(k, dim3(G.ngroups), dim3(SG_THREADS), lds, st, G, x, y, alpha, beta, y16, ldx, ldy);
  return hipGetLastError();
}

hipError_t launch_sg(const SgMat& G, ffx_dtype dt, const void* x, const uint16_t* x16, void* y, uint32_t alpha,
                     uint32_t beta, hipStream_t st, uint16_t* y16) {
  if (G.ngroups == 0) return hipSuccess;
  if (dt == FFX_I32) {
    if (x16) return sg_go<uint16_t, int32_t>(G, x16, (int32_t*)y, alpha, beta, y16, st);
    return sg_go<int32_t, int32_t>(G, (const int32_t*)x, (int32_t*)y, alpha, beta, y16, st);
  }
  if (x16) return sg_go<uint16_t, int64_t>(G, x16, (int64_t*)y, alpha, beta, y16, st);
  return sg_go<int64_t, int64_t>(G, (const int64_t*)x, (int64_t*)y, alpha, beta, y16, st);
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
// (stage, then three or four chunks per wave). One vector, 1,000,000 power-law
// rows (17.2 M entries): 167 us through binned records.
constexpr uint32_t SGT_XROWS = 44 * 1024;  // staged 16-bit x entries
constexpr uint32_t SGT_ROUND = 32;         // groups staged at a time, at most
constexpr int SGT_U = 2;                   // chunks per wave in flight (four: 77 us against 72 in the kernel)
constexpr size_t SGT_LDS = ((size_t)4 << SGT_SHIFT) + SGT_XROWS * 2;

__global__ __launch_bounds__(SG_THREADS) void k_sg_t(SgMat G, const uint16_t* __restrict__ x16, uint32_t P, uint32_t Q,
                                                     uint32_t slots, uint32_t slot_rows, uint32_t mu32,
                                                     uint32_t* __restrict__ part) {
  extern __shared__ __align__(16) unsigned long long acc[];
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  uint32_t* sums = (uint32_t*)acc;
  uint16_t* xs = (uint16_t*)(sums + (1u << SGT_SHIFT));
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
    // the entry words of the wave's first chunks are requested before x is staged
    uint32_t w[U][4], vo[U], cb[U], xo[U];
    auto load_words = [&](uint32_t j) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t jj = j + u * NW;
        u32x4_t e = (u32x4_t)(PAD_WORD);
        vo[u] = cb[u] = xo[u] = 0;
        if (jj < total) {  // the same in the whole wave
          const int k = __builtin_popcountll(__ballot(lane < ng && pre <= jj)) - 1;
          const uint32_t ch = (uint32_t)__builtin_amdgcn_readlane((int)c0, k) + jj -
                              (uint32_t)__builtin_amdgcn_readlane((int)pre, k);
          e = __builtin_nontemporal_load((const u32x4_t*)(G.ent + (size_t)ch * SG_CHUNK) + lane);
          vo[u] = G.choff[ch];
          cb[u] = G.cbase[ch];
          xo[u] = (uint32_t)__builtin_amdgcn_readlane((int)xoff, k);
        }
        w[u][0] = e.x;
        w[u][1] = e.y;
        w[u][2] = e.z;
        w[u][3] = e.w;
      }
    };
    load_words(wave);
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
      if (j != wave) load_words(j);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        uint32_t idx = vo[u], ngen = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const bool gen = (w[u][k] >> TAG_SHIFT) == TAG_GEN;
          idx += sg_lanes_below(__ballot(gen));
          ngen += gen ? 1u : 0u;
        }
        uint32_t q0 = 0, q1 = 0, q2 = 0;
        if (ngen) {
          typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
          const u32x3_t v = __builtin_nontemporal_load((const u32x3_t*)((const uint32_t*)G.val + (idx >> 1)));
          q0 = v.x;
          q1 = v.y;
          q2 = v.z;
        }
        uint32_t at = idx & 1u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t tag = w[u][k] >> TAG_SHIFT;
          const uint32_t d = at < 2 ? q0 : at < 4 ? q1 : q2;
          const uint32_t v = (d >> ((at & 1u) * 16)) & 0xFFFFu;
          at += tag == TAG_GEN ? 1u : 0u;
          const uint32_t col = cb[u] + (w[u][k] & SG_COL_MASK);
          if (tag == TAG_PAD || (col >> SGT_SHIFT) != p) continue;
          const uint32_t xv = xs[xo[u] + ((w[u][k] >> SG_ROW_SHIFT) & (SG_MAX_ROWS - 1))];
          uint32_t t;
          if (tag == TAG_GEN) {
            t = v * xv;                       // below 2^32
            t -= __umulhi(t, mu32) * G.m;     // the quotient is at most two low: below 3m
          } else {
            t = tag == TAG_PLUS ? xv : G.m - xv;
          }
          atomicAdd(&sums[col & ((1u << SGT_SHIFT) - 1)], t);
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
  if (e == hipSuccess) e = raise_lds_limit((const void*)k_sg_t, (int)SGT_LDS);
  if (e != hipSuccess) return e;
  const uint32_t mu32 = (uint32_t)(((uint64_t)1 << 32) / G.m);
  hipLaunchKernelGGL(k_sg_t, dim3(t.P * t.Q), dim3(SG_THREADS), SGT_LDS, st, G, x16, t.P, t.Q, t.slots, t.slot_rows,
                     mu32, part);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_t_parts(dt, G.m, G.mu, G.ncols, part, t.Q, 1, 1, alpha, beta, y, ldy, st);
}

}  // namespace ffx
