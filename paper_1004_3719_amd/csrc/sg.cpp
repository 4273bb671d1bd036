// Column-sorted row groups (layout in sg.h): the host encoder.
#include <algorithm>
#include <cstring>

#include "host.h"

namespace ffx {

void SgEncoded::release() {
  if (alloc) (void)hipFree(alloc);
  alloc = nullptr;
  dm = SgMat{};
  ngroups = 0;
}

namespace {

struct SgPart {  // one group, encoded from offset 0
  std::vector<uint32_t> ent, cbase;
  std::vector<uint16_t> val;
};

// rows [r0, r1) of A mod m: entries sorted by (column, row), cut into chunks of columns within 65,536 of their base
void encode_group(const RCsr& A, int64_t r0, int64_t r1, uint32_t m, bool values, SgPart& P) {
  const int64_t k0 = A.rp[r0], k1 = A.rp[r1];
  // key: column (bits 30..59) | row in the group (bits 16..29) | value (bits 0..15)
  std::vector<uint64_t> key((size_t)(k1 - k0));
  for (int64_t i = r0; i < r1; ++i)
    for (int64_t k = A.rp[i]; k < A.rp[i + 1]; ++k)
      key[k - k0] = ((uint64_t)A.col[k] << 30) | ((uint64_t)(i - r0) << SG_ROW_SHIFT) | A.val[k];
  std::sort(key.begin(), key.end());
  P.ent.reserve(key.size() + key.size() / 16 + SG_CHUNK);
  if (values) P.val.reserve(P.ent.capacity());
  for (size_t q = 0; q < key.size();) {
    const uint32_t base = (uint32_t)(key[q] >> 30);
    size_t n = 0;  // entries of the chunk
    while (n < SG_CHUNK && q + n < key.size() && (uint32_t)(key[q + n] >> 30) - base <= SG_COL_MASK) ++n;
    const size_t at = P.ent.size();
    P.cbase.push_back(base);
    P.ent.resize(at + SG_CHUNK);
    if (values) P.val.resize(at + SG_CHUNK);
    for (size_t t = 0; t < SG_CHUNK; ++t) {
      const uint64_t kk = key[q + std::min(t, n - 1)];
      const bool pad = t >= n;
      const uint32_t col = (uint32_t)(kk >> 30) - base,
                     row = pad ? (uint32_t)(t % (size_t)(r1 - r0)) & (SG_MAX_ROWS - 1)
                               : (uint32_t)(kk >> SG_ROW_SHIFT) & (SG_MAX_ROWS - 1);
      const size_t w = at + 4 * (t % 64) + t / 64;  // entry 64k + l at place 4l + k
      const uint32_t v = (uint32_t)(kk & 0xFFFFu), tag = pad ? TAG_PAD : v == 1 ? TAG_PLUS : v == m - 1 ? TAG_MINUS : TAG_GEN;
      P.ent[w] = (tag << TAG_SHIFT) | (row << SG_ROW_SHIFT) | col;
      if (values) P.val[w] = pad ? 0 : (uint16_t)v;
    }
    q += n;
  }
}

}  // namespace

void encode_sg(const RCsr& A, const Modulus& md, bool split_pm1, int target_groups, bool transposed, int64_t max_col,
               hipStream_t st, SgEncoded* out) {
  out->release();
  if (!md.small()) fail(FFX_EUNSUPPORTED, "column-sorted groups need m <= 65536");
  const int64_t n = A.nrows, nnz = A.nnz();
  if (n == 0) return;
  // groups of consecutive rows, about nnz / target entries each, at most SG_MAX_ROWS rows
  const int64_t want = std::max<int64_t>({(int64_t)std::max(1, target_groups), (n + SG_MAX_ROWS - 1) / SG_MAX_ROWS});
  std::vector<std::pair<int64_t, int64_t>> ranges;
  for (int64_t r = 0; r < n;) {
    const int64_t left = std::max<int64_t>(1, want - (int64_t)ranges.size());
    const int64_t target = (nnz - A.rp[r] + left - 1) / left;
    const int64_t r0 = r;
    ++r;
    while (r < n && r - r0 < (int64_t)SG_MAX_ROWS && A.rp[r + 1] - A.rp[r0] <= target) ++r;
    ranges.push_back({r0, r});
  }
  const int64_t G = (int64_t)ranges.size();
  const bool values =
      !split_pm1 || !std::all_of(A.val.begin(), A.val.end(), [&](uint32_t v) { return v == 1 || v == md.m - 1; });
  std::vector<SgPart> parts(G);
#pragma omp parallel for schedule(dynamic, 1)
  for (int64_t g = 0; g < G; ++g) encode_group(A, ranges[g].first, ranges[g].second, md.m, values, parts[g]);
  std::vector<SgGroup> groups(G);
  size_t nent = 0, nch = 0;
  uint32_t max_rows = 0;
  for (int64_t g = 0; g < G; ++g) {
    groups[g] = SgGroup{(uint32_t)ranges[g].first, (uint32_t)(ranges[g].second - ranges[g].first), (uint32_t)nch,
                        (uint32_t)parts[g].cbase.size()};
    max_rows = std::max(max_rows, groups[g].nrows);
    nent += parts[g].ent.size();
    nch += parts[g].cbase.size();
  }
  // index of the transposed product: the chunks of each group that hold columns of each panel. Its sums
  // are 32-bit sums of terms below 3m, so the longest column must keep them below 2^32.
  const int64_t P = (A.ncols + ((int64_t)1 << SGT_SHIFT) - 1) >> SGT_SHIFT;
  std::vector<uint2> tindex;
  if (transposed && max_col * 3 * (int64_t)md.m < ((int64_t)1 << 32) && P * G <= SGT_MAX_INDEX) {
    tindex.assign((size_t)P * G, make_uint2(0, 0));
#pragma omp parallel for schedule(dynamic, 1)
    for (int64_t g = 0; g < G; ++g) {
      const SgPart& Q = parts[g];
      for (size_t c = 0; c < Q.cbase.size(); ++c) {
        const uint32_t* w = &Q.ent[c * SG_CHUNK];  // first entry at place 0, last (or padding like it) at the end
        const uint32_t lo = (Q.cbase[c] + (w[0] & SG_COL_MASK)) >> SGT_SHIFT,
                       hi = (Q.cbase[c] + (w[SG_CHUNK - 1] & SG_COL_MASK)) >> SGT_SHIFT;
        for (uint32_t p = lo; p <= hi; ++p) {
          uint2& r = tindex[(size_t)p * G + g];
          if (r.y == 0) r.x = (uint32_t)c;
          r.y = (uint32_t)c + 1;
        }
      }
    }
  }
  if (nent >= UINT32_MAX) fail(FFX_EUNSUPPORTED, "column-sorted encoding exceeds 2^32 words");
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t o_g = 0, o_e = o_g + al(G * sizeof(SgGroup)), o_v = o_e + al(nent * 4),
               o_b = o_v + (values ? al(nent * 2) : 0), o_t = o_b + al(nch * 4),
               total = std::max<size_t>(256, o_t + al(tindex.size() * sizeof(uint2)));
  std::vector<unsigned char> host(total, 0);
  std::memcpy(host.data() + o_g, groups.data(), G * sizeof(SgGroup));
  size_t e = 0, c = 0;
  for (int64_t g = 0; g < G; ++g) {
    const SgPart& P = parts[g];
    std::memcpy(host.data() + o_e + e * 4, P.ent.data(), P.ent.size() * 4);
    if (values) std::memcpy(host.data() + o_v + e * 2, P.val.data(), P.val.size() * 2);
    std::memcpy(host.data() + o_b + c * 4, P.cbase.data(), P.cbase.size() * 4);
    e += P.ent.size();
    c += P.cbase.size();
  }
  if (!tindex.empty()) std::memcpy(host.data() + o_t, tindex.data(), tindex.size() * sizeof(uint2));
  if (hipMalloc(&out->alloc, total) != hipSuccess)
    fail(FFX_ENOMEM, "hipMalloc of %zu bytes for the column-sorted groups failed", total);
  if (hipMemcpyAsync(out->alloc, host.data(), total, hipMemcpyHostToDevice, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    out->release();
    fail(FFX_EDEVICE, "upload of the column-sorted groups failed");
  }
  unsigned char* d = (unsigned char*)out->alloc;
  SgMat& M = out->dm;
  M.groups = (const SgGroup*)(d + o_g);
  M.ent = (const uint32_t*)(d + o_e);
  M.val = values ? (const uint16_t*)(d + o_v) : nullptr;
  M.cbase = (const uint32_t*)(d + o_b);
  M.rowmap = nullptr;
  M.tindex = tindex.empty() ? nullptr : (const uint2*)(d + o_t);
  M.ngroups = (uint32_t)G;
  M.max_rows = max_rows;
  M.nrows = (uint32_t)n;
  M.ncols = (uint32_t)A.ncols;
  M.m = md.m;
  M.mu = md.mu;
  out->ngroups = G;
  out->device_bytes = (int64_t)total;
  out->stream_bytes = (int64_t)(G * sizeof(SgGroup) + nent * (values ? 6 : 4) + nch * 4);
}

}  // namespace ffx
