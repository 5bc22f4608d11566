// libcas host side: argument validation, launch planning, segment-table
// upload, kernel launches, cartridge staging and optional kernel timing.
//
// Validation is pure host code and runs before any HIP call, so every error
// path can be exercised on a machine without a GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/cas.h"
#include "cas_host.h"
#include "cas_internal.h"

using namespace cas;

namespace {

thread_local std::string g_err;
thread_local size_t g_ws_needed = 0;

cas_status_t fail(cas_status_t s, const std::string &msg) {
  g_err = msg;
  return s;
}

std::mutex g_tuning_mu;
cas_tuning_t g_tuning = {0, 0};

cas_tuning_t tuning() {
  std::lock_guard<std::mutex> lk(g_tuning_mu);
  return g_tuning;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

struct Interval {
  uintptr_t lo, hi;   // [lo, hi)
  bool write;
  uintptr_t owner;    // identical writes of one owner may coincide (aliased cartridge)
  const char *what;
};

// Every write interval must be disjoint from every other interval (reads and
// writes) of a different owner.
bool overlap_free(std::vector<Interval> &iv, std::string &msg) {
  std::sort(iv.begin(), iv.end(), [](const Interval &a, const Interval &b) { return a.lo < b.lo; });
  uintptr_t max_hi_any = 0, max_hi_wr = 0;
  int any_idx = -1, wr_idx = -1;
  for (size_t i = 0; i < iv.size(); ++i) {
    const Interval &x = iv[i];
    if (x.hi <= x.lo) continue;
    if (x.write && any_idx >= 0 && max_hi_any > x.lo &&
        !(iv[any_idx].write && iv[any_idx].owner == x.owner && iv[any_idx].lo == x.lo &&
          iv[any_idx].hi == x.hi)) {
      msg = std::string("output ") + x.what + " overlaps " + iv[any_idx].what;
      return false;
    }
    if (!x.write && wr_idx >= 0 && max_hi_wr > x.lo) {
      msg = std::string("input ") + x.what + " overlaps output " + iv[wr_idx].what;
      return false;
    }
    if (x.hi > max_hi_any) {
      max_hi_any = x.hi;
      any_idx = (int)i;
    }
    if (x.write && x.hi > max_hi_wr) {
      max_hi_wr = x.hi;
      wr_idx = (int)i;
    }
  }
  return true;
}

struct Plan {
  DType dt;
  int esize;
  int B, Hkv, g, Hq, D;
  bool packed = false;
  int Sq = 0;              // fixed-length rows: q_len
  int64_t T = 0;           // tokens over all rows
  int Smax = 0;            // longest row
  int nrows_max = 0;       // Smax * g
  int nqb_max = 0;         // 64-row blocks of the longest row
  std::vector<int32_t> tok0, len;
  float scale;
  std::vector<DevSeg> segs;
  std::vector<DevRow> rows;
  std::vector<DevTile> tiles;
  std::vector<DevItem> items;       // bf16 forward (or, backward plan, dQ) workgroups in dispatch order
  std::vector<DevCart> carts;
  std::vector<int32_t> uses;
  std::vector<DevWg> order;       // dK/dV workgroups, longest first
  int64_t dkdv_grid = 0;          // dK/dV workgroups launched
  int dkdv_lists = 1, dkdv_list_len = 0, dkdv_list_head = 0, dkdv_bounded = 0;   // bf16 (see DkdvParams)
  int64_t order_cap = 0;          // 128-key tiles x KV heads, with every self tile
  int64_t order_alloc = 0;        // order entries with every self tile
  int64_t max_prefix = 0;
  int fwd_splits = 1, dq_splits = 1;
  int xcds = 8;                   // XCDs of the device (workgroup order)
  int cus = 256;                  // compute units of the device
  int nqblk = 0;   // row blocks of the longest row (forward and dQ)
  bool want_self_grad = false;
  // workspace layout
  size_t off_segs = 0, off_rows = 0, off_tiles = 0, off_items = 0, off_carts = 0, off_uses = 0, off_order = 0,
         off_claim = 0,
         table_bytes = 0;
  size_t off_part_o = 0, off_part_lse = 0, ws_fwd = 0;
  size_t off_nd = 0, off_lse2 = 0, off_part_dq = 0, off_qT = 0, off_doT = 0, ws_bwd = 0;
};

// Compute units and XCDs of the current device, looked up once per device.
// gfx950 has 32 CUs per XCD (256 and 8 on a whole MI355X; a partition shows
// fewer). Without a device (planning-only use) the whole MI355X is assumed.
struct Topology {
  int cus = 256, xcds = 8;
};
std::mutex g_topo_mu;
std::map<int, Topology> g_topo;
Topology device_topology() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return Topology{};
  }
  std::lock_guard<std::mutex> lk(g_topo_mu);
  auto it = g_topo.find(dev);
  if (it != g_topo.end()) return it->second;
  Topology t;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0) {
    t.cus = cus;
    t.xcds = std::max(1, cus / 32);
  } else {
    (void)hipGetLastError();
  }
  g_topo.emplace(dev, t);
  return t;
}

// Key-axis splits of the forward or dQ pass, for base_wgs workgroups unsplit
// that walk avg_tiles key tiles on average and max_tiles at most, one
// workgroup per compute unit at a time (bf16). Costs are in key tiles (about
// 1.2-1.7 us each): a workgroup costs wg_tiles on top of the tiles it walks
// (dispatch, first loads, pipeline fill and drain, epilogue: 11-13 us), a
// split pass merge_tiles for the merge's launch plus the partials' bytes.
//
// Rounds of workgroups decide. Forward and merge, each timed with its launch:
// 32 workgroups' 139 tiles take 53 us in 8 splits, one round, and 67 us in 16,
// two rounds (what aiming at two workgroups per compute unit chose); 24
// workgroups' 18 tiles 32 us unsplit, 26 us in 4 to 10 splits; 152 workgroups'
// 17 tiles 31 us unsplit, 44 us in 2 splits.
//
// Where one round would leave splits of long_tiles or more, one and two
// rounds measure alike (64 workgroups of 2,056 tiles, forward and dQ: 2,287 us
// in 4 splits, 2,320 us in 8); such calls keep two workgroups per compute
// unit. With more workgroups than compute units, two splits at most are tried
// (the partials' memory grows with the queries).
struct SplitCost {
  double wg_tiles, merge_tiles, bytes_per_tile;
  int64_t long_tiles;
};
constexpr SplitCost kBf16Splits{8.0, 3.0, 5e6, 128};   // (partials written, then read)
// fp32: a tile takes 6-13 us, so the fixed costs weigh less, and a long split
// is not worth a second round: 4 splits of 64 workgroups' 28 tiles take 131 us
// in dQ, 8 take 150 us, unsplit 397 us.
constexpr SplitCost kFp32Splits{1.2, 0.7, 3.5e7, INT64_MAX};
int auto_splits(const SplitCost &c, int64_t base_wgs, int64_t avg_tiles, int64_t max_tiles, int64_t partial_bytes,
                int cus) {
  if (base_wgs < 1) return 1;
  const int64_t one_round = std::max<int64_t>(1, cus / base_wgs);
  const int64_t cap = base_wgs > cus ? 2 : std::min<int64_t>(kMaxSplits, std::max<int64_t>(1, max_tiles));
  auto cost = [&](int64_t s) {
    const double rounds = (double)ceil_div(base_wgs * s, cus) * (c.wg_tiles + (double)ceil_div(avg_tiles, s));
    const double x = std::max(rounds, c.wg_tiles + (double)ceil_div(max_tiles, s));
    return s > 1 ? x + c.merge_tiles + (double)s * (double)partial_bytes / c.bytes_per_tile : x;
  };
  if (base_wgs <= cus && ceil_div(max_tiles, one_round) >= c.long_tiles)
    return (int)std::min<int64_t>(ceil_div(2 * (int64_t)cus, base_wgs), kMaxSplits);
  int64_t best = 1;
  for (int64_t s = 2; s <= cap; ++s)
    if (cost(s) < cost(best)) best = s;
  return (int)best;
}

// Workgroups of the bf16 forward and dQ kernels, in dispatch order, with
// `splits` key-axis splits. Workgroup i is dispatched to XCD i mod X (X = 8 on
// a whole MI355X, each XCD with its own L2), and each XCD hands its next
// workgroup to whichever of its CUs frees first. The items are enumerated
// KV head slowest, then batch row (most key tiles first), split, query block,
// and cut into X contiguous shares, share x for XCD x: the workgroups that
// stream one (row, KV head)'s K/V tiles share an L2 and, when X divides the
// KV heads, every XCD gets whole KV heads (the same work). Within a share the
// items go longest first (key tiles walked; ties keep the enumeration
// order): with one workgroup per CU at a time that is the
// longest-processing-time rule, so the shortest start last and the CUs
// finish together. Only query blocks that hold rows are listed.
void build_items(Plan &pl, int splits) {
  std::vector<int> rows(pl.B);
  for (int b = 0; b < pl.B; ++b) rows[b] = b;
  std::stable_sort(rows.begin(), rows.end(), [&](int a, int c) {
    return pl.rows[a].prefix_tiles + ceil_div(pl.len[a], kKeyTile) >
           pl.rows[c].prefix_tiles + ceil_div(pl.len[c], kKeyTile);
  });
  struct E {
    DevItem it;
    int64_t tiles;
  };
  std::vector<E> v;
  for (int kvh = 0; kvh < pl.Hkv; ++kvh)
    for (int b : rows) {
      const int64_t nrows = (int64_t)pl.len[b] * pl.g;
      const int nq = (int)ceil_div(nrows, kBf16RowsPerWg);
      for (int sp = 0; sp < splits; ++sp)
        for (int qb = nq - 1; qb >= 0; --qb) {
          // The kernels' tile range: the prefix, then the self tiles up to
          // the block's last query position, cut evenly over the splits.
          const int64_t r1 = std::min<int64_t>(nrows, (int64_t)(qb + 1) * kBf16RowsPerWg);
          const int64_t nt = pl.rows[b].prefix_tiles + ((r1 - 1) / pl.g) / kKeyTile + 1;
          v.push_back({{qb, sp, b, kvh}, nt * (sp + 1) / splits - nt * sp / splits});
        }
    }
  const size_t n = v.size(), X = (size_t)std::max(1, pl.xcds), per = n / X;
  auto sort_share = [&](size_t lo, size_t hi) {
    std::stable_sort(v.begin() + lo, v.begin() + hi, [](const E &a, const E &c) { return a.tiles > c.tiles; });
  };
  pl.items.resize(n);
  for (size_t x = 0; x < X; ++x) {
    sort_share(x * per, (x + 1) * per);
    for (size_t k = 0; k < per; ++k) pl.items[k * X + x] = v[x * per + k].it;
  }
  // The remainder (fewer than X) is dispatched last.
  sort_share(X * per, n);
  for (size_t i = X * per; i < n; ++i) pl.items[i] = v[i].it;
}

// Shapes, segment table and planning. `bwd` additionally folds aliases and
// builds the dK/dV work list. A positive `fwd_split_cap` bounds the forward's
// key-axis splits. Pure host code.
cas_status_t build_plan(const cas_problem_t *p, bool bwd, Plan &pl, int fwd_split_cap = 0) {
  if (!p) return fail(CAS_ERR_INVALID_ARGUMENT, "problem is NULL");
  // The caller may pass any integer through the C ABI: read the field's
  // bits as an integer (loading an out-of-range enumerator is undefined).
  int32_t dtype_raw = 0;
  static_assert(sizeof(p->dtype) == sizeof(dtype_raw), "cas_dtype_t is 32-bit");
  std::memcpy(&dtype_raw, &p->dtype, sizeof(dtype_raw));
  if (dtype_raw != CAS_DTYPE_BF16 && dtype_raw != CAS_DTYPE_FP32)
    return fail(CAS_ERR_INVALID_ARGUMENT, "unknown dtype");
  if (p->batch < 1 || p->num_kv_heads < 1 || p->group_size < 1 || p->head_dim < 1)
    return fail(CAS_ERR_INVALID_ARGUMENT, "batch, num_kv_heads, group_size and head_dim must be >= 1");
  if (p->head_dim != 64 && p->head_dim != 128)
    return fail(CAS_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (!std::isfinite(p->softmax_scale) || !(p->softmax_scale > 0.0f))
    return fail(CAS_ERR_INVALID_ARGUMENT, "softmax_scale must be finite and > 0");
  const int64_t Hq = (int64_t)p->num_kv_heads * p->group_size;
  if (Hq > (1 << 16)) return fail(CAS_ERR_UNSUPPORTED, "num_kv_heads*group_size above 2^16");
  if ((int64_t)p->num_kv_heads * p->head_dim > (1 << 22))
    return fail(CAS_ERR_UNSUPPORTED, "num_kv_heads*head_dim above 2^22 (self-token stride)");
  // Query layout: per-row token offsets and lengths.
  pl.packed = p->q_offsets != nullptr;
  pl.tok0.resize(p->batch);
  pl.len.resize(p->batch);
  if (pl.packed) {
    if (p->q_len != 0) return fail(CAS_ERR_INVALID_ARGUMENT, "q_len must be 0 when q_offsets is given");
    if (p->q_offsets[0] != 0) return fail(CAS_ERR_INVALID_ARGUMENT, "q_offsets[0] must be 0");
    for (int b = 0; b < p->batch; ++b) {
      if (p->q_offsets[b + 1] < p->q_offsets[b])
        return fail(CAS_ERR_INVALID_ARGUMENT, "q_offsets must be non-decreasing");
      pl.tok0[b] = p->q_offsets[b];
      pl.len[b] = p->q_offsets[b + 1] - p->q_offsets[b];
    }
    pl.T = p->q_offsets[p->batch];
    if (pl.T < 1) return fail(CAS_ERR_INVALID_ARGUMENT, "packed rows hold no query token");
  } else {
    if (p->q_len < 1) return fail(CAS_ERR_INVALID_ARGUMENT, "q_len must be >= 1");
    if ((int64_t)p->batch * p->q_len > INT32_MAX)
      return fail(CAS_ERR_UNSUPPORTED, "batch*q_len above 2^31");
    for (int b = 0; b < p->batch; ++b) {
      pl.tok0[b] = b * p->q_len;
      pl.len[b] = p->q_len;
    }
    pl.T = (int64_t)p->batch * p->q_len;
    pl.Sq = p->q_len;
  }
  pl.Smax = *std::max_element(pl.len.begin(), pl.len.end());
  if (pl.T * Hq > INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "tokens*num_kv_heads*group_size above 2^31");
  if ((int64_t)p->group_size * pl.Smax > (1 << 28))
    return fail(CAS_ERR_UNSUPPORTED, "group_size*(longest row) above 2^28");
  if (pl.T * Hq * p->head_dim > (int64_t)1 << 40)
    return fail(CAS_ERR_UNSUPPORTED, "query tensor too large");
  if (!p->seg_offsets) return fail(CAS_ERR_INVALID_ARGUMENT, "seg_offsets is NULL");
  if (p->seg_offsets[0] != 0) return fail(CAS_ERR_INVALID_ARGUMENT, "seg_offsets[0] must be 0");
  for (int b = 0; b < p->batch; ++b)
    if (p->seg_offsets[b + 1] < p->seg_offsets[b])
      return fail(CAS_ERR_INVALID_ARGUMENT, "seg_offsets must be non-decreasing");
  const int32_t nent = p->seg_offsets[p->batch];
  if (nent > (1 << 20)) return fail(CAS_ERR_UNSUPPORTED, "more than 2^20 segment entries");
  if (nent > 0 && !p->segments) return fail(CAS_ERR_INVALID_ARGUMENT, "segments is NULL");

  pl.dt = dtype_raw == CAS_DTYPE_BF16 ? kBF16 : kFP32;
  pl.esize = dtype_raw == CAS_DTYPE_BF16 ? 2 : 4;
  pl.B = p->batch;
  pl.Hkv = p->num_kv_heads;
  pl.g = p->group_size;
  pl.Hq = (int)Hq;
  pl.D = p->head_dim;
  pl.nrows_max = pl.Smax * pl.g;
  pl.nqb_max = (int)ceil_div(pl.nrows_max, 64);
  pl.scale = p->softmax_scale;

  const int D = pl.D, es = pl.esize, Hkv = pl.Hkv;
  int64_t tblk = 0;
  pl.rows.resize(pl.B);
  for (int b = 0; b < pl.B; ++b) {
    DevRow r{};
    r.seg_begin = (int32_t)pl.segs.size();
    r.tile_begin = (int32_t)pl.tiles.size();
    r.tok0 = pl.tok0[b];
    r.len = pl.len[b];
    r.lse0 = pl.packed ? pl.tok0[b] : (int32_t)((int64_t)b * Hq * pl.Sq);
    r.tblk0 = (int32_t)tblk;
    tblk += (int64_t)Hkv * ceil_div((int64_t)pl.len[b] * pl.g, 64);
    int64_t tiles = 0, plen = 0;
    for (int i = p->seg_offsets[b]; i < p->seg_offsets[b + 1]; ++i) {
      const cas_segment_t &s = p->segments[i];
      if (s.len < 0) return fail(CAS_ERR_INVALID_ARGUMENT, "segment " + std::to_string(i) + ": negative len");
      if (s.len == 0) continue;
      if (!s.k || !s.v) return fail(CAS_ERR_INVALID_ARGUMENT, "segment " + std::to_string(i) + ": NULL k or v");
      if (s.stride_tok < 1 || s.stride_head < 0 || (Hkv > 1 && s.stride_head < 1))
        return fail(CAS_ERR_INVALID_ARGUMENT, "segment " + std::to_string(i) + ": bad strides");
      if (!aligned16(s.k) || !aligned16(s.v) || !aligned16(s.dk) || !aligned16(s.dv) ||
          (s.stride_tok * es) % 16 != 0 || (s.stride_head * es) % 16 != 0)
        return fail(CAS_ERR_ALIGNMENT, "segment " + std::to_string(i) +
                                           ": pointers and strides must be multiples of 16 bytes");
      if (s.len > (1 << 30)) return fail(CAS_ERR_UNSUPPORTED, "segment longer than 2^30 tokens");
      // Tile copies address up to 128 tokens with 32-bit byte offsets.
      if (s.stride_tok > (1 << 22))
        return fail(CAS_ERR_UNSUPPORTED, "segment " + std::to_string(i) + ": token stride above 2^22 elements");
      DevSeg d{};
      d.k = s.k;
      d.v = s.v;
      d.stride_tok = s.stride_tok;
      d.stride_head = s.stride_head;
      d.len = (int32_t)s.len;
      d.tile_begin = (int32_t)tiles;
      for (int64_t key0 = 0; key0 < s.len; key0 += kKeyTile) {
        DevTile t{};
        t.k = (const char *)s.k + key0 * s.stride_tok * es;
        t.v = (const char *)s.v + key0 * s.stride_tok * es;
        t.stride_head = s.stride_head;
        t.stride_tok = (int32_t)s.stride_tok;
        t.nvalid = (int32_t)std::min<int64_t>(kKeyTile, s.len - key0);
        pl.tiles.push_back(t);
      }
      tiles += ceil_div(s.len, kKeyTile);
      plen += s.len;
      pl.segs.push_back(d);
    }
    if (plen + pl.len[b] > (int64_t)1 << 30)
      return fail(CAS_ERR_UNSUPPORTED, "row " + std::to_string(b) + ": prefix longer than 2^30 tokens");
    r.seg_end = (int32_t)pl.segs.size();
    r.prefix_tiles = (int32_t)tiles;
    // The row's causal self tiles follow its prefix tiles; k/v hold byte
    // offsets from k_self/v_self until bind_self_tiles adds the base.
    for (int64_t s0 = 0; s0 < pl.len[b]; s0 += kKeyTile) {
      DevTile t{};
      const int64_t off = (((int64_t)pl.tok0[b] + s0) * Hkv) * D * es;
      t.k = (const void *)(uintptr_t)off;
      t.v = (const void *)(uintptr_t)off;
      t.stride_head = D;
      t.stride_tok = Hkv * D;
      t.nvalid = (int32_t)std::min<int64_t>(kKeyTile, pl.len[b] - s0);
      pl.tiles.push_back(t);
    }
    pl.rows[b] = r;
    pl.max_prefix = std::max(pl.max_prefix, plen);
  }

  const cas_tuning_t tu = tuning();
  const bool bf16 = pl.dt == kBF16;
  const Topology topo = device_topology();
  pl.xcds = topo.xcds;
  pl.cus = topo.cus;
  // Plans one pass for workgroups of rpw rows. The grids are sized for the
  // longest row; the split costs count the workgroups that have rows, and the
  // key tiles that they walk (prefix, then the self tiles up to the block's
  // last position: half of them on average).
  auto plan_splits = [&](const SplitCost &c, int rpw) {
    int64_t base = 0, sum_tiles = 0, max_tiles = 0;
    for (int b = 0; b < pl.B; ++b) {
      if (pl.len[b] == 0) continue;
      const int64_t blocks = Hkv * ceil_div((int64_t)pl.len[b] * pl.g, rpw), self = ceil_div(pl.len[b], kKeyTile);
      base += blocks;
      sum_tiles += blocks * (pl.rows[b].prefix_tiles + (self + 1) / 2);
      max_tiles = std::max(max_tiles, pl.rows[b].prefix_tiles + self);
    }
    return auto_splits(c, base, ceil_div(sum_tiles, std::max<int64_t>(1, base)), max_tiles, pl.T * pl.Hq * D * 4, topo.cus);
  };
  // Forward and dQ have workgroups of the same rows, and so one plan.
  static_assert(kFwdRowsPerWg == kDqRowsPerWg, "one split plan for both passes");
  const int rpw = bf16 ? kBf16RowsPerWg : kFwdRowsPerWg;
  const int auto_n = plan_splits(bf16 ? kBf16Splits : kFp32Splits, rpw);
  pl.fwd_splits = tu.fwd_splits > 0 ? std::min(tu.fwd_splits, kMaxSplits) : auto_n;
  if (fwd_split_cap > 0) pl.fwd_splits = std::min(pl.fwd_splits, fwd_split_cap);
  pl.dq_splits = tu.dq_splits > 0 ? std::min(tu.dq_splits, kMaxSplits) : auto_n;
  pl.nqblk = (int)ceil_div(pl.nrows_max, rpw);
  if ((int64_t)pl.B * Hkv * pl.nqblk * std::max(pl.fwd_splits, pl.dq_splits) > INT32_MAX)
    return fail(CAS_ERR_UNSUPPORTED, "grid too large");
  if (bf16) build_items(pl, bwd ? pl.dq_splits : pl.fwd_splits);

  if (bwd) {
    // Fold entries that name the same cartridge storage into one cartridge.
    std::map<std::tuple<uintptr_t, uintptr_t, int64_t, int64_t, int64_t>, int> index;
    std::vector<std::vector<int32_t>> users;
    std::vector<const cas_segment_t *> first;
    for (int b = 0; b < pl.B; ++b) {
      for (int i = p->seg_offsets[b]; i < p->seg_offsets[b + 1]; ++i) {
        const cas_segment_t &s = p->segments[i];
        if (s.len == 0) continue;
        auto key = std::make_tuple((uintptr_t)s.k, (uintptr_t)s.v, s.len, s.stride_tok, s.stride_head);
        auto it = index.find(key);
        int u;
        if (it == index.end()) {
          u = (int)first.size();
          index.emplace(key, u);
          first.push_back(&s);
          users.emplace_back();
        } else {
          u = it->second;
          if (first[u]->dk != s.dk || first[u]->dv != s.dv)
            return fail(CAS_ERR_INVALID_ARGUMENT, "segment " + std::to_string(i) +
                                                      ": entries sharing k/v storage must share dk/dv");
        }
        users[u].push_back(b);
      }
    }
    int64_t tiles = 0;
    for (size_t u = 0; u < first.size(); ++u) {
      const cas_segment_t &s = *first[u];
      if (!s.dk && !s.dv) continue;
      DevCart c{};
      c.k = s.k;
      c.v = s.v;
      c.dk = s.dk;
      c.dv = s.dv;
      c.stride_tok = s.stride_tok;
      c.stride_head = s.stride_head;
      c.len = (int32_t)s.len;
      c.use_begin = (int32_t)pl.uses.size();
      // Rows without queries add nothing and are left out.
      int64_t nblk = 0;
      for (int32_t b : users[u]) {
        if (pl.len[b] == 0) continue;
        pl.uses.push_back(b);
        nblk += ceil_div((int64_t)pl.len[b] * pl.g, kDkdvQBlock);
      }
      c.use_end = (int32_t)pl.uses.size();
      if (nblk > INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "too many query blocks per cartridge");
      c.nblk = (int32_t)nblk;
      tiles += ceil_div(s.len, kDkdvKeyTile);
      pl.carts.push_back(c);
      // A gradient buffer must not overlap itself under its strides.
      int64_t s1 = s.stride_tok, n1 = s.len, s2 = s.stride_head, n2 = Hkv;
      if (s1 > s2 || n1 == 1) {
        std::swap(s1, s2);
        std::swap(n1, n2);
      }
      bool ok = true;
      if (n1 > 1 && s1 < D) ok = false;
      if (n2 > 1 && (s2 < D || (n1 > 1 && s2 < s1 * n1))) ok = false;
      if (!ok)
        return fail(CAS_ERR_INVALID_ARGUMENT, "cartridge gradient layout overlaps itself");
    }
    if (tiles > INT32_MAX / 2) return fail(CAS_ERR_UNSUPPORTED, "too many key tiles");
    int64_t self_tiles = 0;
    for (int b = 0; b < pl.B; ++b) self_tiles += ceil_div(pl.len[b], kDkdvKeyTile);
    pl.order_cap = (tiles + self_tiles) * Hkv;
    if (tiles + (int64_t)pl.B * ceil_div(pl.Smax, kDkdvKeyTile) > INT32_MAX / 2 || pl.order_cap > INT32_MAX)
      return fail(CAS_ERR_UNSUPPORTED, "too many key tiles");
    pl.order_alloc = pl.order_cap;
    if (!bf16) {
      pl.order_alloc = 0;
      for (const DevCart &c : pl.carts) pl.order_alloc += ceil_div(c.len, kDkdvKeyTileFp32) * Hkv;
      for (int b = 0; b < pl.B; ++b) pl.order_alloc += ceil_div(pl.len[b], kDkdvKeyTileFp32) * Hkv;
      if (pl.order_alloc > INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "too many key tiles");
    }
  }

  // Workspace layout.
  size_t off = 0;
  pl.off_segs = off;
  off = align_up(off + pl.segs.size() * sizeof(DevSeg), 256);
  pl.off_rows = off;
  off = align_up(off + pl.rows.size() * sizeof(DevRow), 256);
  pl.off_tiles = off;
  off = align_up(off + pl.tiles.size() * sizeof(DevTile), 256);
  pl.off_items = off;
  off = align_up(off + pl.items.size() * sizeof(DevItem), 256);
  if (bwd) {
    pl.off_carts = off;
    off = align_up(off + pl.carts.size() * sizeof(DevCart), 256);
    pl.off_uses = off;
    off = align_up(off + pl.uses.size() * sizeof(int32_t), 256);
    pl.off_order = off;
    off = align_up(off + (size_t)pl.order_alloc * sizeof(DevWg), 256);
    pl.off_claim = off;   // claim counters: zero in every table upload
    off = align_up(off + (size_t)pl.xcds * sizeof(int32_t), 256);
  }
  pl.table_bytes = off;
  const size_t plane = (size_t)pl.T * pl.Hq;   // packed rows of all batch rows and KV heads
  if (!bwd) {
    if (pl.fwd_splits > 1) {
      pl.off_part_o = off;
      off = align_up(off + (size_t)pl.fwd_splits * plane * D * 4, 256);
      pl.off_part_lse = off;
      off = align_up(off + (size_t)pl.fwd_splits * plane * (bf16 ? 4 : 8), 256);
    }
    pl.ws_fwd = off;
  } else {
    pl.off_nd = off;
    off = align_up(off + plane * 4, 256);
    pl.off_lse2 = off;
    off = align_up(off + plane * 4, 256);
    if (pl.dt == kBF16) {
      // Transposed Q and dO of every 64-row block (dK/dV operands).
      const size_t tbytes = (size_t)tblk * 64 * D * 2;
      pl.off_qT = off;
      off = align_up(off + tbytes, 256);
      pl.off_doT = off;
      off = align_up(off + tbytes, 256);
    }
    if (pl.dq_splits > 1) {
      pl.off_part_dq = off;
      off = align_up(off + (size_t)pl.dq_splits * plane * D * 4, 256);
    }
    pl.ws_bwd = off;
  }
  return CAS_OK;
}

// dK/dV workgroup list: every cartridge tile (and, with self gradients, every
// self tile of every row) at every KV head, sorted by the number of 64-row
// query blocks the workgroup walks, most first; ties go by KV head, then by
// the tile's position within its cartridge (or the row's self keys), then
// tile order. Longest-first dispatch keeps the long workgroups off the tail;
// the position tie-break lets the workgroups that run side by side on an XCD
// come from all the cartridges (and so rows) of their KV head, instead of
// all walking one row's query blocks.
void build_dkdv_order(Plan &pl, bool with_self) {
  struct E {
    int64_t nblk;
    int32_t owner, pos, kvh;   // pos: tile within its cartridge or the row's self keys
    int32_t cost() const { return (int32_t)std::min<int64_t>(nblk, 1 << 20) + kDkdvFixedCost; }
    DevWg wg() const { return {owner, pos, kvh, cost()}; }
  };
  std::vector<E> v;
  const int key_tile = pl.dt == kBF16 ? kDkdvKeyTile : kDkdvKeyTileFp32;
  v.reserve((size_t)pl.order_alloc);
  for (size_t i = 0; i < pl.carts.size(); ++i) {
    const DevCart &c = pl.carts[i];
    const int n = (int)ceil_div(c.len, key_tile);
    for (int kvh = 0; kvh < pl.Hkv; ++kvh)
      for (int t = 0; t < n; ++t) v.push_back({c.nblk, (int32_t)i, t, kvh});
  }
  if (with_self) {
    for (int b = 0; b < pl.B; ++b) {
      const int64_t nqb = ceil_div((int64_t)pl.len[b] * pl.g, kDkdvQBlock);
      const int n = (int)ceil_div(pl.len[b], key_tile);
      for (int kvh = 0; kvh < pl.Hkv; ++kvh)
        for (int j = 0; j < n; ++j)
          v.push_back({nqb - ((int64_t)j * key_tile * pl.g) / kDkdvQBlock, -1 - b, j, kvh});
    }
  }
  std::stable_sort(v.begin(), v.end(), [](const E &a, const E &b) {
    if (a.nblk != b.nblk) return a.nblk > b.nblk;
    if (a.kvh != b.kvh) return a.kvh < b.kvh;
    return a.pos < b.pos;   // (then cartridges, then rows, in order: the sort is stable)
  });
  pl.order.resize(v.size());
  pl.dkdv_grid = (int64_t)v.size();
  const int X = pl.xcds;
  if (v.empty()) return;
  if (pl.dt != kBF16) {
    // fp32: workgroup i takes entry i. XCD-affine (as below) where the KV
    // heads divide evenly.
    const bool affine = X > 1 && pl.Hkv % X == 0;
    std::vector<std::vector<E>> q(affine ? X : 1);
    for (const E &e : v) q[affine ? e.kvh % X : 0].push_back(e);
    std::vector<size_t> next(q.size(), 0);
    for (size_t i = 0; i < v.size(); ++i) {
      const E &e = q[i % q.size()][next[i % q.size()]++];
      pl.order[i] = e.wg();
    }
    return;
  }
  // bf16: the workgroups, one per compute unit at a time, work through lists of
  // entries, longest first. XCD-affine where the KV heads divide evenly:
  // workgroup i runs on XCD i % X (round-robin dispatch) and starts on list
  // i % X, the entries of KV heads h with h % X == i % X, so the query blocks
  // of one (row, KV head) are streamed by one XCD's L2. Every KV head has the
  // same tiles, so the lists are equally long. Otherwise one list for all.
  // A workgroup claims its next entry when it has finished one, from its own
  // list and then from those with work left: XCDs run at different speeds
  // (up to 4 % apart on one chip), so a fixed share per XCD ends with the
  // slowest, and a new workgroup per entry leaves its compute unit idle for
  // 3-6 us between two of them. After kDkdvStay it ends all the same: with its
  // registers and LDS hardly another kernel fits beside it, so the compute unit
  // is free for other streams' work only between two workgroups.
  const int L = X > 1 && pl.Hkv % X == 0 ? X : 1;
  std::vector<std::vector<E>> q(L);
  for (const E &e : v) q[e.kvh % L].push_back(e);
  const int64_t cnt = (int64_t)q[0].size();
  const int64_t wgs = std::min<int64_t>(cnt, std::max(1, pl.cus / L));   // workgroups of one list
  pl.dkdv_lists = L;
  pl.dkdv_list_len = (int)cnt;
  size_t at = 0;
  for (const std::vector<E> &l : q)
    for (const E &e : l) pl.order[at++] = e.wg();
  // As many workgroups as stays that the list's costs fill, taken in order, and
  // at least one round. The last round stays until nothing is left, which takes
  // every entry whatever the stays came to, and needs no workgroup to find out
  // that there is none. Entries that fill a stay by themselves need no draw
  // where they come first; the shortest two rounds, or an eighth of the list,
  // are drawn all the same.
  int64_t full = 0, stays = 0, cost = 0;
  for (const E &e : q[0]) {
    if (e.cost() >= kDkdvStay) ++full;
    cost += e.cost();
    if (cost >= kDkdvStay) {
      ++stays;
      cost = 0;
    }
  }
  const int64_t n = std::max(wgs, stays);
  pl.dkdv_list_head = (int)std::max(wgs, std::min(full, cnt - std::max(2 * wgs, cnt / 8)));
  pl.dkdv_bounded = (int)(n - wgs);
  pl.dkdv_grid = L * n;
}

// Turns the self-tile offsets of the tile table into pointers.
void bind_self_tiles(Plan &pl, const void *k_self, const void *v_self) {
  for (int b = 0; b < pl.B; ++b) {
    const DevRow &r = pl.rows[b];
    const int n = (int)ceil_div(pl.len[b], kKeyTile);
    for (int i = 0; i < n; ++i) {
      DevTile &t = pl.tiles[r.tile_begin + r.prefix_tiles + i];
      t.k = (const char *)k_self + (uintptr_t)t.k;
      t.v = (const char *)v_self + (uintptr_t)t.v;
    }
  }
}

void add_segment_intervals(const Plan &pl, const cas_problem_t *p, bool with_grads,
                           std::vector<Interval> &iv) {
  const int es = pl.esize;
  for (int i = 0; i < p->seg_offsets[p->batch]; ++i) {
    const cas_segment_t &s = p->segments[i];
    if (s.len == 0) continue;
    const uintptr_t span = (uintptr_t)(((s.len - 1) * s.stride_tok + (pl.Hkv - 1) * s.stride_head + pl.D) * es);
    iv.push_back({(uintptr_t)s.k, (uintptr_t)s.k + span, false, 0, "segment k"});
    iv.push_back({(uintptr_t)s.v, (uintptr_t)s.v + span, false, 0, "segment v"});
    if (with_grads) {
      // Entries of one aliased cartridge carry identical (dk, dv) intervals.
      if (s.dk) iv.push_back({(uintptr_t)s.dk, (uintptr_t)s.dk + span, true, (uintptr_t)s.dk, "segment dk"});
      if (s.dv) iv.push_back({(uintptr_t)s.dv, (uintptr_t)s.dv + span, true, (uintptr_t)s.dv, "segment dv"});
    }
  }
}

// ---------------------------------------------------------------------------
// Pinned staging ring for launch tables (host -> workspace, copied by a
// small kernel on the launch stream).
// ---------------------------------------------------------------------------
constexpr size_t kMinSlotBytes = 1 << 20;
constexpr int kSlots = 8;

struct Ring {
  char *host = nullptr;
  size_t slot_bytes = 0;
  hipEvent_t ev[kSlots] = {};
  bool used[kSlots] = {};
  int next = 0;
};

std::mutex g_ring_mu;
std::map<int, Ring> g_rings;

// Copies `bytes` of launch tables, written by fill() into a pinned slot,
// to the workspace on the stream.
template <typename Fill>
cas_status_t ring_upload(size_t bytes, void *ws, hipStream_t stream, Fill &&fill) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  std::lock_guard<std::mutex> lk(g_ring_mu);
  Ring &r = g_rings[dev];
  if (!r.ev[0]) {
    for (int i = 0; i < kSlots; ++i) {
      e = hipEventCreateWithFlags(&r.ev[i], hipEventDisableTiming);
      if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipEventCreate: ") + hipGetErrorString(e));
    }
  }
  if (!r.host || bytes > r.slot_bytes) {
    // (Re)allocate the pinned ring once every earlier upload from it is done.
    for (int i = 0; i < kSlots; ++i) {
      if (!r.used[i]) continue;
      e = hipEventSynchronize(r.ev[i]);
      if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipEventSynchronize: ") + hipGetErrorString(e));
      r.used[i] = false;
    }
    if (r.host) {
      e = hipHostFree(r.host);
      r.host = nullptr;
      r.slot_bytes = 0;
      if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipHostFree: ") + hipGetErrorString(e));
    }
    size_t sb = kMinSlotBytes;
    while (sb < bytes) sb *= 2;
    // Coherent: the upload kernel reads the slots the host has just
    // rewritten, so no GPU cache may keep an earlier upload's lines.
    e = hipHostMalloc((void **)&r.host, sb * kSlots, hipHostMallocCoherent);
    if (e != hipSuccess) {
      r.host = nullptr;
      r.slot_bytes = 0;
      return fail(CAS_ERR_HIP, std::string("hipHostMalloc: ") + hipGetErrorString(e));
    }
    r.slot_bytes = sb;
  }
  const int slot = r.next;
  r.next = (r.next + 1) % kSlots;
  if (r.used[slot]) {
    e = hipEventSynchronize(r.ev[slot]);
    if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipEventSynchronize: ") + hipGetErrorString(e));
  }
  char *h = r.host + (size_t)slot * r.slot_bytes;
  std::memset(h, 0, bytes);
  fill(h);
  e = launch_table_upload(ws, h, bytes, stream);
  if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("table upload launch: ") + hipGetErrorString(e));
  e = hipEventRecord(r.ev[slot], stream);
  if (e != hipSuccess) return fail(CAS_ERR_HIP, std::string("hipEventRecord: ") + hipGetErrorString(e));
  r.used[slot] = true;
  return CAS_OK;
}

// Writes the launch tables, laid out as in the workspace, to host memory h
// (table_bytes, zeroed by the caller).
void fill_tables(const Plan &pl, bool bwd, char *h) {
  if (!pl.segs.empty()) std::memcpy(h + pl.off_segs, pl.segs.data(), pl.segs.size() * sizeof(DevSeg));
  std::memcpy(h + pl.off_rows, pl.rows.data(), pl.rows.size() * sizeof(DevRow));
  if (!pl.tiles.empty()) std::memcpy(h + pl.off_tiles, pl.tiles.data(), pl.tiles.size() * sizeof(DevTile));
  if (!pl.items.empty()) std::memcpy(h + pl.off_items, pl.items.data(), pl.items.size() * sizeof(DevItem));
  if (bwd) {
    if (!pl.carts.empty()) std::memcpy(h + pl.off_carts, pl.carts.data(), pl.carts.size() * sizeof(DevCart));
    if (!pl.uses.empty()) std::memcpy(h + pl.off_uses, pl.uses.data(), pl.uses.size() * sizeof(int32_t));
    if (!pl.order.empty()) std::memcpy(h + pl.off_order, pl.order.data(), pl.order.size() * sizeof(DevWg));
  }
}

cas_status_t upload_tables(const Plan &pl, bool bwd, void *ws, hipStream_t stream) {
  return ring_upload(pl.table_bytes, ws, stream, [&](char *h) { fill_tables(pl, bwd, h); });
}

// ---------------------------------------------------------------------------
// Cartridge Adam step: validation and launch tables.
// ---------------------------------------------------------------------------
struct AdamPlan {
  std::vector<DevAdamT> tensors;
  std::vector<DevAdamChunk> chunks;
  size_t off_chunks = 0, bytes = 0;
};

float lr_scale(int32_t step, int32_t warmup, int32_t buckets) {
  if (buckets < 1 || step < 0) return NAN;
  if (warmup <= 0 || step >= warmup) return 1.0f;
  // ceil(buckets * step / warmup), at least the first level
  const int64_t lvl = std::max<int64_t>(1, ((int64_t)buckets * step + warmup - 1) / warmup);
  return (float)std::min<int64_t>(lvl, buckets) / (float)buckets;
}

cas_status_t build_adam(const cas_adam_cartridge_t *carts, int32_t n, int32_t Hkv, int32_t D,
                        const cas_adam_config_t *cfg, AdamPlan &ap) {
  if (n < 0) return fail(CAS_ERR_INVALID_ARGUMENT, "n must be >= 0");
  if (n > 0 && !carts) return fail(CAS_ERR_INVALID_ARGUMENT, "carts is NULL");
  if (Hkv < 1) return fail(CAS_ERR_INVALID_ARGUMENT, "num_kv_heads must be >= 1");
  if (D != 64 && D != 128) return fail(CAS_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (cfg) {
    if (!std::isfinite(cfg->lr) || cfg->lr < 0.0f) return fail(CAS_ERR_INVALID_ARGUMENT, "lr must be finite and >= 0");
    if (!(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f) || !(cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f))
      return fail(CAS_ERR_INVALID_ARGUMENT, "beta1 and beta2 must lie in [0, 1)");
    if (!std::isfinite(cfg->eps) || !(cfg->eps > 0.0f)) return fail(CAS_ERR_INVALID_ARGUMENT, "eps must be finite and > 0");
    if (cfg->warmup_buckets < 1 || cfg->warmup_steps < 0)
      return fail(CAS_ERR_INVALID_ARGUMENT, "warmup_buckets must be >= 1 and warmup_steps >= 0");
  }
  std::vector<Interval> iv;
  for (int i = 0; i < n; ++i) {
    const cas_adam_cartridge_t &c = carts[i];
    const std::string who = "cartridge " + std::to_string(i);
    if (c.len < 0 || c.step < 0 || c.frozen_tokens < 0)
      return fail(CAS_ERR_INVALID_ARGUMENT, who + ": len, step and frozen_tokens must be >= 0");
    if (c.len > (1 << 30)) return fail(CAS_ERR_UNSUPPORTED, who + ": longer than 2^30 tokens");
    if (c.len <= c.frozen_tokens) continue;   // nothing to update
    const void *ptrs[8] = {c.k, c.v, c.dk, c.dv, c.m1_k, c.m2_k, c.m1_v, c.m2_v};
    for (const void *q : ptrs)
      if (!q) return fail(CAS_ERR_INVALID_ARGUMENT, who + ": NULL tensor");
    for (const void *q : ptrs)
      if (!aligned16(q)) return fail(CAS_ERR_ALIGNMENT, who + ": tensors must be 16-byte aligned");
    if (c.stride_tok < 1 || c.stride_head < 0 || (Hkv > 1 && c.stride_head < 1))
      return fail(CAS_ERR_INVALID_ARGUMENT, who + ": bad strides");
    if (c.stride_tok % 8 != 0 || c.stride_head % 8 != 0)
      return fail(CAS_ERR_ALIGNMENT, who + ": strides must be multiples of 8 elements");
    int64_t s1 = c.stride_tok, n1 = c.len, s2 = c.stride_head, n2 = Hkv;
    if (s1 > s2 || n1 == 1) {
      std::swap(s1, s2);
      std::swap(n1, n2);
    }
    if ((n1 > 1 && s1 < D) || (n2 > 1 && (s2 < D || (n1 > 1 && s2 < s1 * n1))))
      return fail(CAS_ERR_INVALID_ARGUMENT, who + ": parameter layout overlaps itself");
    const uintptr_t span = (uintptr_t)(((c.len - 1) * c.stride_tok + (int64_t)(Hkv - 1) * c.stride_head + D) * 2);
    const uintptr_t mom = (uintptr_t)c.len * Hkv * D * 4;
    // Every written tensor is its own owner: no two may overlap, even at equal addresses.
    const uintptr_t own = (uintptr_t)i * 8 + 1;
    iv.push_back({(uintptr_t)c.k, (uintptr_t)c.k + span, true, own, "k"});
    iv.push_back({(uintptr_t)c.v, (uintptr_t)c.v + span, true, own + 1, "v"});
    iv.push_back({(uintptr_t)c.dk, (uintptr_t)c.dk + span, false, 0, "dk"});
    iv.push_back({(uintptr_t)c.dv, (uintptr_t)c.dv + span, false, 0, "dv"});
    int j = 2;
    for (float *m : {c.m1_k, c.m2_k, c.m1_v, c.m2_v})
      iv.push_back({(uintptr_t)m, (uintptr_t)m + mom, true, own + j++, "moment"});
  }
  std::string msg;
  if (!overlap_free(iv, msg)) return fail(CAS_ERR_INVALID_ARGUMENT, msg);
  for (int i = 0; i < n; ++i) {
    const cas_adam_cartridge_t &c = carts[i];
    if (c.len <= c.frozen_tokens) continue;
    const double t = (double)c.step + 1.0;
    for (int which = 0; which < 2; ++which) {
      DevAdamT d{};
      d.x = (__bf16 *)(which ? c.v : c.k);
      d.g = (const __bf16 *)(which ? c.dv : c.dk);
      d.m1 = which ? c.m1_v : c.m1_k;
      d.m2 = which ? c.m2_v : c.m2_k;
      d.stride_tok = c.stride_tok;
      d.stride_head = c.stride_head;
      d.len = (int32_t)c.len;
      d.frozen = c.frozen_tokens;
      if (cfg) {
        d.lr = cfg->lr * lr_scale(c.step, cfg->warmup_steps, cfg->warmup_buckets);
        d.bc1 = (float)(1.0 - std::pow((double)cfg->beta1, t));
        d.bc2 = (float)(1.0 - std::pow((double)cfg->beta2, t));
      }
      const int32_t ti = (int32_t)ap.tensors.size();
      ap.tensors.push_back(d);
      for (int64_t tok = c.frozen_tokens; tok < c.len; tok += kAdamChunk) ap.chunks.push_back({ti, (int32_t)tok});
    }
    if (ap.chunks.size() > (size_t)INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "too many chunks");
  }
  ap.off_chunks = align_up(ap.tensors.size() * sizeof(DevAdamT), 256);
  ap.bytes = align_up(ap.off_chunks + ap.chunks.size() * sizeof(DevAdamChunk), 256);
  return CAS_OK;
}

// ---------------------------------------------------------------------------
// Optional per-kernel timing.
// ---------------------------------------------------------------------------
struct TimedLaunch {
  const char *name;
  hipEvent_t a, b;
};

std::mutex g_time_mu;
bool g_timing = false;
std::vector<TimedLaunch> g_pending;
std::vector<hipEvent_t> g_event_pool;
std::map<std::string, std::pair<int, double>> g_totals;

hipEvent_t pooled_event() {
  if (!g_event_pool.empty()) {
    hipEvent_t e = g_event_pool.back();
    g_event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

template <typename F>
hipError_t timed(const char *name, hipStream_t s, F &&launch) {
  bool on;
  {
    std::lock_guard<std::mutex> lk(g_time_mu);
    on = g_timing;
  }
  if (!on) return launch();
  hipEvent_t a, b;
  {
    std::lock_guard<std::mutex> lk(g_time_mu);
    a = pooled_event();
    b = pooled_event();
  }
  if (!a || !b) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(a, s);
  if (e != hipSuccess) return e;
  e = launch();
  if (e != hipSuccess) return e;
  e = hipEventRecord(b, s);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_time_mu);
  g_pending.push_back({name, a, b});
  return hipSuccess;
}

cas_status_t hip_fail(const char *what, hipError_t e) {
  return fail(CAS_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

cas_status_t check_workspace(void *ws, size_t have, size_t need) {
  if (have < need || (need > 0 && !ws)) g_ws_needed = need;
  if (need > 0 && !ws) return fail(CAS_ERR_WORKSPACE, "workspace is NULL");
  if (have < need)
    return fail(CAS_ERR_WORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes, have " +
                                       std::to_string(have));
  if (!aligned16(ws)) return fail(CAS_ERR_ALIGNMENT, "workspace must be 16-byte aligned");
  return CAS_OK;
}

// ---------------------------------------------------------------------------
// Paged decode: validation, key-axis split planning and launch tables.
// ---------------------------------------------------------------------------
constexpr int kMaxDecParts = 64;   // partials of one request

struct DecodePlan {
  int Tq = 0, Hq = 0;
  std::vector<DevDecodeRow> rows;
  std::vector<DevDecodeWork> work;
  std::vector<int32_t> tok_parts;
  int max_parts = 1;
  int shared = 0;   // page runs streamed for several requests
  // 16-row blocks of one workgroup: 2 when a request has more than 16 packed
  // rows, or when that shares enough page runs between more requests, so that
  // those rows take one pass over the keys.
  int row_blocks = 1;
  size_t off_work = 0, off_pages = 0, off_tokparts = 0, off_plse = 0, off_po = 0, bytes = 0;
  size_t alone_bytes = 0;   // of the plan that shares nothing, which the page ids do not change

  // Places nrows rows, nwork workgroups and `parts` partials of every row in the workspace.
  void lay_out(const cas_decode_problem_t *p, int64_t nrows, int64_t nwork, int parts) {
    size_t off = align_up((size_t)nrows * sizeof(DevDecodeRow), 256);
    off_work = off;
    off = align_up(off + (size_t)nwork * sizeof(DevDecodeWork), 256);
    off_pages = off;
    off = align_up(off + (size_t)p->page_offsets[p->batch] * sizeof(int32_t), 256);
    off_tokparts = off;
    off = align_up(off + (size_t)Tq * sizeof(int32_t), 256);
    off_plse = off_po = 0;
    if (parts > 1) {
      const size_t plane = (size_t)Tq * Hq;
      off_plse = off;
      off = align_up(off + (size_t)parts * plane * 4, 256);
      off_po = off;
      off = align_up(off + (size_t)parts * plane * p->head_dim * 4, 256);
    }
    bytes = off;
  }
};

// Consecutive page ids [id0, id1) from index `at` of request b's page list, and
// the shared runs [run0, run1) that it holds, whole and in order.
struct Stretch {
  uint32_t id0, id1;
  int32_t b, at;
  int32_t run0, run1;
};

// A run of page ids that several requests read: npages from id0, first found at
// page_ids[page0]. Its readers are users[user0 .. user0 + nusers).
struct SharedRun {
  uint32_t id0;
  int32_t npages, page0;
  int32_t user0, nusers;
  int64_t saved[2];   // tiles of one KV head saved in blocks of 16 and of 32 rows
};

// Whether ids[0 .. n) are consecutive.
inline bool consecutive(const int32_t *ids, int32_t n) {
  uint32_t off = 0;
  for (int32_t k = 0; k < n; ++k) off |= (uint32_t)ids[k] ^ ((uint32_t)ids[0] + (uint32_t)k);
  return off == 0;
}

// The stretches of at least min_pages pages among the first safe_pages of every
// request's list, in order. One of that length holds one of every min_pages
// indices, so scattered pages cost a look at every min_pages-th of them.
std::vector<Stretch> stretches(const cas_decode_problem_t *p, const std::vector<int32_t> &safe_pages, int min_pages) {
  std::vector<Stretch> st;
  for (int b = 0; b < p->batch; ++b) {
    const int32_t *ids = p->page_ids + p->page_offsets[b];
    const int32_t n = safe_pages[b];
    for (int32_t from = 0, j = min_pages - 1; j < n; j = from + min_pages - 1) {
      int32_t i = j, e = j + 1;
      if (consecutive(ids + from, min_pages)) i = from;
      while (i > from && ids[i] - ids[i - 1] == 1) --i;
      if (e < n && ids[e] - ids[e - 1] == 1)
        while (e + 16 <= n && consecutive(ids + e - 1, 17)) e += 16;
      while (e < n && ids[e] - ids[e - 1] == 1) ++e;
      if (e - i >= min_pages) st.push_back({(uint32_t)ids[i], (uint32_t)ids[i] + (uint32_t)(e - i), b, i, 0, 0});
      from = e;
    }
  }
  return st;
}

// Sorts by the upper 32 bits: short lists by comparison, longer ones by 11 bits
// at a time (2,560 ends 10 us, by comparison 110 us).
void sort_by_id(std::vector<uint64_t> &v) {
  if (v.size() < 96) {
    std::sort(v.begin(), v.end());
    return;
  }
  uint64_t most = 0;
  for (uint64_t x : v) most |= x;
  std::vector<uint64_t> w(v.size());
  for (int sh = 32; sh < 64 && most >> sh; sh += 11) {
    uint32_t at[2048] = {};
    for (uint64_t x : v) ++at[x >> sh & 2047];
    uint32_t sum = 0;
    for (uint32_t &a : at) {
      const uint32_t n = a;
      a = sum;
      sum += n;
    }
    for (uint64_t x : v) w[at[x >> sh & 2047]++] = x;
    v.swap(w);
  }
}

// Runs of at least min_pages that are read at least twice, by id. The ends of
// all stretches cut the id axis into intervals, each read whole by the same
// stretches. Requests usually read whole cartridges, so equal stretches are
// counted together and only the distinct ones' ends are sorted. On one host
// core a plan of 64 requests over 4 of 256 cartridges (16,640 pages, 65 runs)
// takes 33 us, 11 of them to find and value the runs, over 60 of 80 cartridges
// (61,760 pages, 80 runs) 170 us; with as many private or scattered pages 15
// and 12 us.
std::vector<SharedRun> shared_runs(std::vector<Stretch> &st, int min_pages) {
  std::vector<SharedRun> runs;
  if (st.size() < 2) return runs;
  struct Distinct {
    uint32_t id0, id1;
    int32_t readers, run0, run1;
  };
  size_t cap = 4;
  while (cap < 2 * st.size()) cap *= 2;
  std::vector<int32_t> slot(cap, -1), which(st.size());
  std::vector<Distinct> ds;
  ds.reserve(st.size());
  for (size_t i = 0; i < st.size(); ++i) {
    const Stretch &x = st[i];
    size_t h = (size_t)((x.id0 * 0x9e3779b97f4a7c15ull + x.id1 * 0xc2b2ae3d27d4eb4full) >> 32);
    for (;; ++h) {
      int32_t &k = slot[h & (cap - 1)];
      if (k < 0) {
        k = (int32_t)ds.size();
        ds.push_back({x.id0, x.id1, 0, 0, 0});
      }
      if (ds[k].id0 != x.id0 || ds[k].id1 != x.id1) continue;
      ++ds[k].readers;
      which[i] = k;
      break;
    }
  }
  // The ends in order of id, each with its place in ds.
  std::vector<uint64_t> ends(2 * ds.size());
  for (size_t k = 0; k < ds.size(); ++k) {
    ends[2 * k] = (uint64_t)ds[k].id0 << 32 | 2 * k;
    ends[2 * k + 1] = (uint64_t)ds[k].id1 << 32 | (2 * k + 1);
  }
  sort_by_id(ends);
  // Readers of the interval from one id to the next, summed from the
  // differences; run0 and run1 of an end: the runs that lie before it.
  int32_t readers = 0;
  for (size_t k = 0; k < ends.size();) {
    const uint32_t id = (uint32_t)(ends[k] >> 32);
    for (; k < ends.size() && (uint32_t)(ends[k] >> 32) == id; ++k) {
      Distinct &d = ds[(uint32_t)ends[k] / 2];
      const bool last = ends[k] & 1;
      (last ? d.run1 : d.run0) = (int32_t)runs.size();
      readers += last ? -d.readers : d.readers;
    }
    if (readers < 2 || k == ends.size()) continue;
    const uint32_t n = (uint32_t)(ends[k] >> 32) - id;
    if (n >= (uint32_t)min_pages) runs.push_back({id, (int32_t)n, -1, 0, 0, {0, 0}});
  }
  if (runs.empty()) return runs;
  for (size_t i = 0; i < st.size(); ++i) {
    st[i].run0 = ds[which[i]].run0;
    st[i].run1 = ds[which[i]].run1;
  }
  return runs;
}

// `share` false: every request streams its keys by itself.
cas_status_t build_decode(const cas_decode_problem_t *p, DecodePlan &dp, bool share = true) {
  if (!p) return fail(CAS_ERR_INVALID_ARGUMENT, "problem is NULL");
  if (p->batch < 1 || p->num_kv_heads < 1 || p->group_size < 1)
    return fail(CAS_ERR_INVALID_ARGUMENT, "batch, num_kv_heads and group_size must be >= 1");
  if (p->head_dim != 64 && p->head_dim != 128) return fail(CAS_ERR_UNSUPPORTED, "head_dim must be 64 or 128");
  if (!std::isfinite(p->softmax_scale) || !(p->softmax_scale > 0.0f))
    return fail(CAS_ERR_INVALID_ARGUMENT, "softmax_scale must be finite and > 0");
  const int P = p->page_size;
  if (P != 16 && P != 32 && P != 64 && P != 128) return fail(CAS_ERR_UNSUPPORTED, "page_size must be 16, 32, 64 or 128");
  const int64_t Hq = (int64_t)p->num_kv_heads * p->group_size;
  if (Hq > (1 << 16)) return fail(CAS_ERR_UNSUPPORTED, "num_kv_heads*group_size above 2^16");
  if ((int64_t)P * p->num_kv_heads * p->head_dim * 2 >= ((int64_t)1 << 31))
    return fail(CAS_ERR_UNSUPPORTED, "page larger than 2 GiB");
  if (p->num_pages < 1) return fail(CAS_ERR_INVALID_ARGUMENT, "num_pages must be >= 1");
  if (!p->q_offsets || !p->kv_lens || !p->page_offsets || !p->page_ids)
    return fail(CAS_ERR_INVALID_ARGUMENT, "q_offsets, kv_lens, page_offsets and page_ids must be non-NULL");
  if (p->q_offsets[0] != 0 || p->page_offsets[0] != 0)
    return fail(CAS_ERR_INVALID_ARGUMENT, "q_offsets[0] and page_offsets[0] must be 0");
  const int B = p->batch;
  for (int b = 0; b < B; ++b) {
    const int64_t n = (int64_t)p->q_offsets[b + 1] - p->q_offsets[b];
    const int64_t L = p->kv_lens[b];
    if (n < 1) return fail(CAS_ERR_INVALID_ARGUMENT, "request " + std::to_string(b) + ": no query token");
    if (L < n) return fail(CAS_ERR_INVALID_ARGUMENT, "request " + std::to_string(b) + ": kv_len below its query count");
    if (L > (1 << 30)) return fail(CAS_ERR_UNSUPPORTED, "request " + std::to_string(b) + ": more than 2^30 keys");
    if ((int64_t)p->page_offsets[b + 1] - p->page_offsets[b] != ceil_div(L, P))
      return fail(CAS_ERR_INVALID_ARGUMENT, "request " + std::to_string(b) + ": page count must be ceil(kv_len / page_size)");
  }
  const int64_t Tq = p->q_offsets[B];
  if (Tq * Hq > INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "query tokens * heads above 2^31");
  const uint32_t last_page = (uint32_t)(std::min<int64_t>(p->num_pages, (int64_t)1 << 31) - 1);
  uint32_t most_id = 0;   // (a negative id counts as one above every valid one)
  for (int32_t i = 0; i < p->page_offsets[B]; ++i) most_id = std::max(most_id, (uint32_t)p->page_ids[i]);
  for (int32_t i = 0; most_id > last_page; ++i)
    if ((uint32_t)p->page_ids[i] > last_page)
      return fail(CAS_ERR_INVALID_ARGUMENT, "page id " + std::to_string(i) + " out of range");
  dp.Tq = (int)Tq;
  dp.Hq = (int)Hq;
  const int g = p->group_size, Hkv = p->num_kv_heads;
  // Packed rows and row blocks (of 16 and of 32) of every request.
  std::vector<int32_t> rows_of(B), blocks_of[2];
  int32_t rows_max = 0;
  for (int nb = 1; nb <= 2; ++nb) blocks_of[nb - 1].resize(B);
  for (int b = 0; b < B; ++b) {
    rows_of[b] = (p->q_offsets[b + 1] - p->q_offsets[b]) * g;
    blocks_of[0][b] = (int32_t)(((int64_t)rows_of[b] + kDecRows - 1) / kDecRows);
    blocks_of[1][b] = (blocks_of[0][b] + 1) / 2;
    rows_max = std::max(rows_max, rows_of[b]);
  }
  dp.row_blocks = rows_max > kDecRows ? 2 : 1;
  // Page runs shared between requests (typically whole cartridges) are streamed
  // once per 16 or 32 rows of all their readers instead of once per reader. A
  // run is worth it from kMinSharedTiles tiles (a workgroup with a partial of
  // its own costs about three tiles), the call when it streams at most 0.85 of
  // the tiles; two row blocks instead of one have to save another tenth.
  constexpr int kMinSharedTiles = 8;
  std::vector<Stretch> st;
  std::vector<SharedRun> runs;
  if (share && B > 1 && Tq * g <= (1 << 14)) {   // (longer query blocks would only grow the table of rows)
    std::vector<int32_t> safe(B);
    for (int b = 0; b < B; ++b) {
      // The first query of a request sees keys 0 .. kv_len - n.
      const int32_t n = p->q_offsets[b + 1] - p->q_offsets[b];
      safe[b] = (p->kv_lens[b] - n + 1) / P;
    }
    const int min_pages = std::max<int>(1, kMinSharedTiles * kDecTile / P);
    st = stretches(p, safe, min_pages);
    runs = shared_runs(st, min_pages);
  }
  // Streamed key tiles of one KV head, every request on its own and with what
  // the shared runs save, in blocks of 16 and of 32 rows.
  int64_t t_alone[2] = {0, 0};
  for (int b = 0; b < B; ++b) {
    const int64_t nt = ceil_div(p->kv_lens[b], kDecTile);
    for (int k = 0; k < 2; ++k) t_alone[k] += nt * blocks_of[k][b];
  }
  const int nb_alone = dp.row_blocks;
  int nb_shared = nb_alone;
  // Whether sharing pays, with the requests that read alone left out, and the
  // runs' readers and savings. Only runs that save anything are shared.
  std::vector<uint8_t> alone(B, 0);
  struct Sum {
    int64_t rows, blocks[2];
  };
  std::vector<Sum> sums;
  auto value_runs = [&]() {
    if (runs.empty()) return false;
    sums.assign(runs.size(), Sum{0, {0, 0}});
    for (SharedRun &r : runs) r.nusers = 0;
    for (const Stretch &x : st) {
      if (alone[x.b]) continue;
      for (int32_t k = x.run0; k < x.run1; ++k) {
        SharedRun &r = runs[k];
        ++r.nusers;
        if (r.page0 < 0) r.page0 = p->page_offsets[x.b] + x.at + (int32_t)(r.id0 - x.id0);
        sums[k].rows += rows_of[x.b];
        for (int i = 0; i < 2; ++i) sums[k].blocks[i] += blocks_of[i][x.b];
      }
    }
    int64_t t[2] = {t_alone[0], t_alone[1]};
    for (size_t k = 0; k < runs.size(); ++k) {
      const int64_t nt = ceil_div((int64_t)runs[k].npages * P, kDecTile);
      for (int i = 0; i < 2; ++i) {
        runs[k].saved[i] = std::max<int64_t>(0, sums[k].blocks[i] - ceil_div(sums[k].rows, kDecRows * (i + 1))) * nt;
        t[i] -= runs[k].saved[i];
      }
    }
    nb_shared = nb_alone;
    if (nb_shared == 1 && t[1] * 10 <= t[0] * 9) nb_shared = 2;
    return t[nb_shared - 1] * 100 <= t_alone[nb_alone - 1] * 85;
  };
  auto is_shared = [&](int32_t k) { return runs[k].saved[nb_shared - 1] > 0; };
  // f(request, run or -1, first page, one past the last) for the pieces of the
  // requests' page lists, in order: shared runs and what lies between them.
  bool sharing = false;
  auto pieces = [&](auto &&f) {
    size_t i = 0;
    for (int b = 0; b < B; ++b) {
      const int32_t np = p->page_offsets[b + 1] - p->page_offsets[b];
      int32_t at = 0;
      if (sharing)
        for (; i < st.size() && st[i].b == b; ++i) {
          if (alone[b]) continue;
          for (int32_t k = st[i].run0; k < st[i].run1; ++k) {
            if (!is_shared(k)) continue;
            const int32_t first = st[i].at + (int32_t)(runs[k].id0 - st[i].id0);
            if (first > at) f(b, -1, at, first);
            at = first + runs[k].npages;
            f(b, k, first, at);
          }
        }
      if (np > at) f(b, -1, at, np);
    }
  };
  std::vector<int32_t> parts(B, 0);   // partials of every request
  if (!runs.empty()) {
    // Requests over more runs than they may have partials read their keys by
    // themselves; so do those whose runs and stretches between them are more.
    // (The others' runs become fewer by that, never more.)
    for (const Stretch &x : st) parts[x.b] = (int32_t)std::min<int64_t>(kMaxDecParts + 1, (int64_t)parts[x.b] + (x.run1 - x.run0));
    for (int b = 0; b < B; ++b) alone[b] = parts[b] > kMaxDecParts;
    sharing = value_runs();
    if (sharing) {
      std::fill(parts.begin(), parts.end(), 0);
      bool more = false;
      pieces([&](int32_t b, int32_t, int32_t, int32_t) { ++parts[b]; });
      for (int b = 0; b < B; ++b)
        if (parts[b] > kMaxDecParts) more = alone[b] = 1;
      if (more) sharing = value_runs();
    }
  }

  // Segments: the shared runs, then what is left of each request's pages.
  struct Seg {
    int32_t page0, nkeys, full, tiles;
    int32_t user0, nusers;   // readers: users[user0 ..]
    int32_t rows;            // of all its readers
    bool own_end;            // holds the end of its reader's keys
    int32_t pieces;
  };
  std::vector<Seg> segs;
  std::vector<int32_t> users;
  if (sharing) {
    int32_t n = 0;
    for (size_t k = 0; k < runs.size(); ++k) {
      SharedRun &r = runs[k];
      if (!is_shared((int32_t)k)) continue;
      const int32_t nkeys = r.npages * P;
      r.user0 = n;
      n += r.nusers;
      segs.push_back({r.page0, nkeys, nkeys - 1, (nkeys + kDecTile - 1) / kDecTile, r.user0, r.nusers, (int32_t)sums[k].rows, false, 0});
    }
    users.resize(n);
  }
  dp.shared = (int)segs.size();
  pieces([&](int32_t b, int32_t run, int32_t first, int32_t to) {
    if (run >= 0) {
      users[runs[run].user0++] = b;
      return;
    }
    const int32_t np = p->page_offsets[b + 1] - p->page_offsets[b], n = p->q_offsets[b + 1] - p->q_offsets[b];
    const bool end = to == np;
    const int32_t nkeys = (end ? p->kv_lens[b] : to * P) - first * P;
    segs.push_back({p->page_offsets[b] + first, nkeys, end ? nkeys - n : nkeys - 1, (nkeys + kDecTile - 1) / kDecTile,
                    (int32_t)users.size(), 1, rows_of[b], end, 0});
    users.push_back(b);
  });
  // Partials in pieces of at most per_wg tiles: the largest count of a request.
  auto count_parts = [&](int64_t per_wg) {
    std::fill(parts.begin(), parts.end(), 0);
    int32_t most = 0;
    for (const Seg &s : segs) {
      const int32_t n = (int32_t)ceil_div(s.tiles, per_wg);
      for (int32_t u = s.user0; u < s.user0 + s.nusers; ++u) most = std::max(most, parts[users[u]] += n);
    }
    return most;
  };
  // Workgroups of that cut, which the segments then have (kMaxDecParts pieces each at most).
  auto set_pieces = [&](int64_t per_wg) {
    int64_t wgs = 0;
    for (Seg &s : segs) {
      s.pieces = (int32_t)std::min<int64_t>(kMaxDecParts, ceil_div(s.tiles, per_wg));
      wgs += s.pieces * ceil_div(s.rows, kDecRows * dp.row_blocks) * Hkv;
    }
    return wgs;
  };
  // Split planning. Without sharing: workgroups of at least 8 tiles (two per
  // wave), about as many as the compute units hold at once (two each), so the
  // whole step runs in one round of workgroups when the requests allow it.
  // With sharing there are many segments of a cartridge's length, whose
  // workgroups need no further cutting while they fill the compute units:
  // pieces of at most 32 tiles, 64 requests over 4 of 256 cartridges of 32 tiles
  // 136 us (143 us with one of at most 85), 50 over 3 of 16 27 us (31 us in
  // pieces of 8). Fewer workgroups than compute units: shorter pieces, as far
  // as 8 tiles and a request's partials allow; longer runs than its partials
  // hold in pieces of 32: longer pieces.
  const int64_t cus = device_topology().cus;
  const int64_t per_wg_alone = std::max<int64_t>(8, ceil_div(t_alone[nb_alone - 1] * Hkv, 2 * cus));
  dp.row_blocks = sharing ? nb_shared : nb_alone;
  int64_t wgs = 0;
  if (!sharing) {
    wgs = set_pieces(per_wg_alone);
  } else {
    // What the same requests need when they share nothing.
    int64_t alone_wgs = 0, most = 1;
    for (int b = 0; b < B; ++b) {
      const int64_t n = std::min<int64_t>(kMaxDecParts, ceil_div(ceil_div(p->kv_lens[b], kDecTile), per_wg_alone));
      alone_wgs += n * blocks_of[nb_alone - 1][b] * Hkv;
      most = std::max(most, n);
    }
    dp.lay_out(p, Tq * g, alone_wgs, (int)most);
    dp.alone_bytes = dp.bytes;
    int64_t least = 8;   // the shortest pieces that a request's partials allow
    if (count_parts(least) > kMaxDecParts) {
      int64_t most = least;
      for (const Seg &s : segs) most = std::max<int64_t>(most, s.tiles);
      while (least + 1 < most) {   // (pieces of `least` are too many, of `most` are not)
        const int64_t mid = (least + most) / 2;
        (count_parts(mid) > kMaxDecParts ? least : most) = mid;
      }
      least = most;
    }
    for (int64_t per_wg = std::max<int64_t>(32, least); (wgs = set_pieces(per_wg)) < cus && per_wg > least;)
      per_wg = std::max(least, per_wg / 2);
  }
  std::fill(parts.begin(), parts.end(), 0);
  int64_t nrows = 0;
  for (const Seg &s : segs) {
    nrows += s.rows;
    for (int32_t u = s.user0; u < s.user0 + s.nusers; ++u) parts[users[u]] += s.pieces;
  }
  if (wgs > INT32_MAX || nrows > INT32_MAX) return fail(CAS_ERR_UNSUPPORTED, "too many workgroups");
  dp.tok_parts.resize(Tq);
  for (int b = 0; b < B; ++b) {
    dp.max_parts = std::max(dp.max_parts, parts[b]);
    for (int32_t t = p->q_offsets[b]; t < p->q_offsets[b + 1]; ++t) dp.tok_parts[t] = parts[b];
  }
  // Rows and workgroups. The workgroups go longest range first, ties in the
  // order of segment, KV head, row block, piece: the first walk counts the
  // lengths (a segment's pieces have two at most), the second puts each
  // workgroup in its place.
  const int rows_per_wg = kDecRows * dp.row_blocks;
  std::vector<int32_t> next_part(B, 0);
  std::map<int32_t, int64_t, std::greater<int32_t>> at;   // length -> workgroups, then the next one's place
  dp.rows.resize((size_t)nrows);
  DevDecodeRow *row = dp.rows.data();
  for (const Seg &s : segs) {
    for (int32_t u = s.user0; u < s.user0 + s.nusers; ++u) {
      const int32_t b = users[u], q0 = p->q_offsets[b], n = p->q_offsets[b + 1] - q0;
      const int32_t part = parts[b] > 1 ? next_part[b] : -1;
      for (int32_t i = 0; i < n; ++i)
        for (int32_t h = 0; h < g; ++h) *row++ = {(q0 + i) * (int32_t)Hq + h, s.own_end ? s.full + i : s.nkeys - 1, part};
      next_part[b] += s.pieces;
    }
    const int64_t wgs_of_piece = ceil_div(s.rows, rows_per_wg) * Hkv;
    const int32_t longer = s.tiles % s.pieces;
    at[s.tiles / s.pieces] += (s.pieces - longer) * wgs_of_piece;
    if (longer) at[s.tiles / s.pieces + 1] += longer * wgs_of_piece;
  }
  int64_t place = 0;
  for (auto &x : at) {
    const int64_t n = x.second;
    x.second = place;
    place += n;
  }
  dp.work.resize((size_t)wgs);
  struct Piece {
    int32_t t0, t1;
    int64_t *place;
  };
  std::vector<Piece> cut;
  int32_t row0 = 0;
  for (const Seg &s : segs) {
    const int32_t len = s.tiles / s.pieces;
    int64_t *const places[2] = {&at[len], s.tiles % s.pieces ? &at[len + 1] : nullptr};
    cut.resize(s.pieces);
    for (int32_t i = 0, t0 = 0; i < s.pieces; ++i) {
      const int32_t t1 = (int32_t)((int64_t)s.tiles * (i + 1) / s.pieces);
      cut[i] = {t0, t1, places[t1 - t0 - len]};
      t0 = t1;
    }
    for (int kvh = 0; kvh < Hkv; ++kvh)
      for (int32_t r = 0; r < s.rows; r += rows_per_wg)
        for (int32_t i = 0; i < s.pieces; ++i)
          dp.work[(*cut[i].place)++] = {s.page0, s.nkeys, s.full, kvh, cut[i].t0, cut[i].t1, row0 + r,
                                        std::min(rows_per_wg, s.rows - r), i};
    row0 += s.rows;
  }
  dp.lay_out(p, nrows, wgs, dp.max_parts);
  if (!sharing) dp.alone_bytes = dp.bytes;
  return CAS_OK;
}

}  // namespace

namespace cas {

cas_status_t set_error(cas_status_t s, const std::string &msg) { return fail(s, msg); }

cas_status_t set_hip_error(const char *what, hipError_t e) { return hip_fail(what, e); }

hipError_t enqueue_copies(const HostCopy *c, int n, hipMemcpyKind kind, hipStream_t s) {
  const char *run_src = nullptr;
  char *run_dst = nullptr;
  size_t run_bytes = 0;
  auto flush = [&]() -> hipError_t {
    hipError_t e = hipSuccess;
    if (run_bytes) e = hipMemcpyAsync(run_dst, run_src, run_bytes, kind, s);
    run_bytes = 0;
    return e;
  };
  for (int i = 0; i < n; ++i) {
    if (c[i].bytes == 0) continue;
    const char *src = (const char *)c[i].src;
    char *dst = (char *)c[i].dst;
    if (run_bytes && src == run_src + run_bytes && dst == run_dst + run_bytes) {
      run_bytes += c[i].bytes;
      continue;
    }
    hipError_t e = flush();
    if (e != hipSuccess) return e;
    run_src = src;
    run_dst = dst;
    run_bytes = c[i].bytes;
  }
  return flush();
}

cas_status_t prefix_attn_fwd_run(const cas_problem_t *p, const void *q, const void *k_self,
                                 const void *v_self, void *o, float *lse, void *workspace,
                                 size_t ws_bytes, hipStream_t stream, ScratchAddressFn scratch) {
  Plan pl;
  cas_status_t s = build_plan(p, false, pl);
  if (s != CAS_OK) return s;
  if (scratch) {
    // The workspace is the fixed scratch: fewer key-axis splits (smaller
    // partials) until it fits. Only the rounding order of the merge changes.
    while (pl.ws_fwd > ws_bytes && pl.fwd_splits > 1) {
      // Bytes per split (partials) from this plan; the rebuilt
      // plan is checked again since each region is rounded up to 256 bytes.
      const size_t per_split = (pl.ws_fwd - pl.table_bytes) / (size_t)pl.fwd_splits;
      const size_t room = ws_bytes > pl.table_bytes ? ws_bytes - pl.table_bytes : 0;
      size_t cap = per_split ? room / per_split : 1;
      cap = std::max<size_t>(1, std::min<size_t>(cap, (size_t)pl.fwd_splits - 1));
      pl = Plan{};
      s = build_plan(p, false, pl, (int)cap);
      if (s != CAS_OK) return s;
    }
    if (pl.ws_fwd > ws_bytes)
      return fail(CAS_ERR_UNSUPPORTED, "launch tables need " + std::to_string(pl.ws_fwd) +
                                           " bytes, above the " + std::to_string(ws_bytes) +
                                           "-byte scratch of the no-allocation forward");
  }
  if (!q || !k_self || !v_self || !o) return fail(CAS_ERR_INVALID_ARGUMENT, "q, k_self, v_self and o must be non-NULL");
  if (!aligned16(q) || !aligned16(k_self) || !aligned16(v_self) || !aligned16(o) || ((uintptr_t)lse & 3u))
    return fail(CAS_ERR_ALIGNMENT, "tensors must be 16-byte aligned (lse 4-byte)");
  const uintptr_t qbytes = (uintptr_t)pl.T * pl.Hq * pl.D * pl.esize;
  const uintptr_t kvbytes = (uintptr_t)pl.T * pl.Hkv * pl.D * pl.esize;
  std::vector<Interval> iv;
  iv.push_back({(uintptr_t)q, (uintptr_t)q + qbytes, false, 0, "q"});
  iv.push_back({(uintptr_t)k_self, (uintptr_t)k_self + kvbytes, false, 0, "k_self"});
  iv.push_back({(uintptr_t)v_self, (uintptr_t)v_self + kvbytes, false, 0, "v_self"});
  iv.push_back({(uintptr_t)o, (uintptr_t)o + qbytes, true, (uintptr_t)o, "o"});
  if (lse) iv.push_back({(uintptr_t)lse, (uintptr_t)lse + (uintptr_t)pl.T * pl.Hq * 4, true, (uintptr_t)lse, "lse"});
  add_segment_intervals(pl, p, false, iv);
  std::string msg;
  if (!overlap_free(iv, msg)) return fail(CAS_ERR_INVALID_ARGUMENT, msg);
  if (scratch) {
    // Everything is validated: only now touch the device.
    hipError_t e = scratch(&workspace);
    if (e != hipSuccess) return hip_fail("hipGetSymbolAddress (no-allocation scratch)", e);
  } else {
    s = check_workspace(workspace, ws_bytes, pl.ws_fwd);
    if (s != CAS_OK) return s;
  }

  bind_self_tiles(pl, k_self, v_self);
  if (scratch) {
    // No pinned staging ring: the tables travel as kernel arguments.
    std::vector<char> h(pl.table_bytes, 0);
    fill_tables(pl, false, h.data());
    hipError_t e = launch_table_args_upload(h.data(), pl.table_bytes, workspace, stream);
    if (e != hipSuccess) return hip_fail("table upload launch", e);
  } else {
    s = upload_tables(pl, false, workspace, stream);
    if (s != CAS_OK) return s;
  }
  // Kernel timing records pooled events, which the no-allocation path must
  // not create: it launches directly.
  auto launch = [&](const char *name, auto &&f) -> hipError_t {
    return scratch ? f() : timed(name, stream, f);
  };
  char *ws = (char *)workspace;
  FwdParams fp{};
  fp.q = q;
  fp.k_self = k_self;
  fp.v_self = v_self;
  fp.o = o;
  fp.lse = lse;
  fp.part_o = pl.fwd_splits > 1 ? (float *)(ws + pl.off_part_o) : nullptr;
  fp.part_lse = pl.fwd_splits > 1 ? (float *)(ws + pl.off_part_lse) : nullptr;
  fp.segs = (const DevSeg *)(ws + pl.off_segs);
  fp.rows = (const DevRow *)(ws + pl.off_rows);
  fp.tiles = (const DevTile *)(ws + pl.off_tiles);
  fp.items = (const DevItem *)(ws + pl.off_items);
  fp.plane = pl.T * pl.Hq;
  fp.B = pl.B;
  fp.Smax = pl.Smax;
  fp.Hkv = pl.Hkv;
  fp.g = pl.g;
  fp.nrows_max = pl.nrows_max;
  fp.nqblk = pl.nqblk;
  fp.splits = pl.fwd_splits;
  fp.lse_hs = pl.packed ? (int32_t)pl.T : pl.Sq;
  fp.n_items = (int32_t)pl.items.size();
  fp.scale_log2 = pl.scale * 1.4426950408889634f;
  hipError_t e = launch("fwd", [&] { return launch_fwd(fp, pl.dt, pl.D, stream); });
  if (e != hipSuccess) return hip_fail("fwd launch", e);
  if (pl.fwd_splits > 1) {
    MergeParams mp{};
    mp.part_o = fp.part_o;
    mp.part_lse = fp.part_lse;
    mp.o = o;
    mp.lse = lse;
    mp.rows = fp.rows;
    mp.plane = fp.plane;
    mp.B = pl.B;
    mp.Hkv = pl.Hkv;
    mp.g = pl.g;
    mp.nrows_max = pl.nrows_max;
    mp.splits = pl.fwd_splits;
    mp.lse_hs = fp.lse_hs;
    e = launch("fwd_merge", [&] { return launch_fwd_merge(mp, pl.dt, pl.D, stream); });
    if (e != hipSuccess) return hip_fail("fwd_merge launch", e);
  }
  return CAS_OK;
}

}  // namespace cas

extern "C" {

int32_t cas_abi_version(void) { return CAS_ABI_VERSION; }

const char *cas_status_string(cas_status_t s) {
  switch (s) {
    case CAS_OK: return "CAS_OK";
    case CAS_ERR_INVALID_ARGUMENT: return "CAS_ERR_INVALID_ARGUMENT";
    case CAS_ERR_UNSUPPORTED: return "CAS_ERR_UNSUPPORTED";
    case CAS_ERR_ALIGNMENT: return "CAS_ERR_ALIGNMENT";
    case CAS_ERR_NOT_PINNED: return "CAS_ERR_NOT_PINNED";
    case CAS_ERR_WORKSPACE: return "CAS_ERR_WORKSPACE";
    case CAS_ERR_HIP: return "CAS_ERR_HIP";
    case CAS_ERR_IO: return "CAS_ERR_IO";
  }
  return "CAS_ERR_UNKNOWN";
}

const char *cas_last_error_message(void) { return g_err.c_str(); }

size_t cas_last_workspace_needed(void) { return g_ws_needed; }

float cas_adam_lr_scale(int32_t step, int32_t warmup_steps, int32_t warmup_buckets) {
  return lr_scale(step, warmup_steps, warmup_buckets);
}

cas_status_t cas_paged_decode_workspace_size(const cas_decode_problem_t *p, size_t *bytes) {
  if (!bytes) return fail(CAS_ERR_INVALID_ARGUMENT, "bytes is NULL");
  DecodePlan dp;
  cas_status_t s = build_decode(p, dp);
  if (s != CAS_OK) return s;
  *bytes = std::max(dp.bytes, dp.alone_bytes);
  return CAS_OK;
}

cas_status_t cas_paged_decode_plan_info(const cas_decode_problem_t *p, cas_decode_plan_info_t *info, int32_t *rows,
                                        int32_t *work) {
  if (!info) return fail(CAS_ERR_INVALID_ARGUMENT, "info is NULL");
  DecodePlan dp;
  cas_status_t s = build_decode(p, dp);
  if (s != CAS_OK) return s;
  *info = cas_decode_plan_info_t{};
  for (const DevDecodeWork &w : dp.work) info->key_tiles += w.tile1 - w.tile0;
  info->workgroups = (int32_t)dp.work.size();
  info->num_rows = (int32_t)dp.rows.size();
  info->row_blocks = dp.row_blocks;
  info->max_partials = dp.max_parts;
  info->shared_runs = dp.shared;
  info->ws_bytes = dp.bytes;
  static_assert(sizeof(DevDecodeRow) == 12 && sizeof(DevDecodeWork) == 36, "tables of 32-bit values");
  if (rows) std::memcpy(rows, dp.rows.data(), dp.rows.size() * sizeof(DevDecodeRow));
  if (work) std::memcpy(work, dp.work.data(), dp.work.size() * sizeof(DevDecodeWork));
  return CAS_OK;
}

static cas_status_t run_decode(const cas_decode_problem_t *p, const DecodePlan &plan, const void *q, const void *k_pages,
                               const void *v_pages, void *o, float *lse, void *workspace, size_t ws_bytes,
                               void *hip_stream) {
  if (!q || !k_pages || !v_pages || !o) return fail(CAS_ERR_INVALID_ARGUMENT, "q, k_pages, v_pages and o must be non-NULL");
  if (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(o) || ((uintptr_t)lse & 3u))
    return fail(CAS_ERR_ALIGNMENT, "tensors must be 16-byte aligned (lse 4-byte)");
  const uintptr_t qbytes = (uintptr_t)plan.Tq * plan.Hq * p->head_dim * 2;
  const uintptr_t pool = (uintptr_t)p->num_pages * p->page_size * p->num_kv_heads * p->head_dim * 2;
  std::vector<Interval> iv;
  iv.push_back({(uintptr_t)q, (uintptr_t)q + qbytes, false, 0, "q"});
  iv.push_back({(uintptr_t)k_pages, (uintptr_t)k_pages + pool, false, 0, "k_pages"});
  iv.push_back({(uintptr_t)v_pages, (uintptr_t)v_pages + pool, false, 0, "v_pages"});
  iv.push_back({(uintptr_t)o, (uintptr_t)o + qbytes, true, 1, "o"});
  if (lse) iv.push_back({(uintptr_t)lse, (uintptr_t)lse + (uintptr_t)plan.Tq * plan.Hq * 4, true, 2, "lse"});
  std::string msg;
  if (!overlap_free(iv, msg)) return fail(CAS_ERR_INVALID_ARGUMENT, msg);
  // A workspace for the same lengths that share nothing: neither do these.
  DecodePlan unshared;
  const bool room = ws_bytes >= plan.bytes || ws_bytes < plan.alone_bytes || !workspace;
  cas_status_t s = room ? CAS_OK : build_decode(p, unshared, false);
  if (s != CAS_OK) return s;
  const DecodePlan &dp = room ? plan : unshared;
  s = check_workspace(workspace, ws_bytes, ws_bytes < dp.bytes ? std::max(dp.bytes, dp.alone_bytes) : dp.bytes);
  if (s != CAS_OK) return s;
  hipStream_t stream = (hipStream_t)hip_stream;
  char *ws = (char *)workspace;
  const int npage_ids = p->page_offsets[p->batch];
  s = ring_upload(dp.off_plse ? dp.off_plse : dp.bytes, workspace, stream, [&](char *h) {
    std::memcpy(h, dp.rows.data(), dp.rows.size() * sizeof(DevDecodeRow));
    std::memcpy(h + dp.off_work, dp.work.data(), dp.work.size() * sizeof(DevDecodeWork));
    if (npage_ids) std::memcpy(h + dp.off_pages, p->page_ids, (size_t)npage_ids * sizeof(int32_t));
    std::memcpy(h + dp.off_tokparts, dp.tok_parts.data(), dp.tok_parts.size() * sizeof(int32_t));
  });
  if (s != CAS_OK) return s;
  DecodeParams kp{};
  kp.q = q;
  kp.k_pages = k_pages;
  kp.v_pages = v_pages;
  kp.o = o;
  kp.lse = lse;
  kp.rows = (const DevDecodeRow *)ws;
  kp.work = (const DevDecodeWork *)(ws + dp.off_work);
  kp.page_ids = (const int32_t *)(ws + dp.off_pages);
  kp.tok_parts = (const int32_t *)(ws + dp.off_tokparts);
  kp.part_lse = dp.max_parts > 1 ? (float *)(ws + dp.off_plse) : nullptr;
  kp.part_o = dp.max_parts > 1 ? (float *)(ws + dp.off_po) : nullptr;
  kp.plane = (int64_t)dp.Tq * dp.Hq;
  kp.Hkv = p->num_kv_heads;
  kp.g = p->group_size;
  kp.page_size = p->page_size;
  kp.Tq = dp.Tq;
  kp.scale_log2 = p->softmax_scale * 1.4426950408889634f;
  hipError_t e = timed("decode", stream, [&] { return launch_decode_bf16(kp, p->head_dim, (int)dp.work.size(), dp.row_blocks, stream); });
  if (e != hipSuccess) return hip_fail("decode launch", e);
  if (dp.max_parts > 1) {
    e = timed("decode_merge", stream, [&] { return launch_decode_merge_bf16(kp, p->head_dim, dp.max_parts, stream); });
    if (e != hipSuccess) return hip_fail("decode_merge launch", e);
  }
  return CAS_OK;
}

cas_status_t cas_paged_decode_fwd(const cas_decode_problem_t *p, const void *q, const void *k_pages,
                                  const void *v_pages, void *o, float *lse, void *workspace,
                                  size_t ws_bytes, void *hip_stream) {
  DecodePlan dp;
  cas_status_t s = build_decode(p, dp);
  if (s != CAS_OK) return s;
  return run_decode(p, dp, q, k_pages, v_pages, o, lse, workspace, ws_bytes, hip_stream);
}

struct cas_decode_plan {
  cas_decode_problem_t p;         // its tables are the copies below
  std::vector<int32_t> tables;    // q_offsets, kv_lens, page_offsets, page_ids as they were validated
  DecodePlan dp;
};

cas_status_t cas_paged_decode_plan_create(const cas_decode_problem_t *p, cas_decode_plan_t **plan, size_t *ws_bytes) {
  if (!plan || !ws_bytes) return fail(CAS_ERR_INVALID_ARGUMENT, "plan or ws_bytes is NULL");
  *plan = nullptr;
  auto pl = std::make_unique<cas_decode_plan>();
  cas_status_t s = build_decode(p, pl->dp);
  if (s != CAS_OK) return s;
  const size_t B = (size_t)p->batch, ids = (size_t)p->page_offsets[B];
  pl->tables.reserve(3 * B + 2 + ids);
  auto copy = [&](const int32_t *src, size_t n) {
    const int32_t *at = pl->tables.data() + pl->tables.size();
    pl->tables.insert(pl->tables.end(), src, src + n);
    return at;
  };
  pl->p = *p;
  pl->p.q_offsets = copy(p->q_offsets, B + 1);
  pl->p.kv_lens = copy(p->kv_lens, B);
  pl->p.page_offsets = copy(p->page_offsets, B + 1);
  pl->p.page_ids = copy(p->page_ids, ids);
  *ws_bytes = std::max(pl->dp.bytes, pl->dp.alone_bytes);
  *plan = pl.release();
  return CAS_OK;
}

cas_status_t cas_paged_decode_run(const cas_decode_plan_t *plan, const void *q, const void *k_pages,
                                  const void *v_pages, void *o, float *lse, void *workspace,
                                  size_t ws_bytes, void *hip_stream) {
  if (!plan) return fail(CAS_ERR_INVALID_ARGUMENT, "plan is NULL");
  return run_decode(&plan->p, plan->dp, q, k_pages, v_pages, o, lse, workspace, ws_bytes, hip_stream);
}

int32_t cas_paged_decode_plan_matches(const cas_decode_plan_t *plan, const cas_decode_problem_t *p) {
  if (!plan || !p || !p->q_offsets || !p->kv_lens || !p->page_offsets || !p->page_ids) return 0;
  const cas_decode_problem_t &o = plan->p;
  if (p->batch != o.batch || p->num_kv_heads != o.num_kv_heads || p->group_size != o.group_size || p->head_dim != o.head_dim ||
      p->softmax_scale != o.softmax_scale || p->page_size != o.page_size || p->num_pages != o.num_pages)
    return 0;
  auto same = [](const int32_t *a, const int32_t *b, size_t n) { return std::memcmp(a, b, n * sizeof(int32_t)) == 0; };
  const size_t B = (size_t)o.batch;
  return same(p->q_offsets, o.q_offsets, B + 1) && same(p->kv_lens, o.kv_lens, B) &&
         same(p->page_offsets, o.page_offsets, B + 1) && same(p->page_ids, o.page_ids, (size_t)o.page_offsets[B]);
}

cas_status_t cas_paged_decode_plan_destroy(cas_decode_plan_t *plan) {
  delete plan;
  return CAS_OK;
}

cas_status_t cas_cartridge_adam_workspace_size(const cas_adam_cartridge_t *carts, int32_t n,
                                               int32_t num_kv_heads, int32_t head_dim, size_t *bytes) {
  if (!bytes) return fail(CAS_ERR_INVALID_ARGUMENT, "bytes is NULL");
  AdamPlan ap;
  cas_status_t s = build_adam(carts, n, num_kv_heads, head_dim, nullptr, ap);
  if (s != CAS_OK) return s;
  *bytes = ap.bytes;
  return CAS_OK;
}

cas_status_t cas_cartridge_adam(const cas_adam_cartridge_t *carts, int32_t n, int32_t num_kv_heads,
                                int32_t head_dim, const cas_adam_config_t *cfg, void *workspace,
                                size_t ws_bytes, void *hip_stream) {
  if (!cfg) return fail(CAS_ERR_INVALID_ARGUMENT, "cfg is NULL");
  AdamPlan ap;
  cas_status_t s = build_adam(carts, n, num_kv_heads, head_dim, cfg, ap);
  if (s != CAS_OK) return s;
  if (ap.chunks.empty()) return CAS_OK;
  s = check_workspace(workspace, ws_bytes, ap.bytes);
  if (s != CAS_OK) return s;
  hipStream_t stream = (hipStream_t)hip_stream;
  s = ring_upload(ap.bytes, workspace, stream, [&](char *h) {
    std::memcpy(h, ap.tensors.data(), ap.tensors.size() * sizeof(DevAdamT));
    std::memcpy(h + ap.off_chunks, ap.chunks.data(), ap.chunks.size() * sizeof(DevAdamChunk));
  });
  if (s != CAS_OK) return s;
  AdamParams p{};
  p.tensors = (const DevAdamT *)workspace;
  p.chunks = (const DevAdamChunk *)((char *)workspace + ap.off_chunks);
  p.Hkv = num_kv_heads;
  p.beta1 = cfg->beta1;
  p.beta2 = cfg->beta2;
  p.omb1 = 1.0f - cfg->beta1;
  p.omb2 = 1.0f - cfg->beta2;
  p.eps = cfg->eps;
  hipError_t e = timed("adam", stream, [&] { return launch_adam_bf16(p, head_dim, (int)ap.chunks.size(), stream); });
  if (e != hipSuccess) return hip_fail("adam launch", e);
  return CAS_OK;
}

cas_status_t cas_set_tuning(const cas_tuning_t *t) {
  if (!t) return fail(CAS_ERR_INVALID_ARGUMENT, "tuning is NULL");
  if (t->fwd_splits < 0 || t->dq_splits < 0 || t->fwd_splits > kMaxSplits || t->dq_splits > kMaxSplits)
    return fail(CAS_ERR_INVALID_ARGUMENT, "splits must be in [0, " + std::to_string(kMaxSplits) + "]");
  std::lock_guard<std::mutex> lk(g_tuning_mu);
  g_tuning = *t;
  return CAS_OK;
}

cas_status_t cas_get_tuning(cas_tuning_t *t) {
  if (!t) return fail(CAS_ERR_INVALID_ARGUMENT, "tuning is NULL");
  *t = tuning();
  return CAS_OK;
}

cas_status_t cas_prefix_attn_workspace_size(const cas_problem_t *p, int backward, size_t *bytes) {
  if (!bytes) return fail(CAS_ERR_INVALID_ARGUMENT, "bytes is NULL");
  Plan pl;
  cas_status_t s = build_plan(p, backward != 0, pl);
  if (s != CAS_OK) return s;
  *bytes = backward ? pl.ws_bwd : pl.ws_fwd;
  return CAS_OK;
}

cas_status_t cas_plan_info(const cas_problem_t *p, cas_plan_info_t *out) {
  if (!out) return fail(CAS_ERR_INVALID_ARGUMENT, "out is NULL");
  Plan pf, pb;
  cas_status_t s = build_plan(p, false, pf);
  if (s != CAS_OK) return s;
  s = build_plan(p, true, pb);
  if (s != CAS_OK) return s;
  out->fwd_splits = pf.fwd_splits;
  out->dq_splits = pb.dq_splits;
  out->fwd_workgroups = pf.dt == kBF16 ? (int32_t)pf.items.size() : pf.nqblk * pf.Hkv * pf.B * pf.fwd_splits;
  out->dkdv_workgroups = (int32_t)pb.order_cap;
  out->unique_segments = (int32_t)pb.carts.size();
  out->total_key_tiles = (int32_t)(pb.order_cap / pb.Hkv);
  out->max_prefix_len = pf.max_prefix;
  out->ws_fwd_bytes = pf.ws_fwd;
  out->ws_bwd_bytes = pb.ws_bwd;
  return CAS_OK;
}

cas_status_t cas_prefix_attn_fwd(const cas_problem_t *p, const void *q, const void *k_self,
                                 const void *v_self, void *o, float *lse, void *workspace,
                                 size_t ws_bytes, void *hip_stream) {
  return prefix_attn_fwd_run(p, q, k_self, v_self, o, lse, workspace, ws_bytes, (hipStream_t)hip_stream,
                             nullptr);
}

cas_status_t cas_prefix_attn_bwd(const cas_problem_t *p, const void *q, const void *k_self,
                                 const void *v_self, const void *o, const float *lse,
                                 const void *d_o, void *dq, void *dk_self, void *dv_self,
                                 void *workspace, size_t ws_bytes, void *hip_stream) {
  Plan pl;
  cas_status_t s = build_plan(p, true, pl);
  if (s != CAS_OK) return s;
  if (!q || !k_self || !v_self || !o || !lse || !d_o)
    return fail(CAS_ERR_INVALID_ARGUMENT, "q, k_self, v_self, o, lse and d_o must be non-NULL");
  if (!aligned16(q) || !aligned16(k_self) || !aligned16(v_self) || !aligned16(o) || !aligned16(d_o) ||
      !aligned16(dq) || !aligned16(dk_self) || !aligned16(dv_self) || ((uintptr_t)lse & 3u))
    return fail(CAS_ERR_ALIGNMENT, "tensors must be 16-byte aligned (lse 4-byte)");
  const uintptr_t qbytes = (uintptr_t)pl.T * pl.Hq * pl.D * pl.esize;
  const uintptr_t kvbytes = (uintptr_t)pl.T * pl.Hkv * pl.D * pl.esize;
  std::vector<Interval> iv;
  iv.push_back({(uintptr_t)q, (uintptr_t)q + qbytes, false, 0, "q"});
  iv.push_back({(uintptr_t)k_self, (uintptr_t)k_self + kvbytes, false, 0, "k_self"});
  iv.push_back({(uintptr_t)v_self, (uintptr_t)v_self + kvbytes, false, 0, "v_self"});
  iv.push_back({(uintptr_t)o, (uintptr_t)o + qbytes, false, 0, "o"});
  iv.push_back({(uintptr_t)lse, (uintptr_t)lse + (uintptr_t)pl.T * pl.Hq * 4, false, 0, "lse"});
  iv.push_back({(uintptr_t)d_o, (uintptr_t)d_o + qbytes, false, 0, "d_o"});
  if (dq) iv.push_back({(uintptr_t)dq, (uintptr_t)dq + qbytes, true, (uintptr_t)dq, "dq"});
  if (dk_self) iv.push_back({(uintptr_t)dk_self, (uintptr_t)dk_self + kvbytes, true, (uintptr_t)dk_self, "dk_self"});
  if (dv_self) iv.push_back({(uintptr_t)dv_self, (uintptr_t)dv_self + kvbytes, true, (uintptr_t)dv_self, "dv_self"});
  add_segment_intervals(pl, p, true, iv);
  std::string msg;
  if (!overlap_free(iv, msg)) return fail(CAS_ERR_INVALID_ARGUMENT, msg);
  s = check_workspace(workspace, ws_bytes, pl.ws_bwd);
  if (s != CAS_OK) return s;

  hipStream_t stream = (hipStream_t)hip_stream;
  bind_self_tiles(pl, k_self, v_self);
  build_dkdv_order(pl, dk_self || dv_self);
  s = upload_tables(pl, true, workspace, stream);
  if (s != CAS_OK) return s;
  char *ws = (char *)workspace;
  float *nd = (float *)(ws + pl.off_nd);
  float *lse2 = (float *)(ws + pl.off_lse2);
  const float scale_log2 = pl.scale * 1.4426950408889634f;

  PreParams pp{};
  pp.o = o;
  pp.d_o = d_o;
  pp.lse = lse;
  pp.nd = nd;
  pp.lse2 = lse2;
  pp.rows = (const DevRow *)(ws + pl.off_rows);
  pp.B = pl.B;
  pp.Hkv = pl.Hkv;
  pp.g = pl.g;
  pp.nrows_max = pl.nrows_max;
  pp.nqb_max = pl.nqb_max;
  pp.lse_hs = pl.packed ? (int32_t)pl.T : pl.Sq;
  pp.q = q;
  pp.qT = pl.dt == kBF16 ? ws + pl.off_qT : nullptr;
  pp.doT = pl.dt == kBF16 ? ws + pl.off_doT : nullptr;
  // bf16: the statistics and the transposed Q / dO blocks in one pass.
  hipError_t e = timed("bwd_pre", stream, [&] {
    return pl.dt == kBF16 ? launch_bwd_prologue_bf16(pp, pl.D, stream) : launch_bwd_pre(pp, pl.dt, pl.D, stream);
  });
  if (e != hipSuccess) return hip_fail("bwd_pre launch", e);

  const int n_wg = (int)pl.dkdv_grid;
  auto run_dq = [&]() -> hipError_t {
    if (!dq) return hipSuccess;
    DqParams dp{};
    dp.q = q;
    dp.k_self = k_self;
    dp.v_self = v_self;
    dp.d_o = d_o;
    dp.nd = nd;
    dp.lse2 = lse2;
    dp.dq = dq;
    dp.part_dq = pl.dq_splits > 1 ? (float *)(ws + pl.off_part_dq) : nullptr;
    dp.segs = (const DevSeg *)(ws + pl.off_segs);
    dp.tiles = (const DevTile *)(ws + pl.off_tiles);
    dp.items = (const DevItem *)(ws + pl.off_items);
    dp.rows = (const DevRow *)(ws + pl.off_rows);
    dp.plane = pl.T * pl.Hq;
    dp.B = pl.B;
    dp.Smax = pl.Smax;
    dp.Hkv = pl.Hkv;
    dp.g = pl.g;
    dp.nrows_max = pl.nrows_max;
    dp.nqblk = pl.nqblk;
    dp.splits = pl.dq_splits;
    dp.n_items = (int32_t)pl.items.size();
    dp.scale_log2 = scale_log2;
    dp.scale = pl.scale;
    hipError_t r = timed("dq", stream, [&] { return launch_dq(dp, pl.dt, pl.D, stream); });
    if (r != hipSuccess || pl.dq_splits <= 1) return r;
    DqReduceParams rp{};
    rp.part_dq = dp.part_dq;
    rp.dq = dq;
    rp.rows = dp.rows;
    rp.plane = dp.plane;
    rp.B = pl.B;
    rp.Hkv = pl.Hkv;
    rp.g = pl.g;
    rp.nrows_max = pl.nrows_max;
    rp.splits = pl.dq_splits;
    rp.scale = pl.scale;
    return timed("dq_reduce", stream, [&] { return launch_dq_reduce(rp, pl.dt, pl.D, stream); });
  };
  if (n_wg > 0) {
    DkdvParams kp{};
    kp.q = q;
    kp.k_self = k_self;
    kp.v_self = v_self;
    kp.d_o = d_o;
    kp.nd = nd;
    kp.lse2 = lse2;
    kp.qT = pp.qT;
    kp.doT = pp.doT;
    kp.dk_self = dk_self;
    kp.dv_self = dv_self;
    kp.carts = (const DevCart *)(ws + pl.off_carts);
    kp.uses = (const int32_t *)(ws + pl.off_uses);
    kp.rows = pp.rows;
    kp.order = (const DevWg *)(ws + pl.off_order);
    kp.claim = (int32_t *)(ws + pl.off_claim);
    kp.lists = pl.dkdv_lists;
    kp.list_len = pl.dkdv_list_len;
    kp.list_head = pl.dkdv_list_head;
    kp.bounded = pl.dkdv_bounded;
    kp.B = pl.B;
    kp.Hkv = pl.Hkv;
    kp.g = pl.g;
    kp.scale_log2 = scale_log2;
    kp.scale = pl.scale;
    e = timed("dkdv", stream, [&] { return launch_dkdv(kp, pl.dt, pl.D, n_wg, stream); });
    if (e != hipSuccess) return hip_fail("dkdv launch", e);
  }
  e = run_dq();
  if (e != hipSuccess) return hip_fail("dq launch", e);
  return CAS_OK;
}

cas_status_t cas_cartridge_stage(const cas_stage_copy_t *copies, int32_t n, void *side_stream,
                                 void *done_event) {
  if (n < 0) return fail(CAS_ERR_INVALID_ARGUMENT, "n must be >= 0");
  if (n > 0 && !copies) return fail(CAS_ERR_INVALID_ARGUMENT, "copies is NULL");
  for (int i = 0; i < n; ++i) {
    if (copies[i].bytes == 0) continue;
    if (!copies[i].host_src || !copies[i].dev_dst)
      return fail(CAS_ERR_INVALID_ARGUMENT, "copy " + std::to_string(i) + ": NULL pointer");
  }
  for (int i = 0; i < n; ++i) {
    const cas_stage_copy_t &c = copies[i];
    if (c.bytes == 0) continue;
    const void *ends[2] = {c.host_src, (const char *)c.host_src + c.bytes - 1};
    for (const void *ptr : ends) {
      hipPointerAttribute_t a;
      hipError_t e = hipPointerGetAttributes(&a, ptr);
      if (e != hipSuccess || a.type != hipMemoryTypeHost) {
        (void)hipGetLastError();
        return fail(CAS_ERR_NOT_PINNED, "copy " + std::to_string(i) + ": host_src is not pinned host memory");
      }
    }
    hipPointerAttribute_t d;
    hipError_t e = hipPointerGetAttributes(&d, c.dev_dst);
    if (e != hipSuccess || d.type != hipMemoryTypeDevice) {
      (void)hipGetLastError();
      return fail(CAS_ERR_INVALID_ARGUMENT, "copy " + std::to_string(i) + ": dev_dst is not device memory");
    }
  }
  std::vector<HostCopy> list((size_t)n);
  for (int i = 0; i < n; ++i) list[i] = {copies[i].host_src, copies[i].dev_dst, copies[i].bytes};
  hipStream_t s = (hipStream_t)side_stream;
  {
    hipError_t e = enqueue_copies(list.data(), n, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail("hipMemcpyAsync", e);
  }
  if (done_event) {
    hipError_t e = hipEventRecord((hipEvent_t)done_event, s);
    if (e != hipSuccess) return hip_fail("hipEventRecord", e);
  }
  return CAS_OK;
}

cas_status_t cas_timing_enable(int enable) {
  std::lock_guard<std::mutex> lk(g_time_mu);
  g_timing = enable != 0;
  return CAS_OK;
}

cas_status_t cas_timing_reset(void) {
  std::lock_guard<std::mutex> lk(g_time_mu);
  for (auto &t : g_pending) {
    (void)hipEventSynchronize(t.b);
    g_event_pool.push_back(t.a);
    g_event_pool.push_back(t.b);
  }
  g_pending.clear();
  g_totals.clear();
  return CAS_OK;
}

cas_status_t cas_timing_read(cas_kernel_time_t *out, int32_t cap, int32_t *n_out) {
  if (!n_out || (cap > 0 && !out)) return fail(CAS_ERR_INVALID_ARGUMENT, "NULL output");
  std::lock_guard<std::mutex> lk(g_time_mu);
  for (auto &t : g_pending) {
    hipError_t e = hipEventSynchronize(t.b);
    if (e != hipSuccess) return hip_fail("hipEventSynchronize", e);
    float ms = 0.0f;
    e = hipEventElapsedTime(&ms, t.a, t.b);
    if (e != hipSuccess) return hip_fail("hipEventElapsedTime", e);
    auto &acc = g_totals[t.name];
    acc.first += 1;
    acc.second += ms;
    g_event_pool.push_back(t.a);
    g_event_pool.push_back(t.b);
  }
  g_pending.clear();
  int32_t i = 0;
  for (auto &kv : g_totals) {
    if (i < cap) {
      std::memset(out[i].name, 0, sizeof(out[i].name));
      std::strncpy(out[i].name, kv.first.c_str(), sizeof(out[i].name) - 1);
      out[i].launches = kv.second.first;
      out[i].total_ms = kv.second.second;
    }
    ++i;
  }
  *n_out = i;
  return CAS_OK;
}

}  // extern "C"
