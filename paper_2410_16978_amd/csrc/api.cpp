// Host side of the C ABI declared in include/gsr.h: argument checks,
// workspace layout and the launch sequence of each entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/gsr.h"
#include "common.hpp"

using namespace gsr;

namespace {

constexpr size_t kAlign = 256;

#define HIP_TRY(expr)                      \
  do {                                     \
    if ((expr) != hipSuccess) return GSR_EHIP; \
  } while (0)

#define HIP_TRY_E(expr)                          \
  do {                                           \
    const hipError_t e_ = (expr);                \
    if (e_ != hipSuccess) return e_;             \
  } while (0)

// Lays buffers out in a byte arena; with base == nullptr it only measures.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <typename T> T* take(size_t count) {
    off = (off + kAlign - 1) / kAlign * kAlign;
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// Sort control block: digit counts and offsets of every pass, pass tickets.
// Cleared at the start of each call.
struct SortCtl {
  uint32_t hist[kMaxSortPasses * 256];
  uint32_t pass_ctr[kMaxSortPasses];
  uint32_t scan_ticket;
  uint32_t tile_class[kTileClasses];  // tiles per size class (forward order)
  uint32_t seg_ticket;                // next large tile of the block depth sort
  uint32_t pad[6];
  uint32_t hist12[4096];              // tile counts of the one-pass tile grouping
};

struct PipeBufs {
  ViewD* views = nullptr;
  uint32_t* req_rec = nullptr;
  uint32_t* n_tiles = nullptr;
  uint32_t* offsets = nullptr;
  uint64_t* scan_status = nullptr;  // look-back words of the offsets scan
  uint4* tile_box = nullptr;
  uint64_t* keys_a = nullptr;
  uint64_t* keys_b = nullptr;
  uint32_t* rec_of = nullptr;
  SortCtl* ctl = nullptr;
  uint32_t* status = nullptr;
  uint32_t* class_list = nullptr;  // [kTileClasses][X] tiles by size class
  float* g_pair = nullptr;
  float* g_col = nullptr;    // [R][3] colour gradient of each record (backward)
  uint32_t* g_max = nullptr;       // [n] bits of each Gaussian's largest alpha T (backward)
  uint32_t* alive = nullptr;       // [P] bytes (as words): 1 where a pair's partials were written (backward)
  uint32_t* order_cnt = nullptr;   // [kBatchClasses] batches per work class (backward)
  uint32_t* order_list = nullptr;  // [kBatchClasses][batch capacity] batch indices by class (backward)
  // batch only (the single-call path keeps these in the caller's state)
  float* records = nullptr;
  uint32_t* vals = nullptr;
  uint32_t* ranges = nullptr;
  uint32_t* counters = nullptr;
  uint32_t* sel = nullptr;
  // order-first (order.hip): the record sort, the pairs, and the control
  // words (cleared in one range: tickets, digit counts, unit words, the
  // look-back words of the record passes and the emission)
  uint32_t* boxes = nullptr;  // null: in the state's pair_emit
  uint32_t* sort_keys = nullptr;  // [2][S]
  uint32_t* sort_vals = nullptr;  // [2][S]
  uint32_t* pair_tiles = nullptr;  // [2][P]
  uint32_t* pair_counts = nullptr;  // [blocks + 1][256], above 65536 tiles [blocks + 1][512]
  uint32_t* order_ctl = nullptr;
  size_t order_ctl_words = 0;
};

// Sizes of a call that orders its records before it pairs them.
struct OrderPlan {
  bool on = false;
  bool box4 = false;       // tile boxes of four bytes (no view beyond 255 tiles a side)
  bool own_boxes = false;  // tile boxes in the workspace, not in the state's pair_emit
  size_t S = 0;            // sort slots: records of all sort units
  size_t rec_blocks = 0, seq_blocks = 0;
  uint32_t rec_tile = 0, seq_tile = 0;  // rec_tile, emit_tile of the call's records
  bool small = true;       // every unit has at most kRecSmall records
  bool bound = false;      // for workspace_bytes: the largest sizes of either path's buffers
};

// Whether a call orders its records before it pairs them (one that shares an
// order always does).  Ordering first moves about 12 bytes a record four
// times and 6 a pair twice, where the per-tile path moves 12 a pair twice (up
// to 4096 tiles once) and then sorts every tile; its 14 launches between the
// projection and the blend (two tile digits) cost about 30 us more than the
// other's 6 on small calls.  Measured, per-tile against
// order-first, whole frames, us: beyond 4096 tiles 197 / 192 at 1.0M pairs and
// 158 / 169 at 0.5M (1100 x 1000), 1141 / 860 at 12.5M (2 x 1M records); up
// to 4096 tiles 165 / 190 at 1.0M, 247 / 241 at 2.0M and 870 / 621 at 10M
// (1024 x 1024).
//
// With many pairs a tile the per-tile sort has few blocks at work, and a tile
// beyond 8192 pairs passes through global memory in one of them; how uneven
// the tiles are is not known here.  From 2048 pairs a tile on, order-first is
// ahead even of evenly filled tiles where there is at most one a compute unit
// (158 / 145 at 200, 223 / 172 at 72), beyond that from about 3072 (a step of
// 361 tiles of 1972 pairs 224 / 268, frames of 625 tiles of 2892 278 / 322
// and of 3499 285 / 308, of 7516 381 / 322); it is far ahead of layered shells
// (286 / 183 at 100 tiles of 1815 pairs on average, 2606 / 1106 at 64 of 30k).
// Below, evenly filled tiles are faster sorted by tile (122 / 167 at 1024 tiles
// of 1208; a step of four views, 676 tiles of 1530, 298 / 345), shells are not
// (291 / 214 at 1024 of 1409): one would lose more than it did before this path
// was there, the other only stays what it was, so these are sorted by tile.
// Up to 4096 tiles the same holds above 2^21 pairs in a smaller measure (2500
// tiles, evenly filled 158 / 190 at 2.2M and 352 / 338 at 11M; shells 254 / 221
// at 2.1M, 741 / 493 at 7.9M).
//
// Below two pair slots a record the record passes outweigh the pairs, unless
// tiles are that full; and the boxes of all records, which the backward reads
// from the pair_emit array, fit there if they are of four bytes.
//
// All of that is in pairs, and only a call that reads its pair count back knows
// them before it orders anything; any other goes by its slots, as the caller
// sized them.  One that reads it starts by its slots too and turns to the
// per-tile path if the pairs do not pay: the default capacity of four slots a
// Gaussian and view is often a quarter filled.  One layer of four shown, wall
// time of such a call before there were two paths / ordered first / turned:
// 186 / 215 / 171 at 531k pairs and 231 / 265 / 206 at 1.0M of 800 x 800, 256
// / 286 / 216 at 695k of 512 x 512, 173 / 188 / 142 at 178k of 400 x 400.  Up
// to 256 tiles, one a compute unit, it stays: the largest tile bounds the
// per-tile sort, and ordering first was ahead at any filling (262 / 238 / 207
// for one layer of four at 256 x 256 and 256k pairs, but 1975 / 1103 / 1397
// for the innermost of eight, 472k pairs in few of the tiles).
constexpr uint32_t kOrderMinPairs = 1u << 20, kOrderMinPairsFull = 3u << 16, kOrderFewTiles = 256;
bool order_full(uint64_t X, uint64_t pairs) {
  return pairs >= kOrderMinPairsFull && pairs >= (X <= kOrderFewTiles ? 2048 : 3072) * X;
}
bool order_pays(uint64_t X, uint32_t pairs) {
  return order_full(X, pairs) || pairs >= (tile_sort12(X, pairs) ? 2 * kOrderMinPairs : kOrderMinPairs);
}
bool order_first(uint64_t X, uint32_t P, uint64_t R, bool box4) {
  return P >= (order_full(X, P) && box4 ? R : 2 * R) && order_pays(X, P);
}

// Words of the order-first path that are zero on entry.
size_t order_ctl_words(const OrderPlan& op, size_t n_views) {
  return 8 + n_views * (2 + 4 * 256) + 2 * op.seq_blocks + 4 * 256 * op.rec_blocks;
}

size_t carve(Carver& c, PipeBufs& b, size_t n_views, size_t R, size_t P, size_t n_req, bool batch,
             size_t X, bool backward, const OrderPlan& op) {
  b.views = c.take<ViewD>(std::max<size_t>(n_views, 1));
  b.req_rec = c.take<uint32_t>(n_req + 1);
  b.n_tiles = c.take<uint32_t>(std::max<size_t>(R, 1));
  b.scan_status = c.take<uint64_t>(scan_tiles((uint32_t)R));
  b.ctl = c.take<SortCtl>(1);
  if (op.on) {
    if (op.own_boxes) b.boxes = c.take<uint32_t>((op.box4 ? 1 : 2) * std::max<size_t>(R, 1));
    b.sort_keys = c.take<uint32_t>(2 * std::max<size_t>(op.S, 1));
    b.sort_vals = c.take<uint32_t>(2 * std::max<size_t>(op.S, 1));
    b.pair_tiles = c.take<uint32_t>(2 * (std::max<size_t>(P, 1) + 4));
    b.pair_counts =
        op.bound ? c.take<uint32_t>(((size_t)1 << kPairBits) *
                                    (std::min<size_t>(P / kPairStepSmall + 1, kPairBlocks) + 1))
                 : c.take<uint32_t>((X > 65536 ? (size_t)1 << kPairBits : 256) *
                                    ((size_t)pair_pass_blocks((uint32_t)P) + 1));
    b.order_ctl_words = order_ctl_words(op, n_views);
    b.order_ctl = c.take<uint32_t>(b.order_ctl_words);
  } else {
    b.tile_box = c.take<uint4>(std::max<size_t>(R, 1));  // (where sort_keys is: forward_impl may turn)
    b.keys_a = c.take<uint64_t>(std::max<size_t>(P, 1));
    b.keys_b = c.take<uint64_t>(std::max<size_t>(P, 1));
    b.rec_of = c.take<uint32_t>(std::max<size_t>(P, 1));
    b.status = c.take<uint32_t>(std::max(
        sort_status_words((uint32_t)P),
        op.bound || tile_sort12(X, (uint32_t)P)
            ? tile_sort12_status_words((uint32_t)std::min<size_t>(P, kT12MaxPairs)) : 0));
  }
  b.class_list = c.take<uint32_t>(kTileClasses * std::max<size_t>(X, 1));
  if (backward) {
    b.g_pair = c.take<float>(12 * (std::max<size_t>(P, 1) + 1));  // + one zero entry, index P
    b.g_col = c.take<float>(3 * std::max<size_t>(R, 1));
    b.g_max = c.take<uint32_t>(std::max<size_t>(R / std::max<size_t>(n_views, 1), 1));
    b.alive = c.take<uint32_t>(std::max<size_t>(P, 1) / 4 + 1);
    b.order_cnt = c.take<uint32_t>(kBatchClasses);
    b.order_list = c.take<uint32_t>(kBatchClasses * (P / kBatch + X + 1));
  }
  if (batch) {
    b.offsets = c.take<uint32_t>(R + 1);
    b.records = c.take<float>(kRecordFloats * std::max<size_t>(R, 1));
    b.vals = c.take<uint32_t>(2 * std::max<size_t>(P, 1));
    b.ranges = c.take<uint32_t>(2 * std::max<size_t>(X, 1));
    b.counters = c.take<uint32_t>(4);
    b.sel = c.take<uint32_t>(1);
  }
  return c.off + kAlign;
}

// The order-first plan of the largest buffers: R records in `rec_blocks`
// short pass blocks, own_boxes if any call of the kind keeps its boxes in the
// workspace.
OrderPlan bound_plan(size_t R, size_t rec_blocks, size_t seq_blocks, bool own_boxes) {
  OrderPlan op;
  op.on = op.bound = true;
  op.own_boxes = own_boxes;
  op.S = R;
  op.rec_blocks = rec_blocks;
  op.seq_blocks = seq_blocks;
  return op;
}

// Bytes a workspace of a call has to have.  Which path a call takes turns on
// its sizes, and a pair slot takes 8 bytes on one and 20 or more on the other;
// so that a workspace sized for a call also holds every smaller one, and a
// batch needs no more than the sum of its requests alone (what a server
// budgets), the size is that of the larger layout, with buffers that only
// grow with the sizes, whichever path the call takes.
size_t workspace_bytes(size_t n_views, size_t R, size_t P, size_t n_req, bool batch, size_t X,
                       const OrderPlan& bound) {
  Carver by_tile(nullptr), by_record(nullptr);
  PipeBufs b;
  OrderPlan off;
  off.bound = true;
  return std::max(carve(by_tile, b, n_views, R, P, n_req, batch, X, !batch, off),
                  carve(by_record, b, n_views, R, P, n_req, batch, X, !batch, bound));
}

// One launch zeroes everything a call expects to start at zero: the sort
// control block (digit counts, tickets), the pair count (all four counter
// words for a batch, whose counters live in the workspace; a forward
// state's overflow and error words are sticky, cleared by
// gsr_forward_check), the tile ranges, the scan's and the radix passes'
// look-back words, the sorted-buffer selector and (forward) the
// batch-to-tile map.
// The global radix passes cover only the tile bits of the keys (bits 32
// up); the depth bits are sorted per tile segment.
constexpr int kDepthPasses = 4;
int tile_pass_end(uint64_t total_tiles) {
  int b = 0;
  while (b < 32 && (1ull << b) < total_tiles) ++b;
  return kDepthPasses + (b + 7) / 8;
}

// The views array goes to the device in the arguments of the clear launch as
// far as they hold it (four views), the rest in upload launches of its own;
// never by a copy from pageable host memory.
hipError_t upload_views(ViewD* dst, const ViewD* src, int n_views, WordUpload& up, hipStream_t s) {
  const size_t words = sizeof(ViewD) / 4 * (size_t)n_views, here = std::min(words, sizeof(up.w) / 4);
  up.dst = reinterpret_cast<uint32_t*>(dst);
  up.n = (uint32_t)here;
  std::memcpy(up.w, src, 4 * here);
  return launch_upload(up.dst + here, reinterpret_cast<const uint32_t*>(src) + here, words - here, s);
}

// The look-back words of the per-tile path's radix passes, as the next range
// of a clear.  (The one-pass grouping's block counts are written before they
// are read.)
void tile_pass_words(const PipeBufs& b, size_t X, uint32_t P, ClearSet& cs) {
  const size_t stride = sort_status_stride(P);
  const int pb = kDepthPasses, pe = tile_pass_end(X);
  cs.p[cs.n_ranges] = b.status + (size_t)pb * stride;
  cs.n[cs.n_ranges++] = (size_t)(pe - pb) * stride;
}

hipError_t clear_workspace(const PipeBufs& b, uint32_t* counters, bool sticky_flags, uint32_t* ranges, size_t X,
                           size_t R, uint32_t P, uint32_t* sel, hipStream_t s, const WordUpload* up,
                           uint32_t* batch_tile = nullptr, size_t n_batches = 0) {
  ClearSet cs{};
  cs.p[0] = reinterpret_cast<uint32_t*>(b.ctl);
  cs.n[0] = sizeof(SortCtl) / 4;
  cs.p[1] = counters;
  cs.n[1] = sticky_flags ? 1 : 4;
  cs.p[2] = ranges;
  cs.n[2] = 2 * X;
  cs.p[3] = reinterpret_cast<uint32_t*>(b.scan_status);
  cs.n[3] = 2 * (size_t)scan_tiles((uint32_t)R);
  cs.p[4] = sel;  // the sorted-buffer selector
  cs.n[4] = 1;
  cs.n_ranges = 5;
  if (b.order_ctl) {
    cs.p[cs.n_ranges] = b.order_ctl;
    cs.n[cs.n_ranges++] = b.order_ctl_words;
  } else if (!tile_sort12(X, P)) {
    tile_pass_words(b, X, P, cs);
  }
  if (batch_tile && n_batches) {
    cs.p[cs.n_ranges] = batch_tile;
    cs.n[cs.n_ranges++] = n_batches;
  }
  return launch_clear_multi(cs, s, up);
}

// The order-first fields of a call's views, in view order: unit by unit the
// slots and pass blocks of its records, view by view its emission blocks.
// lead[v] is v for a view that owns its unit's order, else the view whose
// order it follows; cam[v] (nullable entries) the sort camera of a unit
// that shares one; n[v] the records of the view's model.
void plan_order(OrderPlan& op, std::vector<ViewD>& views, const std::vector<int>& lead,
                const std::vector<const gsr_camera*>& cam, const std::vector<uint32_t>& n) {
  for (size_t v = 0; v < views.size(); ++v) {
    ViewD& d = views[v];
    d.sort_off = (uint32_t)op.S;
    d.sort_n = n[v];
    d.sort_blk = (uint32_t)op.rec_blocks;
    d.seq_blk = (uint32_t)op.seq_blocks;
    d.sort_lead = (uint32_t)lead[v];
    op.seq_blocks += div_up(n[v], op.seq_tile);
    if (lead[v] != (int)v) {
      d.sort_mode = kSortFollow;
      continue;
    }
    d.sort_mode = cam[v] ? kSortCamera : kSortOwn;
    if (cam[v]) {
      for (int j = 0; j < 3; ++j) d.sort_r[j] = cam[v]->R[6 + j];
      d.sort_t = cam[v]->t[2];
    }
    op.S += n[v];
    op.small = op.small && n[v] <= kRecSmall;
    op.rec_blocks += div_up(n[v], op.rec_tile);
  }
}

OrderBufs order_bufs(const PipeBufs& b, const OrderPlan& op, int n_views, size_t X, uint32_t P, const uint32_t* boxes,
                     uint32_t* pair_vals, uint32_t* counters, uint32_t* ranges, uint32_t* sel) {
  OrderBufs o;
  std::memset(&o, 0, sizeof(o));
  o.views = b.views;
  o.n_views = n_views;
  o.n_tiles = (uint32_t)X;
  o.rec_blocks = (uint32_t)op.rec_blocks;
  o.seq_blocks = (uint32_t)op.seq_blocks;
  o.seq_tile = op.seq_tile;
  o.rec_tile = op.rec_tile;
  o.small = op.small;
  o.keys_a = b.sort_keys;
  o.keys_b = b.sort_keys + std::max<size_t>(op.S, 1);
  o.vals_a = b.sort_vals;
  o.vals_b = b.sort_vals + std::max<size_t>(op.S, 1);
  o.boxes = boxes;
  o.box4 = op.box4;
  o.counters = counters;
  o.cap = P;
  o.tile_a = b.pair_tiles;
  o.tile_b = b.pair_tiles + ((std::max<size_t>(P, 1) + 3) & ~(size_t)3);
  o.rec_a = pair_vals;
  o.rec_b = pair_vals + P;
  o.ranges = ranges;
  o.sel = sel;
  uint32_t* w = b.order_ctl;  // the 64-bit words first (8-byte aligned)
  o.emit_status = reinterpret_cast<uint64_t*>(w);
  w += 2 * op.seq_blocks;
  o.tickets = w;
  w += 8;
  o.unit = w;
  w += 2 * (size_t)n_views;
  o.rec_hist = w;
  w += 4 * 256 * (size_t)n_views;
  o.rec_status = w;
  o.pair_counts = b.pair_counts;
  return o;
}

bool model_ok(const gsr_model* m) {
  if (!m || m->n < 0 || m->sh_degree < 0 || m->sh_degree > 3) return false;
  if (m->raw != 0 && m->raw != 1) return false;
  if (m->format == GSR_FORMAT_F32)
    return m->n == 0 || (m->mean && m->scale && m->quat && m->opacity && m->sh && m->layer);
  if (m->format != GSR_FORMAT_HALF_PACKED && m->format != GSR_FORMAT_HALF_CODEBOOK) return false;
  const gsr_compressed* c = m->compressed;
  if (m->raw != 0 || !c || c->reserved != 0) return false;
  if (m->n == 0) return true;
  if (!m->layer || !c->mean || !c->scale || !c->quat || !c->opacity || !c->sh_dc) return false;
  if (m->sh_degree == 0) return true;  // no higher coefficients to read
  if (m->format == GSR_FORMAT_HALF_PACKED) {
    for (int ch = 0; ch < 3; ++ch)
      if (!std::isfinite(c->sh_lo[ch]) || !std::isfinite(c->sh_step[ch])) return false;
    return c->sh_packed != nullptr;
  }
  return c->sh_index && c->codebook && c->codebook_size >= 1 && c->codebook_size <= 65536;
}

bool camera_ok(const gsr_camera& c) {
  return c.width > 0 && c.height > 0 && c.width <= 65535 * kTile && c.height <= 65535 * kTile && c.fx > 0.f &&
         c.fy > 0.f;
}

bool view_ok(const gsr_view_state& v) {
  if (v.mip_2d != 0 && (v.mip_2d != 1 || !(v.mip_2d_var > 0.f) || !std::isfinite(v.mip_2d_var))) return false;
  return v.n_clip >= 0 && v.n_clip <= GSR_MAX_CLIP && (v.sort_shared == 0 || v.sort_shared == 1);
}

// Order-first sizes of a call of n_views views of one model.
OrderPlan single_plan(int64_t n, int n_views, int32_t width, int32_t height, uint32_t P, bool shared) {
  OrderPlan op;
  const uint32_t tx = div_up((uint32_t)width, (uint32_t)kTile), ty = div_up((uint32_t)height, (uint32_t)kTile);
  const uint64_t X = (uint64_t)tx * ty * n_views;
  op.box4 = tx <= (uint32_t)kBox4Tiles && ty <= (uint32_t)kBox4Tiles;
  op.on = shared || order_first(X, P, (uint64_t)n * n_views, op.box4);
  if (!op.on) return op;
  op.own_boxes = shared;  // a forward that shares an order has no backward
  const int units = shared ? 1 : n_views;
  op.S = (size_t)units * n;
  op.rec_tile = rec_tile((uint64_t)n * units);
  op.rec_blocks = (size_t)units * div_up((uint32_t)n, op.rec_tile);
  op.small = (uint64_t)n <= kRecSmall;
  op.seq_tile = emit_tile((uint64_t)n * n_views);
  op.seq_blocks = (size_t)n_views * div_up((uint32_t)n, op.seq_tile);
  return op;
}

// workspace_bytes of such a call; shared: of a forward that shares an order too.
size_t single_workspace_bytes(int64_t n, int n_views, int32_t width, int32_t height, uint32_t P, bool shared) {
  const size_t X = (size_t)n_views * div_up((uint32_t)width, (uint32_t)kTile) * div_up((uint32_t)height, (uint32_t)kTile);
  return workspace_bytes((size_t)n_views, (size_t)n * n_views, P, 0, false, X,
                         bound_plan((size_t)n * n_views, (size_t)n_views * div_up((uint32_t)n, kRecTileSmall),
                                    (size_t)n_views * div_up((uint32_t)n, kEmitTileSmall), shared));
}

uint32_t tiles_of(const gsr_camera& c) {
  return div_up((uint32_t)c.width, (uint32_t)kTile) * div_up((uint32_t)c.height, (uint32_t)kTile);
}

ViewD make_view(const gsr_camera& c, const gsr_view_state& vs) {
  ViewD v;
  std::memset(&v, 0, sizeof(v));
  std::memcpy(v.R, c.R, sizeof(v.R));
  std::memcpy(v.t, c.t, sizeof(v.t));
  v.fx = c.fx; v.fy = c.fy; v.cx = c.cx; v.cy = c.cy; v.znear = c.znear; v.guard = c.guard;
  v.W = c.width; v.H = c.height;
  v.tiles_x = (int32_t)div_up((uint32_t)c.width, (uint32_t)kTile);
  v.tiles_y = (int32_t)div_up((uint32_t)c.height, (uint32_t)kTile);
  v.layer_mask = vs.layer_mask;
  v.n_clip = vs.n_clip;
  for (int k = 0; k < vs.n_clip; ++k) {
    for (int j = 0; j < 3; ++j) v.clip[k].n[j] = vs.clip[k].n[j];
    v.clip[k].d = vs.clip[k].d;
    v.clip[k].bits = vs.clip[k].layer_bits;
  }
  for (int j = 0; j < 3; ++j) v.bg[j] = vs.bg[j];
  for (int l = 0; l < 32; ++l) v.layer_op[l] = vs.layer_fade ? vs.layer_opacity[l] : 1.f;
  v.mip_2d = vs.mip_2d ? 1u : 0u;
  v.mip_var = vs.mip_2d_var;
  return v;
}

ModelD make_model(const gsr_model& m) {
  ModelD d;
  std::memset(&d, 0, sizeof(d));
  d.n = m.n; d.D = m.sh_degree;
  d.mean = m.mean; d.scale = m.scale; d.quat = m.quat; d.opacity = m.opacity; d.sh = m.sh; d.layer = m.layer;
  d.raw = m.raw;
  d.fmt = m.format;
  d.filter_3d = m.filter_3d;
  if (m.format != GSR_FORMAT_F32 && m.compressed) {
    const gsr_compressed& c = *m.compressed;
    d.h_mean = c.mean; d.h_scale = c.scale; d.h_quat = c.quat; d.h_opacity = c.opacity; d.h_dc = c.sh_dc;
    d.sh_packed = c.sh_packed; d.sh_index = c.sh_index; d.codebook = c.codebook;
    for (int ch = 0; ch < 3; ++ch) { d.sh_lo[ch] = c.sh_lo[ch]; d.sh_step[ch] = c.sh_step[ch]; }
    d.codebook_size = (uint32_t)c.codebook_size;
  }
  return d;
}

// Jobs: the views of one model in chunks of kMaxJobViews.
std::vector<JobD> make_jobs(const ModelD& m, const std::vector<int>& view_ids) {
  std::vector<JobD> jobs;
  for (size_t i = 0; i < view_ids.size(); i += kMaxJobViews) {
    JobD j;
    std::memset(&j, 0, sizeof(j));
    j.m = m;
    j.n_views = (int32_t)std::min<size_t>(kMaxJobViews, view_ids.size() - i);
    for (int k = 0; k < j.n_views; ++k) j.view[k] = view_ids[i + k];
    jobs.push_back(j);
  }
  return jobs;
}



}  // namespace

struct gsr_timer {
  std::vector<hipEvent_t> pool;
  size_t used = 0;
  struct Mark { int stage; size_t e0, e1; };
  std::vector<Mark> marks;

  hipEvent_t next() {
    if (used == pool.size()) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return nullptr;
      pool.push_back(e);
    }
    return pool[used++];
  }
};

namespace {

// Event pair around one stage when a timer is attached.
struct StageScope {
  gsr_timer* t;
  int stage;
  hipStream_t s;
  size_t e0 = 0;
  bool ok = false;
  StageScope(gsr_timer* tm, int st, hipStream_t str) : t(tm), stage(st), s(str) {
    if (!t) return;
    hipEvent_t e = t->next();
    if (!e) return;
    e0 = t->used - 1;
    ok = hipEventRecord(e, s) == hipSuccess;
  }
  ~StageScope() {
    if (!t || !ok) return;
    hipEvent_t e = t->next();
    if (!e) return;
    if (hipEventRecord(e, s) == hipSuccess) t->marks.push_back({stage, e0, t->used - 1});
  }
};

bool state_ok(const gsr_fwd_state* st) {
  return st && st->records && st->offsets && st->pair_vals && st->sort_sel && st->pair_emit && st->ranges &&
         st->pixel_state && st->last && st->checkpoints && st->batch_map && st->counters &&
         st->pair_capacity < (1u << 30);
}

bool single_view_args_ok(const gsr_model* model, int32_t n_views, const gsr_camera* cams,
                         const gsr_view_state* views) {
  if (!model_ok(model) || n_views <= 0 || !cams || !views) return false;
  for (int v = 0; v < n_views; ++v) {
    if (!camera_ok(cams[v]) || !view_ok(views[v])) return false;
    if (cams[v].width != cams[0].width || cams[v].height != cams[0].height) return false;
  }
  if ((uint64_t)model->n * (uint64_t)n_views >= (1ull << 31)) return false;
  return true;
}

}  // namespace

extern "C" {

gsr_status gsr_timer_create(gsr_timer** out) {
  if (!out) return GSR_EINVAL;
  *out = new gsr_timer();
  return GSR_OK;
}

void gsr_timer_destroy(gsr_timer* t) {
  if (!t) return;
  for (hipEvent_t e : t->pool) (void)hipEventDestroy(e);
  delete t;
}

gsr_status gsr_timer_read(gsr_timer* t, float* ms, uint32_t* calls) {
  if (!t) return GSR_EINVAL;
  float acc[GSR_N_STAGES] = {0};
  uint32_t cnt[GSR_N_STAGES] = {0};
  gsr_status st = GSR_OK;
  for (const gsr_timer::Mark& m : t->marks) {
    float x = 0.f;
    if (hipEventSynchronize(t->pool[m.e1]) != hipSuccess ||
        hipEventElapsedTime(&x, t->pool[m.e0], t->pool[m.e1]) != hipSuccess) {
      st = GSR_EHIP;
      continue;
    }
    acc[m.stage] += x;
    cnt[m.stage] += 1;
  }
  t->marks.clear();
  t->used = 0;
  for (int k = 0; k < GSR_N_STAGES; ++k) {
    if (ms) ms[k] = acc[k];
    if (calls) calls[k] = cnt[k];
  }
  return st;
}

const char* gsr_status_string(gsr_status s) {
  switch (s) {
    case GSR_OK: return "ok";
    case GSR_EINVAL: return "invalid argument";
    case GSR_ENOSPACE: return "workspace or pair capacity too small";
    case GSR_EHIP: return "HIP runtime error";
    case GSR_EDEVICE: return "device-side error";
  }
  return "unknown status";
}

uint32_t gsr_batch_capacity(uint32_t pair_capacity, uint32_t total_tiles) {
  return pair_capacity / (uint32_t)kBatch + total_tiles + 1;
}

size_t gsr_workspace_size(int32_t n, int32_t n_views, int32_t width, int32_t height, uint32_t pair_capacity,
                          int32_t shared_order) {
  if (n < 0 || n_views <= 0 || width <= 0 || height <= 0 || pair_capacity >= (1u << 30)) return 0;
  return single_workspace_bytes(n, n_views, width, height, pair_capacity, shared_order != 0);
}

gsr_status gsr_adam_step(int32_t n, int32_t sh_degree, uint32_t trainable_layers, const uint8_t* layer,
                         const gsr_adam_group* groups, float beta1, float beta2, float eps, int32_t step,
                         float* activity, void* stream) {
  if (n < 0 || sh_degree < 0 || sh_degree > 3 || !groups || step < 1) return GSR_EINVAL;
  if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f)) return GSR_EINVAL;
  if (n == 0) return GSR_OK;
  if (!layer) return GSR_EINVAL;
  const int planes[kAdamGroups] = {3, 3, 4, 1, 3 * (sh_degree + 1) * (sh_degree + 1)};
  AdamArgs a;
  const double bc1 = 1.0 - std::pow((double)beta1, (double)step);
  const double bc2 = 1.0 - std::pow((double)beta2, (double)step);
  for (int gi = 0; gi < kAdamGroups; ++gi) {
    const gsr_adam_group& g = groups[gi];
    if (!g.param || !g.grad || !g.exp_avg || !g.exp_avg_sq || !(g.lr >= 0.f)) return GSR_EINVAL;
    a.g[gi] = AdamGroupD{g.param, g.exp_avg, g.exp_avg_sq, g.grad, planes[gi], (float)((double)g.lr / bc1)};
  }
  a.one_minus_b1 = 1.f - beta1;
  a.b2 = beta2;
  a.one_minus_b2 = 1.f - beta2;
  a.bc2_sqrt = (float)std::sqrt(bc2);
  a.eps = eps;
  HIP_TRY(launch_adam(n, a, layer, trainable_layers, activity, static_cast<hipStream_t>(stream)));
  return GSR_OK;
}

gsr_status gsr_update_activity(int32_t n, int32_t sh_degree, uint32_t trainable_layers, const float* mean_before,
                               const float* mean_after, const float* log_scale_before, const float* log_scale_after,
                               const float* sh_before, const float* sh_after, const uint8_t* layer, float* activity,
                               void* stream) {
  if (n < 0 || sh_degree < 0 || sh_degree > 3) return GSR_EINVAL;
  if (n == 0) return GSR_OK;
  if (!mean_before || !mean_after || !log_scale_before || !log_scale_after || !sh_before || !sh_after || !layer ||
      !activity)
    return GSR_EINVAL;
  HIP_TRY(launch_update_activity(n, sh_degree, trainable_layers, mean_before, mean_after, log_scale_before,
                                 log_scale_after, sh_before, sh_after, layer, activity,
                                 static_cast<hipStream_t>(stream)));
  return GSR_OK;
}

}  // extern "C"

namespace {

// The forward of gsr_rasterize_forward on a given scratch workspace; the
// layout is the forward's and the backward's (backward_layout, what
// gsr_workspace_size measures) or the forward's alone.
gsr_status forward_impl(const gsr_model* model, int32_t n_views, const gsr_camera* cams,
                        const gsr_view_state* views, gsr_fwd_state* state, void* ws, size_t ws_bytes, float* rgb,
                        float* alpha, uint32_t* n_pairs_host, const gsr_debug* debug, gsr_timer* timer,
                        void* stream, bool backward_layout) {
  if (!single_view_args_ok(model, n_views, cams, views) || !state || !ws || !rgb || !alpha) return GSR_EINVAL;
  if (!state_ok(state)) return GSR_EINVAL;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const int W = cams[0].width, H = cams[0].height;
  const uint32_t n = (uint32_t)model->n;
  const uint32_t R = n * (uint32_t)n_views;
  const uint32_t P = state->pair_capacity;
  const uint32_t tiles_per_view = tiles_of(cams[0]);
  const uint64_t X = (uint64_t)tiles_per_view * n_views;
  if (X >= kBatchTileMask || state->batch_capacity < gsr_batch_capacity(P, (uint32_t)X)) return GSR_EINVAL;
  const size_t plane = (size_t)W * H;
  // one depth order for all views: by the depth in views[0].sort_cam
  const bool shared = views[0].sort_shared != 0;
  OrderPlan op = single_plan(n, n_views, W, H, P, shared);
  if (backward_layout && single_workspace_bytes(n, n_views, W, H, P, shared) > ws_bytes) return GSR_ENOSPACE;
  Carver c(ws);
  PipeBufs b;
  if (carve(c, b, n_views, R, P, 0, false, X, backward_layout, op) > ws_bytes) return GSR_ENOSPACE;

  std::vector<ViewD> hv(n_views);
  std::vector<int> ids(n_views);
  for (int v = 0; v < n_views; ++v) {
    ViewD d = make_view(cams[v], views[v]);
    d.tile_off = (uint32_t)v * tiles_per_view;
    d.rec_off = (uint32_t)v * n;
    d.rgb = rgb + 3 * plane * v;
    d.alpha = alpha + plane * v;
    d.pix = state->pixel_state + 4 * plane * v;
    d.last = state->last + plane * v;
    hv[v] = d;
    ids[v] = v;
  }
  uint32_t* boxes = nullptr;
  if (op.on) {
    boxes = op.own_boxes ? b.boxes : state->pair_emit;
    std::vector<int> lead(ids);
    std::vector<const gsr_camera*> cam(n_views, nullptr);
    if (shared) {
      std::fill(lead.begin(), lead.end(), 0);
      cam[0] = &views[0].sort_cam;
      hv[0].sort_whole = n_views <= kMaxJobViews;  // (one projection job)
    }
    OrderPlan made = op;
    made.S = made.rec_blocks = made.seq_blocks = 0;
    plan_order(made, hv, lead, cam, std::vector<uint32_t>(n_views, n));
  }
  WordUpload up;
  HIP_TRY(upload_views(b.views, hv.data(), n_views, up, s));
  HIP_TRY(clear_workspace(b, state->counters, true, state->ranges, X, R, P, state->sort_sel, s, &up,
                          state->batch_map + X + 1, state->batch_capacity));
  const ModelD md = make_model(*model);
  {
    StageScope sc(timer, GSR_STAGE_PROJECT, s);
    for (const JobD& j : make_jobs(md, ids))
      HIP_TRY(launch_project(j, b.views, state->records, b.n_tiles, b.tile_box, boxes, op.box4, b.sort_keys, state->counters,
                             s));
  }
  OrderBufs o;
  if (op.on)
    o = order_bufs(b, op, n_views, X, P, boxes, state->pair_vals, state->counters, state->ranges, state->sort_sel);
  {
    StageScope sc(timer, GSR_STAGE_SCAN, s);
    if (op.on)
      HIP_TRY(launch_order_scan(o, b.n_tiles, state->offsets, b.scan_status, &b.ctl->scan_ticket, R, s));
    else
      HIP_TRY(launch_scan(b.n_tiles, state->offsets, b.scan_status, &b.ctl->scan_ticket, R, state->counters, P, s));
  }
  BoxSource by_box{};
  if (n_pairs_host) {
    // the pair count, and the sticky error word (this call's scan, or an
    // earlier call on this state that nobody checked)
    uint32_t cnt[3] = {0, 0, 0};
    HIP_TRY(hipMemcpyAsync(cnt, state->counters, sizeof(cnt), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    *n_pairs_host = cnt[kCntPairs];
    if (cnt[kCntError]) return GSR_EDEVICE;
    if (cnt[kCntPairs] > P) {
      HIP_TRY(launch_clear_u32(state->counters + kCntOverflow, 1, s));  // this call's overflow is reported now
      return GSR_ENOSPACE;
    }
    // Too few pairs to order the records first: by tile from here on, in that
    // path's layout of the workspace, which holds the views, counts and sort
    // words where they are and the depth keys in its tile boxes' place.  The
    // boxes stay in pair_emit, where the backward looks for them.  (An
    // inspected call stays: the debug copies are of the path it started on.)
    if (op.on && !shared && !debug && X > kOrderFewTiles && !order_pays(X, cnt[kCntPairs])) {
      Carver ct(ws);
      PipeBufs bt;
      if (carve(ct, bt, n_views, R, P, 0, false, X, backward_layout, OrderPlan{}) > ws_bytes) return GSR_ENOSPACE;
      by_box = BoxSource{boxes, b.sort_keys, n, tiles_per_view, (uint32_t)hv[0].tiles_x, op.box4};
      b = bt;
      op.on = false;
      if (!tile_sort12(X, P)) {
        ClearSet cs{};
        tile_pass_words(b, X, P, cs);
        HIP_TRY(launch_clear_multi(cs, s, nullptr));
      }
    }
  }
  if (op.on) {
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      HIP_TRY(launch_order(o, s));
    }
    {
      StageScope sc(timer, GSR_STAGE_RANGES, s);
      HIP_TRY(launch_tile_order(state->ranges, (uint32_t)X, b.ctl->tile_class, b.class_list, s));
    }
    if (debug)
      HIP_TRY(launch_order_debug(o, R, state->records, state->offsets, debug->tile_box, debug->keys_emit,
                                 debug->vals_emit, debug->keys_sorted, s));
  } else {
    {
      StageScope sc(timer, GSR_STAGE_DUPLICATE, s);
      HIP_TRY(launch_duplicate(b.n_tiles, state->offsets, b.tile_box, R, state->counters, P, b.keys_a,
                               state->pair_vals, b.rec_of, by_box, s));
    }
    if (debug) {
      if (debug->keys_emit) HIP_TRY(hipMemcpyAsync(debug->keys_emit, b.keys_a, 8ull * P, hipMemcpyDeviceToDevice, s));
      if (debug->vals_emit) HIP_TRY(hipMemcpyAsync(debug->vals_emit, b.rec_of, 4ull * P, hipMemcpyDeviceToDevice, s));
    }
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      if (tile_sort12(X, P))
        HIP_TRY(launch_tile_sort12(b.keys_a, b.keys_b, state->pair_vals, state->pair_vals + P, state->counters, P,
                                   (uint32_t)X, b.ctl->hist12, b.status, state->ranges, b.ctl->tile_class,
                                   b.class_list, state->sort_sel, state->counters + kCntError, s));
      else
        HIP_TRY(launch_sort(b.keys_a, b.keys_b, state->pair_vals, state->pair_vals + P, state->counters, P,
                            kDepthPasses, tile_pass_end(X), b.ctl->hist, b.status, b.ctl->pass_ctr,
                            state->sort_sel, state->counters + kCntError, s));
    }
    {
      StageScope sc(timer, GSR_STAGE_RANGES, s);
      if (!tile_sort12(X, P)) {  // (the one-pass grouping writes the ranges and classes itself)
        HIP_TRY(launch_ranges(b.keys_a, b.keys_b, state->sort_sel, state->counters, P, (uint32_t)X, state->ranges, s));
        HIP_TRY(launch_tile_order(state->ranges, (uint32_t)X, b.ctl->tile_class, b.class_list, s));
      }
    }
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      HIP_TRY(launch_sort_segments(b.keys_a, b.keys_b, state->pair_vals, state->pair_vals + P, state->sort_sel,
                                   state->ranges, (uint32_t)X, b.rec_of, state->counters, P,
                                   by_box.boxes ? nullptr : state->pair_emit,
                                   debug ? debug->keys_sorted : nullptr, b.ctl->tile_class, b.class_list,
                                   &b.ctl->seg_ticket, state->counters + kCntError, s));
    }
  }
  uint32_t* batch_tile = state->batch_map + X + 1;
  {
    StageScope sc(timer, GSR_STAGE_BLEND, s);
    HIP_TRY(launch_blend_fwd(b.views, n_views, (uint32_t)X, state->records, R, state->pair_vals,
                                  state->sort_sel, P, state->ranges, batch_tile, state->batch_capacity,
                                  nullptr, shared ? nullptr : reinterpret_cast<float4*>(state->checkpoints), b.ctl->tile_class,
                                  b.class_list, s));
  }
  if (debug) {
    if (debug->n_tiles) HIP_TRY(hipMemcpyAsync(debug->n_tiles, b.n_tiles, 4ull * R, hipMemcpyDeviceToDevice, s));
    if (debug->tile_box && !op.on)
      HIP_TRY(hipMemcpyAsync(debug->tile_box, b.tile_box, 16ull * R, hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
  }
  return GSR_OK;
}

}  // namespace

extern "C" {

gsr_status gsr_rasterize_forward(const gsr_model* model, int32_t n_views, const gsr_camera* cams,
                                 const gsr_view_state* views, gsr_fwd_state* state, void* ws, size_t ws_bytes,
                                 float* rgb, float* alpha, uint32_t* n_pairs_host, const gsr_debug* debug,
                                 gsr_timer* timer, void* stream) {
  return forward_impl(model, n_views, cams, views, state, ws, ws_bytes, rgb, alpha, n_pairs_host, debug, timer,
                      stream, true);
}

}  // extern "C"

// ---------------------------------------------------------------- no allocation
// The scratch of gsr_rasterize_forward_noalloc: a file-scope device array
// (one copy per GPU, held until the process ends).  Host code never uses the
// array's name as an address (on the host it is a stand-in symbol): each
// device's address comes from hipGetSymbolAddress, taken once per device
// with that device current and kept here.
namespace {

constexpr size_t kNoallocScratchBytes = (size_t)GSR_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) uint8_t scratch[kNoallocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

gsr_status scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return GSR_EHIP;
  if (dev < 0 || dev >= kMaxDevices) return GSR_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GSR_EHIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return GSR_OK;
}

}  // namespace

extern "C" {

gsr_status gsr_rasterize_forward_noalloc(const gsr_model* model, int32_t n_views, const gsr_camera* cams,
                                         const gsr_view_state* views, gsr_fwd_state* state, float* rgb,
                                         float* alpha, uint32_t* n_pairs_host, void* stream) {
  if (!single_view_args_ok(model, n_views, cams, views) || !state || !rgb || !alpha || !state_ok(state))
    return GSR_EINVAL;
  const uint64_t X = (uint64_t)tiles_of(cams[0]) * (uint64_t)n_views;
  // One rule refuses a size or not, whichever path the call takes: the
  // per-tile path's scratch and, of a shared order, what one takes that sorts
  // the Gaussians and pairs each view in their order (two buffers of keys and
  // values, the sort's words, and the records' sequence).  The order-first
  // path needs less.
  const bool shared = views[0].sort_shared != 0;
  const size_t n = (size_t)model->n, R = n * (size_t)n_views;
  const uint32_t P = state->pair_capacity;
  Carver rule(nullptr), own(nullptr);
  PipeBufs b;
  size_t need = carve(rule, b, (size_t)n_views, R, P, 0, false, X, false, OrderPlan{});
  if (shared) {
    const size_t keys = std::max<size_t>(n, 1), recs = std::max<size_t>(R, 1);
    for (int half = 0; half < 2; ++half) rule.take<uint64_t>(keys);
    for (int half = 0; half < 2; ++half) rule.take<uint32_t>(keys);
    rule.take<SortCtl>(1);
    rule.take<uint32_t>(sort_status_words((uint32_t)keys));
    rule.take<uint32_t>(4);
    for (int words = 0; words < 2; ++words) rule.take<uint32_t>(recs);
    rule.take<uint4>(recs);
    need = rule.off + kAlign;
  }
  need = std::max(need, carve(own, b, (size_t)n_views, R, P, 0, false, X, false,
                              single_plan(model->n, n_views, cams[0].width, cams[0].height, P, shared)));
  if (need > kNoallocScratchBytes) return GSR_ENOSPACE;
  void* ws = nullptr;
  const gsr_status st = scratch_of_current_device(&ws);
  if (st != GSR_OK) return st;
  return forward_impl(model, n_views, cams, views, state, ws, kNoallocScratchBytes, rgb, alpha, n_pairs_host,
                      nullptr, nullptr, stream, false);
}

gsr_status gsr_forward_check(const gsr_fwd_state* state, uint32_t* n_pairs_host, void* stream) {
  if (!state || !state->counters) return GSR_EINVAL;
  uint32_t cnt[4] = {0, 0, 0, 0};
  const hipStream_t s = static_cast<hipStream_t>(stream);
  HIP_TRY(hipMemcpyAsync(cnt, state->counters, sizeof(cnt), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  // the overflow and error words are reported once: cleared for the calls to come
  HIP_TRY(launch_clear_u32(state->counters + kCntOverflow, 2, s));
  if (n_pairs_host) *n_pairs_host = cnt[kCntPairs];
  if (cnt[kCntError]) return GSR_EDEVICE;
  if (cnt[kCntOverflow]) return GSR_ENOSPACE;
  return GSR_OK;
}

gsr_status gsr_rasterize_backward(const gsr_model* model, int32_t n_views, const gsr_camera* cams,
                                  const gsr_view_state* views, const gsr_fwd_state* state, const float* dL_drgb,
                                  const float* dL_dalpha, uint32_t trainable_layers, void* ws, size_t ws_bytes,
                                  const gsr_grads* grads, float* max_contrib, float* activity, gsr_timer* timer,
                                  void* stream) {
  if (!single_view_args_ok(model, n_views, cams, views) || !state || !ws || !grads) return GSR_EINVAL;
  if (n_views > kMaxJobViews || views[0].sort_shared || model->format != GSR_FORMAT_F32 || model->filter_3d)
    return GSR_EINVAL;
  for (int v = 0; v < n_views; ++v)
    if (views[v].mip_2d) return GSR_EINVAL;  // the Mip filters are rendered, not differentiated
  if (model->n > 0 && (!grads->g_mean || !grads->g_scale || !grads->g_quat || !grads->g_opacity || !grads->g_sh))
    return GSR_EINVAL;
  if (!state_ok(state)) return GSR_EINVAL;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const int W = cams[0].width, H = cams[0].height;
  const uint32_t n = (uint32_t)model->n;
  const uint32_t R = n * (uint32_t)n_views;
  const uint32_t P = state->pair_capacity;
  const uint32_t tiles_per_view = tiles_of(cams[0]);
  const uint64_t X = (uint64_t)tiles_per_view * n_views;
  const size_t plane = (size_t)W * H;
  Carver c(ws);
  PipeBufs b;
  const OrderPlan op = single_plan(n, n_views, W, H, P, false);
  if (single_workspace_bytes(n, n_views, W, H, P, false) > ws_bytes ||
      carve(c, b, n_views, R, P, 0, false, X, true, op) > ws_bytes)
    return GSR_ENOSPACE;
  std::vector<ViewD> hv(n_views);
  std::vector<int> ids(n_views);
  for (int v = 0; v < n_views; ++v) {
    ViewD d = make_view(cams[v], views[v]);
    d.tile_off = (uint32_t)v * tiles_per_view;
    d.rec_off = (uint32_t)v * n;
    d.pix = state->pixel_state + 4 * plane * v;
    d.last = state->last + plane * v;
    hv[v] = d;
    ids[v] = v;
  }
  if (n == 0) return GSR_OK;
  if (X >= kBatchTileMask || state->batch_capacity < gsr_batch_capacity(P, (uint32_t)X)) return GSR_EINVAL;
  // batch indices are below P / 256 + X + 1 (the order list's row length)
  const uint32_t n_batches = std::min(state->batch_capacity, gsr_batch_capacity(P, (uint32_t)X));
  {
    WordUpload up;
    HIP_TRY(upload_views(b.views, hv.data(), n_views, up, s));
    ClearSet cs{};
    cs.p[0] = b.order_cnt;
    cs.n[0] = kBatchClasses;
    cs.p[1] = b.alive;
    cs.n[1] = (size_t)P / 4 + 1;
    cs.p[2] = reinterpret_cast<uint32_t*>(b.g_pair + 12 * (size_t)P);  // the zero entry
    cs.n[2] = 12;
    cs.p[3] = b.g_max;
    cs.n[3] = max_contrib ? n : 0;
    cs.n_ranges = 4;
    HIP_TRY(launch_clear_multi(cs, s, up.n ? &up : nullptr));
  }
  const uint32_t* batch_tile = state->batch_map + X + 1;
  {
    StageScope sc(timer, GSR_STAGE_BWD_ORDER, s);
    HIP_TRY(launch_batch_order(batch_tile, n_batches, b.order_cnt, b.order_list, s));
  }
  {
    StageScope sc(timer, GSR_STAGE_BLEND_BWD, s);
    HIP_TRY(launch_blend_bwd(b.views, n_views, state->records, R, state->pair_vals, state->sort_sel, P,
                             state->ranges, reinterpret_cast<const float4*>(state->checkpoints), batch_tile,
                             n_batches, b.order_cnt, b.order_list, dL_drgb, dL_dalpha, state->pair_emit,
                             op.on ? state->pair_emit : nullptr, op.box4, state->offsets,
                             b.g_pair, reinterpret_cast<uint8_t*>(b.alive), max_contrib ? b.g_max : nullptr, s));
  }
  const ModelD md = make_model(*model);
  {
    StageScope sc(timer, GSR_STAGE_PROJECT_BWD, s);
    for (const JobD& j : make_jobs(md, ids))
      HIP_TRY(launch_project_bwd(j, b.views, state->records, state->offsets, b.g_pair,
                                 reinterpret_cast<const uint8_t*>(b.alive), P,
                                 state->counters, trainable_layers, grads->g_mean, grads->g_scale, grads->g_quat,
                                 grads->g_opacity, grads->g_sh, b.g_col, b.g_max, max_contrib, activity,
                                 grads->densify_grad, grads->densify_count, s));
  }
  return GSR_OK;
}

// ---------------------------------------------------------------- batch
namespace {

struct BatchPlan {
  std::vector<ViewD> views;
  std::vector<uint32_t> req_rec;
  uint64_t R = 0, X = 0;
  uint64_t rec_blocks = 0, seq_blocks = 0;  // of short blocks (bound_plan)
  // with any request sharing one depth order between its eyes, or where
  // order_first says so, the records are ordered before they are paired
  OrderPlan order;
};

bool plan_batch(const gsr_model* models, int32_t n_models, const gsr_request* reqs, int32_t n_req,
                uint32_t pair_capacity, BatchPlan& bp) {
  if (!models || n_models <= 0 || !reqs || n_req <= 0) return false;
  for (int m = 0; m < n_models; ++m)
    if (!model_ok(&models[m])) return false;
  bp.req_rec.assign(n_req + 1, 0);
  for (int q = 0; q < n_req; ++q) {
    const gsr_request& r = reqs[q];
    if (r.model < 0 || r.model >= n_models || r.n_views < 1 || r.n_views > 2 || !view_ok(r.vs)) return false;
    bp.req_rec[q] = (uint32_t)bp.R;
    for (int e = 0; e < r.n_views; ++e) {
      if (!camera_ok(r.cam[e]) || !r.rgb[e] || !r.alpha[e]) return false;
      ViewD d = make_view(r.cam[e], r.vs);
      d.model = (uint32_t)r.model;
      d.request = (uint32_t)q;
      d.rec_off = (uint32_t)bp.R;
      d.tile_off = (uint32_t)bp.X;
      d.rgb = r.rgb[e];
      d.alpha = r.alpha[e];
      bp.views.push_back(d);
      bp.R += (uint64_t)models[r.model].n;
      bp.rec_blocks += div_up((uint32_t)models[r.model].n, kRecTileSmall);
      bp.seq_blocks += div_up((uint32_t)models[r.model].n, kEmitTileSmall);
      bp.X += tiles_of(r.cam[e]);
    }
  }
  bp.req_rec[n_req] = (uint32_t)bp.R;
  if (bp.R >= (1ull << 31) || bp.X >= (1ull << 31)) return false;
  bool shared = false;
  for (int q = 0; q < n_req; ++q) shared = shared || reqs[q].vs.sort_shared != 0;
  bp.order.box4 = true;
  for (const ViewD& d : bp.views) bp.order.box4 = bp.order.box4 && d.tiles_x <= kBox4Tiles && d.tiles_y <= kBox4Tiles;
  bp.order.on = shared || order_first(bp.X, pair_capacity, bp.R, bp.order.box4);
  if (bp.order.on) {
    bp.order.own_boxes = true;
    bp.order.seq_tile = emit_tile(bp.R);
    bp.order.rec_tile = rec_tile(bp.R);
    // each view is a sort unit by its own depth, except the eyes of a
    // request that shares one order: the first eye sorts by the request's
    // sort camera, the second follows it
    std::vector<int> lead;
    std::vector<const gsr_camera*> cam;
    std::vector<uint32_t> n;
    std::vector<uint32_t> views_of(n_models, 0u);
    for (int q = 0; q < n_req; ++q) {
      const gsr_request& r = reqs[q];
      const bool sh = r.vs.sort_shared != 0;
      const int first = (int)lead.size();
      for (int e = 0; e < r.n_views; ++e) {
        lead.push_back(sh ? first : first + e);
        cam.push_back(sh && e == 0 ? &r.vs.sort_cam : nullptr);
        n.push_back((uint32_t)models[r.model].n);
      }
      // (a model's views go through the projection kMaxJobViews at a time)
      const uint32_t j0 = views_of[r.model], j1 = j0 + (uint32_t)r.n_views;
      bp.views[first].sort_whole = j0 / kMaxJobViews == (j1 - 1) / kMaxJobViews;
      views_of[r.model] = j1;
    }
    plan_order(bp.order, bp.views, lead, cam, n);
  }
  return true;
}

size_t batch_workspace_bytes(const BatchPlan& bp, int32_t n_req, uint32_t P) {
  return workspace_bytes(bp.views.size(), bp.R, P, n_req, true, bp.X,
                         bound_plan(bp.R, bp.rec_blocks, bp.seq_blocks, true));
}

}  // namespace

size_t gsr_batch_workspace_size(const gsr_model* models, int32_t n_models, const gsr_request* reqs, int32_t n_req,
                                uint32_t pair_capacity) {
  BatchPlan bp;
  if (!plan_batch(models, n_models, reqs, n_req, pair_capacity, bp) || pair_capacity >= (1u << 30)) return 0;
  return batch_workspace_bytes(bp, n_req, pair_capacity);
}

gsr_status gsr_render_batch(const gsr_model* models, int32_t n_models, const gsr_request* reqs, int32_t n_req,
                            uint32_t pair_capacity, void* ws, size_t ws_bytes, int32_t* req_status, gsr_timer* timer,
                            void* stream) {
  BatchPlan bp;
  if (!plan_batch(models, n_models, reqs, n_req, pair_capacity, bp) || !ws || !req_status || pair_capacity >= (1u << 30))
    return GSR_EINVAL;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const uint32_t P = pair_capacity;
  const uint32_t R = (uint32_t)bp.R;
  const int n_views = (int)bp.views.size();
  Carver c(ws);
  PipeBufs b;
  if (batch_workspace_bytes(bp, n_req, P) > ws_bytes ||
      carve(c, b, n_views, R, P, n_req, true, bp.X, false, bp.order) > ws_bytes)
    return GSR_ENOSPACE;
  WordUpload up;
  HIP_TRY(upload_views(b.views, bp.views.data(), n_views, up, s));
  HIP_TRY(launch_upload(b.req_rec, bp.req_rec.data(), (size_t)n_req + 1, s));
  HIP_TRY(clear_workspace(b, b.counters, false, b.ranges, bp.X, R, P, b.sel, s, &up));
  {
    StageScope sc(timer, GSR_STAGE_PROJECT, s);
    for (int m = 0; m < n_models; ++m) {
      std::vector<int> ids;
      for (int v = 0; v < n_views; ++v)
        if ((int)bp.views[v].model == m) ids.push_back(v);
      if (ids.empty()) continue;
      const ModelD md = make_model(models[m]);
      for (const JobD& j : make_jobs(md, ids))
        HIP_TRY(launch_project(j, b.views, b.records, b.n_tiles, b.tile_box, b.boxes, bp.order.box4, b.sort_keys, b.counters, s));
    }
  }
  OrderBufs o;
  if (bp.order.on) o = order_bufs(b, bp.order, n_views, bp.X, P, b.boxes, b.vals, b.counters, b.ranges, b.sel);
  {
    StageScope sc(timer, GSR_STAGE_SCAN, s);
    if (bp.order.on)
      HIP_TRY(launch_order_scan(o, b.n_tiles, b.offsets, b.scan_status, &b.ctl->scan_ticket, R, s));
    else
      HIP_TRY(launch_scan(b.n_tiles, b.offsets, b.scan_status, &b.ctl->scan_ticket, R, b.counters, P, s));
    // (ordered records are emitted view by view, so a request's pairs end at
    // offsets[req_rec[q + 1]] in either order)
    HIP_TRY(launch_batch_status(b.req_rec, n_req, b.offsets, P, b.counters, req_status, s));
  }
  if (bp.order.on) {
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      HIP_TRY(launch_order(o, s));
    }
    StageScope sc(timer, GSR_STAGE_RANGES, s);
    HIP_TRY(launch_tile_order(b.ranges, (uint32_t)bp.X, b.ctl->tile_class, b.class_list, s));
  } else {
    {
      StageScope sc(timer, GSR_STAGE_DUPLICATE, s);
      HIP_TRY(launch_duplicate(b.n_tiles, b.offsets, b.tile_box, R, b.counters, P, b.keys_a, b.vals, b.rec_of,
                               BoxSource{}, s));
    }
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      if (tile_sort12(bp.X, P))
        HIP_TRY(launch_tile_sort12(b.keys_a, b.keys_b, b.vals, b.vals + P, b.counters, P, (uint32_t)bp.X,
                                   b.ctl->hist12, b.status, b.ranges, b.ctl->tile_class, b.class_list, b.sel,
                                   b.counters + kCntError, s));
      else
        HIP_TRY(launch_sort(b.keys_a, b.keys_b, b.vals, b.vals + P, b.counters, P, kDepthPasses,
                            tile_pass_end(bp.X), b.ctl->hist, b.status, b.ctl->pass_ctr, b.sel,
                            b.counters + kCntError, s));
    }
    {
      StageScope sc(timer, GSR_STAGE_RANGES, s);
      if (!tile_sort12(bp.X, P)) {  // (the one-pass grouping writes the ranges and classes itself)
        HIP_TRY(launch_ranges(b.keys_a, b.keys_b, b.sel, b.counters, P, (uint32_t)bp.X, b.ranges, s));
        HIP_TRY(launch_tile_order(b.ranges, (uint32_t)bp.X, b.ctl->tile_class, b.class_list, s));
      }
    }
    {
      StageScope sc(timer, GSR_STAGE_SORT, s);
      HIP_TRY(launch_sort_segments(b.keys_a, b.keys_b, b.vals, b.vals + P, b.sel, b.ranges, (uint32_t)bp.X, b.rec_of,
                                   b.counters, P, nullptr, nullptr, b.ctl->tile_class, b.class_list,
                                   &b.ctl->seg_ticket, b.counters + kCntError, s));
    }
  }
  {
    StageScope sc(timer, GSR_STAGE_BLEND, s);
    HIP_TRY(launch_blend_fwd(b.views, n_views, (uint32_t)bp.X, b.records, R, b.vals, b.sel, P, b.ranges,
                                  nullptr, 0, req_status, nullptr, b.ctl->tile_class, b.class_list, s));
  }
  HIP_TRY(launch_batch_error(b.counters, n_req, req_status, s));
  return GSR_OK;
}

gsr_status gsr_activate(const gsr_model* model, float* scale_out, float* opacity_out, void* stream) {
  if (!model_ok(model) || model->format != GSR_FORMAT_F32 || (model->n > 0 && (!scale_out || !opacity_out)))
    return GSR_EINVAL;
  HIP_TRY(launch_activate(make_model(*model), scale_out, opacity_out, static_cast<hipStream_t>(stream)));
  return GSR_OK;
}

size_t gsr_l1_loss_workspace_size(int32_t n_views, int32_t width, int32_t height) {
  if (n_views <= 0 || n_views > kMaxJobViews || width <= 0 || height <= 0) return 0;
  const uint64_t hw = (uint64_t)width * (uint64_t)height;
  if (hw * (uint64_t)n_views >= (1ull << 31)) return 0;
  return 8 * (size_t)std::min<uint32_t>(l1_loss_blocks(n_views, (int)hw), 1024u);
}

gsr_status gsr_l1_alpha_loss(int32_t n_views, int32_t width, int32_t height, const float* rgb, const float* alpha,
                             const float* target_rgb, const float* target_alpha, const float* bg_host, void* ws,
                             size_t ws_bytes, float* loss, const float* g_loss, float* dL_drgb, float* dL_dalpha,
                             void* stream) {
  const size_t need = gsr_l1_loss_workspace_size(n_views, width, height);
  if (need == 0 || !rgb || !alpha || !target_rgb || !target_alpha || !bg_host || !ws) return GSR_EINVAL;
  if ((dL_drgb == nullptr) != (dL_dalpha == nullptr)) return GSR_EINVAL;
  if (ws_bytes < need) return GSR_ENOSPACE;
  HIP_TRY(launch_l1_loss(n_views, width * height, rgb, alpha, target_rgb, target_alpha, bg_host,
                         static_cast<float*>(ws), loss, g_loss, dL_drgb, dL_dalpha, static_cast<hipStream_t>(stream)));
  return GSR_OK;
}

}  // extern "C"
