// Order-first pair lists: the records of every view are sorted by depth
// before they are paired, each view's pairs are emitted in that order, and a
// stable grouping by tile leaves every tile's pairs in depth order (ties in
// record order), the order a sort of the pairs by (tile, depth, record)
// gives.  A record covers several tiles, so sorting the records moves far
// fewer items than sorting the pairs, no pair carries a depth, and no tile
// needs a sort of its own.
//
// Stages (all sizes known on the host only as bounds; every count is read on
// the device):
//   k_scan_hist  the scan of the tile counts in record order, and the digit
//                counts of the records' depth keys, per sort unit
//   k_rec_pass   four stable 8-bit passes per unit; the first drops culled
//                records (k_rec_small instead for units of at most 8192)
//   k_emit       the pairs (tile, record) in the sorted order, with the scan
//                of the tile counts (decoupled look-back) in the same launch
//   k_pair_*     stable passes over the tile digits (at most 9 bits each):
//                count, scan, scatter
//   k_tile_runs  the tiles' [start, end)
//
// A sort unit is one view (its own depth), or the views of a stereo frame
// that share one order (the depth in the sort camera).  A unit's keys and
// records lie in consecutive slots; the passes run over the blocks of all
// units in one launch and look back within a unit only, so no pass orders
// the units.
//
// Pairs carry 2 bytes of tile (4 above 65536 tiles) and 4 of record.
#include <algorithm>

#include "common.hpp"
#include "scan.hpp"

namespace gsr {

constexpr uint32_t kOrdFlagAgg = 1u << 30;
constexpr uint32_t kOrdFlagIncl = 2u << 30;
constexpr uint32_t kOrdValueMask = (1u << 30) - 1;
constexpr uint32_t kOrdSpinLimit = 1u << 22;
constexpr int kRecPasses = 4;

__device__ __forceinline__ uint64_t ord_lanes_below() {
  const int lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// The view that owns block `blk` of the record passes (sort_blk) or of the
// emission (seq_blk): the last whose first block is not beyond it.  A view
// without blocks (a follower in the record passes, an empty model) starts
// where the next one does, so the next one is taken.
__device__ __forceinline__ int view_of_rec_block(const ViewD* __restrict__ views, int n_views, uint32_t blk) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].sort_blk <= blk) lo = mid; else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ int view_of_seq_block(const ViewD* __restrict__ views, int n_views, uint32_t blk) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].seq_blk <= blk) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// One digit's exclusive prefix over the blocks before `lb` of a chain whose
// words are st[j * 256 + t]: four predecessors per step (the chain's first
// block is always inclusive, so the walk ends at j >= 0), bounded.
__device__ __forceinline__ uint32_t look_back(const uint32_t* __restrict__ st, int lb, uint32_t t,
                                              uint32_t* __restrict__ err) {
  constexpr int kWin = 4;
  uint32_t excl = 0, spins = 0;
  int j = lb - 1;
  while (j >= 0) {
    uint32_t sv[kWin];
#pragma unroll
    for (int k = 0; k < kWin; ++k)
      sv[k] = j - k >= 0 ? __hip_atomic_load(&st[(size_t)(j - k) * 256 + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                         : 0u;
    int used = 0;
    bool found = false;
#pragma unroll
    for (int k = 0; k < kWin; ++k) {
      if (found || used < k) break;
      const uint32_t f = sv[k] & ~kOrdValueMask;
      if (f == 0) break;
      excl += sv[k] & kOrdValueMask;
      used = k + 1;
      found = f == kOrdFlagIncl;
    }
    if (found) break;
    j -= used;
    if (used == 0) {
      if (++spins > kOrdSpinLimit) {
        atomicOr(err, 1u);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return excl;
}

// ---------------------------------------------------------------- record sort
constexpr int kRecThreads = 512;
constexpr int kRecWaves = kRecThreads / 64;
constexpr int kRecHistItems = 8;
static_assert(kRecThreads * kRecHistItems == (int)kRecTileSmall && kRecThreads * 16 == (int)kRecTile, "records per pass block");

// Digit counts [view][pass][256] of the kept records' keys.  A block takes a
// run of pass blocks and adds its counts once per unit it meets.  The top
// byte (sign and exponent) is nearly constant: a wave whose lanes agree adds
// once.
__device__ __forceinline__ void rec_hist(const ViewD* __restrict__ views, int n_views,
                                         const uint32_t* __restrict__ keys, uint32_t n_blk,
                                         uint32_t* __restrict__ hist, uint32_t blk, uint32_t n_blocks,
                                         uint32_t tile) {
  __shared__ uint32_t lh[kRecPasses * 256];
  const int t = threadIdx.x;
  for (int i = t; i < kRecPasses * 256; i += kRecThreads) lh[i] = 0;
  __syncthreads();
  const uint32_t b0 = (uint32_t)((uint64_t)n_blk * blk / n_blocks);
  const uint32_t b1 = (uint32_t)((uint64_t)n_blk * (blk + 1) / n_blocks);
  int cur = -1;
  auto flush = [&](int v) {
    __syncthreads();
    for (int i = t; i < kRecPasses * 256; i += kRecThreads) {
      const uint32_t c = lh[i];
      if (c) atomicAdd(&hist[(size_t)v * (kRecPasses * 256) + i], c);
      lh[i] = 0;
    }
    __syncthreads();
  };
  for (uint32_t b = b0; b < b1; ++b) {
    const int v = view_of_rec_block(views, n_views, b);
    if (v != cur) {
      if (cur >= 0) flush(cur);
      cur = v;
    }
    const ViewD& V = views[v];
    for (uint32_t sub = 0; sub < tile; sub += kRecTileSmall) {
      const uint32_t base = (b - V.sort_blk) * tile + sub;
      uint32_t k[kRecHistItems];
#pragma unroll
      for (int r = 0; r < kRecHistItems; ++r) {
        const uint32_t i = base + (uint32_t)(r * kRecThreads) + t;
        k[r] = i < V.sort_n ? keys[V.sort_off + i] : kSortCulled;
      }
#pragma unroll
      for (int r = 0; r < kRecHistItems; ++r) {
        const bool ok = k[r] != kSortCulled;
        const uint64_t m = __ballot(ok);
        if (ok) {
#pragma unroll
          for (int q = 0; q < kRecPasses - 1; ++q) atomicAdd(&lh[q * 256 + ((k[r] >> (8 * q)) & 255u)], 1u);
          const uint32_t d = k[r] >> 24, d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
          if (__ballot(d == d0) == m) {
            if ((m & ord_lanes_below()) == 0ull) atomicAdd(&lh[3 * 256 + d0], (uint32_t)__popcll(m));
          } else {
            atomicAdd(&lh[3 * 256 + d], 1u);
          }
        }
      }
    }
  }
  if (cur >= 0) flush(cur);
}

// The scan of the tile counts in record order (the pair count, and where the
// backward keeps each record's partials) and the digit counts in one launch:
// neither needs the other.
template <int ITEMS>
__global__ void __launch_bounds__(kRecThreads)
k_scan_hist(const ViewD* __restrict__ views, int n_views, const uint32_t* __restrict__ keys, uint32_t n_blk,
            uint32_t* __restrict__ hist, uint32_t n_scan, const uint32_t* __restrict__ n_tiles, uint32_t n_rec,
            uint32_t* __restrict__ offsets, uint64_t* __restrict__ status, uint32_t* __restrict__ ticket,
            uint32_t* __restrict__ counters, uint32_t cap, uint32_t rec_tile) {
  if (blockIdx.x < n_scan)
    scan_block<kRecThreads, ITEMS>(n_tiles, n_rec, offsets, status, ticket, counters, cap, n_scan);
  else
    rec_hist(views, n_views, keys, n_blk, hist, blockIdx.x - n_scan, gridDim.x - n_scan, rec_tile);
}

// Units of at most kRecSmall records each: a block sorts one in LDS, in place
// of the digit counts and four passes.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallItems = 8;
static_assert(kSmallThreads * kSmallItems == kRecSmall, "records of a small unit");

__global__ void __launch_bounds__(kSmallThreads)
k_rec_small(const ViewD* __restrict__ views, const uint32_t* __restrict__ keys, uint32_t* __restrict__ keys_out,
            uint32_t* __restrict__ vals_out, uint32_t* __restrict__ unit) {
  __shared__ uint16_t wave_cnt[kSmallWaves][256];
  __shared__ uint32_t s_keys[kRecSmall];
  __shared__ uint16_t s_vals[kRecSmall];
  __shared__ uint32_t s_start[256], s_w[kSmallWaves], s_or[kSmallWaves], s_and[kSmallWaves];
  const ViewD& V = views[blockIdx.x];
  if (V.sort_mode == kSortFollow) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t n = min(V.sort_n, (uint32_t)kRecSmall), off = V.sort_off;
  // wave w takes the I x 64 records from w I x 64 on
  int I = (int)div_up(n, (uint32_t)kSmallThreads);
  uint32_t wbase = (uint32_t)(wave * I * 64 + lane);
  // the kept records, in record order
  uint32_t key[kSmallItems], val[kSmallItems], rank[kSmallItems];
  uint32_t kept = 0, any = 0u, all = 0xFFFFFFFFu;
#pragma unroll
  for (int r = 0; r < kSmallItems; ++r) {
    const uint32_t i = wbase + r * 64;
    key[r] = r < I && i < n ? keys[off + i] : kSortCulled;
  }
#pragma unroll
  for (int r = 0; r < kSmallItems; ++r) {
    const bool ok = key[r] != kSortCulled;
    const uint64_t m = __ballot(ok);
    rank[r] = kept + (uint32_t)__popcll(m & ord_lanes_below());
    kept += (uint32_t)__popcll(m);
    any |= ok ? key[r] : 0u;
    all &= ok ? key[r] : 0xFFFFFFFFu;
  }
  any = wave_or(any);
  all = ~wave_or(~all);
  if (lane == 0) {
    s_w[wave] = kept;
    s_or[wave] = any;
    s_and[wave] = all;
  }
  __syncthreads();
  uint32_t K = 0, w0 = 0;
#pragma unroll
  for (int w = 0; w < kSmallWaves; ++w) {
    if (w < wave) w0 += s_w[w];
    K += s_w[w];
    any |= s_or[w];
    all &= s_and[w];
  }
  const uint32_t differ = any & ~all;  // a byte the keys agree on needs no pass
#pragma unroll
  for (int r = 0; r < kSmallItems; ++r)
    if (key[r] != kSortCulled) {
      s_keys[w0 + rank[r]] = key[r];
      s_vals[w0 + rank[r]] = (uint16_t)(wbase + r * 64);
    }
  I = (int)div_up(K, (uint32_t)kSmallThreads);
  wbase = (uint32_t)(wave * I * 64 + lane);
  for (int pass = 0; pass < kRecPasses; ++pass) {
    if (((differ >> (8 * pass)) & 255u) == 0u) continue;
    for (int i = t; i < kSmallWaves * 256 / 2; i += kSmallThreads)
      reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r) {
      if (r >= I) break;
      const uint32_t i = wbase + r * 64;
      const bool ok = i < K;
      key[r] = ok ? s_keys[i] : 0u;
      val[r] = ok ? s_vals[i] : 0u;
      const uint32_t d = (key[r] >> (8 * pass)) & 255u;
      const uint64_t peers = match_digit<8>(d, ok);
      const uint64_t front = peers & ord_lanes_below();
      uint32_t pre = 0;
      if (ok) pre = wave_cnt[wave][d];
      __builtin_amdgcn_wave_barrier();
      if (ok && front == 0) wave_cnt[wave][d] = (uint16_t)(pre + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
      rank[r] = pre + (uint32_t)__popcll(front);
    }
    __syncthreads();
    uint32_t cnt = 0, inc = 0;
    if (t < 256) {
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        const uint32_t c = wave_cnt[w][t];
        wave_cnt[w][t] = (uint16_t)cnt;
        cnt += c;
      }
      inc = wave_scan_add(cnt);
      if (lane == 63) s_w[wave] = inc;
    }
    __syncthreads();
    if (t < 256) {
      uint32_t o = inc - cnt;
      for (int w = 0; w < wave; ++w) o += s_w[w];
      s_start[t] = o;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallItems; ++r)
      if (r < I && wbase + r * 64 < K) {
        const uint32_t d = (key[r] >> (8 * pass)) & 255u;
        const uint32_t pos = s_start[d] + wave_cnt[wave][d] + rank[r];
        s_keys[pos] = key[r];
        s_vals[pos] = (uint16_t)val[r];
      }
    __syncthreads();
  }
  __syncthreads();
  const uint32_t rec0 = V.rec_off;
  for (uint32_t i = t; i < K; i += kSmallThreads) {
    keys_out[off + i] = s_keys[i];
    vals_out[off + i] = rec0 + s_vals[i];
  }
  if (t == 0) {
    unit[2 * blockIdx.x] = K;
    unit[2 * blockIdx.x + 1] = 1u;  // the second buffers
  }
}

// One stable pass.  The first reads every slot of the unit in record order,
// drops the culled ones and always moves; a later pass whose digit is the
// same for the whole unit is skipped (one that is the same for every unit
// before it takes a ticket; *needed: the others).  unit[2 v], unit[2 v + 1]:
// the unit's kept records and the buffer that holds them after the last pass.
template <bool FIRST, int kRecItems>
__global__ void __launch_bounds__(kRecThreads, 4)
k_rec_pass(const ViewD* __restrict__ views, int n_views, uint32_t* __restrict__ keys0, uint32_t* __restrict__ keys1,
           uint32_t* __restrict__ vals0, uint32_t* __restrict__ vals1, const uint32_t* __restrict__ hist,
           uint32_t* __restrict__ status, uint32_t* __restrict__ ticket, uint32_t* __restrict__ unit,
           uint32_t* __restrict__ needed, uint32_t* __restrict__ err, int pass) {
  constexpr uint32_t kTileRec = kRecThreads * kRecItems;
  __shared__ uint32_t s_bid, s_triv;
  __shared__ uint16_t wave_cnt[kRecWaves][256];
  __shared__ uint32_t s_global[256];
  __shared__ uint32_t s_w[4], s_hw[4];
  __shared__ uint32_t s_keys[kTileRec], s_vals[kTileRec];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (!FIRST && ((*needed >> pass) & 1u) == 0u) return;  // every unit agrees on this byte
  if (t == 0) {
    s_bid = atomicAdd(ticket, 1u);
    s_triv = 0;
  }
  for (int i = t; i < kRecWaves * 256 / 2; i += kRecThreads) reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[i] = 0;
  __syncthreads();
  const uint32_t gblk = s_bid;
  const int v = view_of_rec_block(views, n_views, gblk);
  const uint32_t off = views[v].sort_off, lb = gblk - views[v].sort_blk;
  uint32_t hv[kRecPasses], hc = 0, hinc = 0;
  if (t < 256) {
#pragma unroll
    for (int q = 0; q < kRecPasses; ++q) hv[q] = hist[(size_t)v * (kRecPasses * 256) + q * 256 + t];
#pragma unroll
    for (int q = 0; q < kRecPasses; ++q)
      if (q == pass) hc = hv[q];
    hinc = wave_scan_add(hc);
    if (lane == 63) s_hw[wave] = hinc;
  }
  __syncthreads();
  const uint32_t K = s_hw[0] + s_hw[1] + s_hw[2] + s_hw[3];
  if (t < 256) {
#pragma unroll
    for (int q = 1; q < kRecPasses; ++q)
      if (hv[q] == K) atomicOr(&s_triv, 1u << q);
  }
  __syncthreads();
  const uint32_t triv = s_triv, moves = ((1u << kRecPasses) - 1u) & ~triv;
  if (FIRST && lb == 0 && t == 0) {
    unit[2 * v] = K;
    unit[2 * v + 1] = (uint32_t)__popc(moves) & 1u;
    atomicOr(needed, moves);
  }
  if (!FIRST && ((triv >> pass) & 1u)) return;
  const uint32_t moved = (uint32_t)__popc(moves & ((1u << pass) - 1u));
  const uint32_t n_in = FIRST ? views[v].sort_n : K;
  const uint32_t base = lb * kTileRec;
  if (base >= n_in) return;
  const bool src = !FIRST && (moved & 1u);
  const uint32_t* kin = (src ? keys1 : keys0) + off;
  const uint32_t* vin = (src ? vals1 : vals0) + off;
  uint32_t* kout = (src ? keys0 : keys1) + off;
  uint32_t* vout = (src ? vals0 : vals1) + off;
  const uint32_t rec0 = views[v].rec_off;
  const int shift = 8 * pass;
  uint32_t key[kRecItems], val[kRecItems], rank[kRecItems];
  bool ok[kRecItems];
  const uint32_t wbase = base + (uint32_t)wave * (kRecItems * 64);
#pragma unroll
  for (int r = 0; r < kRecItems; ++r) {
    const uint32_t i = wbase + r * 64 + lane;
    ok[r] = i < n_in;
    key[r] = ok[r] ? kin[i] : 0u;
    if (FIRST) {
      ok[r] = ok[r] && key[r] != kSortCulled;
      val[r] = rec0 + i;
    } else {
      val[r] = ok[r] ? vin[i] : 0u;
    }
  }
  // rank within the wave, in input order (round-major, then lane)
#pragma unroll
  for (int r = 0; r < kRecItems; ++r) {
    const uint32_t d = (key[r] >> shift) & 255u;
    const uint64_t peers = match_digit<8>(d, ok[r]);
    const uint64_t front = peers & ord_lanes_below();
    uint32_t pre = 0;
    if (ok[r]) pre = wave_cnt[wave][d];
    __builtin_amdgcn_wave_barrier();
    if (ok[r] && front == 0) wave_cnt[wave][d] = (uint16_t)(pre + (uint32_t)__popcll(peers));
    __builtin_amdgcn_wave_barrier();
    rank[r] = pre + (uint32_t)__popcll(front);
  }
  __syncthreads();
  // thread t < 256 owns digit t: the block count, look-back, wave offsets
  uint32_t* st = status + (size_t)views[v].sort_blk * 256;
  uint32_t cnt = 0, inc = 0, cw[kRecWaves];
  if (t < 256) {
#pragma unroll
    for (int w = 0; w < kRecWaves; ++w) cw[w] = wave_cnt[w][t];
#pragma unroll
    for (int w = 0; w < kRecWaves; ++w) cnt += cw[w];
    inc = wave_scan_add(cnt);
    if (lane == 63) s_w[wave] = inc;
    __hip_atomic_store(&st[(size_t)lb * 256 + t], (lb == 0 ? kOrdFlagIncl : kOrdFlagAgg) | cnt, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (t < 256) {
    uint32_t o = inc - cnt, doff = hinc - hc;
    for (int w = 0; w < wave; ++w) {
      o += s_w[w];
      doff += s_hw[w];
    }
    uint32_t excl = 0;
    if (lb > 0) {
      excl = look_back(st, (int)lb, (uint32_t)t, err);
      __hip_atomic_store(&st[(size_t)lb * 256 + t], kOrdFlagIncl | ((excl + cnt) & kOrdValueMask), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    s_global[t] = doff + excl - o;  // of an item at LDS position p: p + s_global
#pragma unroll
    for (int w = 0; w < kRecWaves; ++w) {
      wave_cnt[w][t] = (uint16_t)o;
      o += cw[w];
    }
  }
  __syncthreads();
  const uint32_t n_items = s_w[0] + s_w[1] + s_w[2] + s_w[3];
  // order the block's records by digit in LDS (stable), then write digit runs
#pragma unroll
  for (int r = 0; r < kRecItems; ++r)
    if (ok[r]) {
      const uint32_t pos = wave_cnt[wave][(key[r] >> shift) & 255u] + rank[r];
      s_keys[pos] = key[r];
      s_vals[pos] = val[r];
    }
  __syncthreads();
  for (uint32_t i = t; i < n_items; i += kRecThreads) {
    const uint32_t k = s_keys[i];
    const uint32_t dst = s_global[(k >> shift) & 255u] + i;
    if (dst < K) {
      kout[dst] = k;
      vout[dst] = s_vals[i];
    } else {
      atomicOr(err, 2u);  // inconsistent offsets: never write out of range
    }
  }
}

// ---------------------------------------------------------------- emission
// A block takes 1024 or 4096 positions of a view's sorted records, by a
// ticket.  A wave loads the boxes of its share, scans their tile counts, and
// the block finds where its pairs start by look-back; then every
// wave writes its pairs, 64 at a time with its lanes on consecutive pairs,
// so the writes are coalesced and a large splat spreads over the wave.  The
// owner of each pair: the records starting among the 64 leave their lane at
// their first pair, a running maximum over the lanes carries it on.  Bound by
// the gather of the boxes in depth order: with eight bytes each 770 us on 162M
// pairs of 32M records (410 with the gather at consecutive addresses), with
// four 714; on 12.5M pairs of 1.1M records 57.6 and 55.9.
constexpr int kEmitThreads = 1024;
constexpr int kEmitWaves = kEmitThreads / 64;
constexpr uint64_t kEmAgg = 1ull << 62;
constexpr uint64_t kEmIncl = 2ull << 62;
constexpr uint64_t kEmValue = (1ull << 62) - 1;

// Inclusive running maximum over the wave.
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
  return x;
}

// Orders a wave's own LDS accesses (they execute in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename TT, int ROUNDS>
__global__ void __launch_bounds__(kEmitThreads)
k_emit(const ViewD* __restrict__ views, int n_views, const uint32_t* __restrict__ vals0,
       const uint32_t* __restrict__ vals1, const uint32_t* __restrict__ unit, const uint32_t* __restrict__ boxes, bool box4,
       uint32_t* __restrict__ counters, uint32_t cap, TT* __restrict__ tiles, uint32_t* __restrict__ recs,
       uint64_t* __restrict__ status, uint32_t* __restrict__ ticket) {
  __shared__ uint32_t s_bid;
  __shared__ uint64_t s_excl, s_w[kEmitWaves];  // (a block's 4096 records of 2^20 tiles each pass 2^32)
  // of a wave's records: first pair among its 64's, first tile less that, box width, record
  __shared__ uint4 s_rec[kEmitWaves][ROUNDS * 64];
  __shared__ uint32_t s_mark[kEmitWaves][64];  // 1 + the index of the record that starts at each of 64 pairs
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  s_mark[wave][lane] = 0u;
  const uint32_t lim = min(cap, counters[kCntPairs]);
  if (t == 0) s_bid = atomicAdd(ticket, 1u);
  __syncthreads();
  const uint32_t bid = s_bid;
  const int v = view_of_seq_block(views, n_views, bid);
  const ViewD& V = views[v];
  const int lead = V.sort_mode == kSortFollow ? min((int)V.sort_lead, n_views - 1) : v;
  const uint32_t n_seq = min(unit[2 * lead], views[lead].sort_n);
  const uint32_t* vals = (unit[2 * lead + 1] ? vals1 : vals0) + views[lead].sort_off;
  const uint32_t rec_lead = views[lead].rec_off, rec0 = V.rec_off, n_rec = views[lead].sort_n;
  const uint32_t p0 = (bid - V.seq_blk) * (uint32_t)(kEmitThreads * ROUNDS) + (uint32_t)wave * (ROUNDS * 64) + lane;
  uint32_t rec[ROUNDS], off[ROUNDS], tot[ROUNDS];
  uint2 bx[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t p = p0 + r * 64;
    rec[r] = p < n_seq ? vals[p] - rec_lead : 0xFFFFFFFEu;  // the Gaussian
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (rec[r] < n_rec) {
      rec[r] += rec0;
    } else {  // past the end, or an inconsistent order (its pairs are dropped)
      if (rec[r] != 0xFFFFFFFEu) atomicOr(&counters[kCntError], 64u);
      rec[r] = 0xFFFFFFFFu;
    }
  }
  if (box4) {  // (uniform; apart, so that a thread's loads are in flight together)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) bx[r] = rec[r] != 0xFFFFFFFFu ? load_box(boxes, rec[r], true) : make_uint2(0u, 0u);
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) bx[r] = rec[r] != 0xFFFFFFFFu ? load_box(boxes, rec[r], false) : make_uint2(0u, 0u);
  }
  const uint32_t tx = (uint32_t)V.tiles_x, toff = V.tile_off;
  uint64_t sum = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t nt = (bx[r].y & 0xFFFFu) * (bx[r].y >> 16);
    const uint32_t inc = wave_scan_add(nt);
    off[r] = nt ? inc - nt : 0xFFFFFFFFu;  // (never in a window)
    s_rec[wave][r * 64 + lane] = make_uint4(inc - nt, toff + (bx[r].x >> 16) * tx + (bx[r].x & 0xFFFFu) - (inc - nt),
                                              max(bx[r].y & 0xFFFFu, 1u), rec[r]);
    tot[r] = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    sum += tot[r];
  }
  if (lane == 0) s_w[wave] = sum;
  __syncthreads();
  if (wave == 0) {
    uint64_t total = 0;
#pragma unroll
    for (int w = 0; w < kEmitWaves; ++w) total += s_w[w];
    if (lane == 0)
      __hip_atomic_store(&status[bid], (bid == 0 ? kEmIncl : kEmAgg) | total, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    uint64_t excl = 0;
    if (bid > 0) {
      int j = (int)bid - 1;  // window [j - 63, j]
      uint32_t spins = 0;
      for (;;) {
        const int idx = j - lane;
        const uint64_t sv =
            idx >= 0 ? __hip_atomic_load(&status[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kEmIncl;
        const uint64_t flag = sv & ~kEmValue;
        const uint64_t ready = __ballot(flag != 0);
        const uint64_t incl = __ballot(flag == kEmIncl);
        const int first = incl ? __builtin_ctzll(incl) : 64;
        const uint64_t need = first < 63 ? ((2ull << first) - 1) : ~0ull;
        if ((ready & need) != need) {
          if (++spins > kOrdSpinLimit) {
            if (lane == 0) atomicOr(&counters[kCntError], 16u);
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        uint64_t x = (lane <= first && idx >= 0) ? (sv & kEmValue) : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        excl += x;
        if (first < 64) break;
        j -= 64;
      }
      if (lane == 0)
        __hip_atomic_store(&status[bid], kEmIncl | ((excl + total) & kEmValue), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) s_excl = excl;
  }
  __syncthreads();
  uint64_t w64 = s_excl;
  for (int w = 0; w < wave; ++w) w64 += s_w[w];
  // pairs at or beyond the limit are dropped
  uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)min(w64, (uint64_t)lim));
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t n_r = min(tot[r], lim - w0);
    // indices grow over the pairs, so a mark left by earlier pairs is at most
    // the running maximum and needs no clearing
    uint32_t carry = (uint32_t)(r * 64);
    for (uint32_t b = 0; b < n_r; b += 64) {
      const uint32_t e = b + (uint32_t)lane;
      if (off[r] - b < 64u) s_mark[wave][off[r] - b] = (uint32_t)(r * 64 + lane) + 1u;
      wave_lds_fence();
      const uint32_t m = max(wave_scan_max(s_mark[wave][lane]), carry);
      carry = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
      const uint4 own = s_rec[wave][max(m, 1u) - 1u];
      wave_lds_fence();
      if (e < n_r) {
        const uint32_t j = e - own.x;
        // row j / w of the box: with half a step added, the float quotient's
        // error (below 2^-22) cannot reach the next integer for j < 2^20
        uint32_t dy = (uint32_t)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)own.z));
        if (j >= (1u << 20)) dy = j / own.z;
        tiles[w0 + e] = (TT)(own.y + e + __umul24(dy, tx - own.z));
        recs[w0 + e] = own.w;
      }
    }
    w0 += n_r;
  }
}

// ---------------------------------------------------------------- tile grouping
// One stable pass is three launches with nothing to wait for inside them:
// each of the (about 512) blocks counts the digits of its contiguous share of
// the pairs, a scan turns the counts into where each block's items of each
// digit go, and every block then walks its share 512 ITEMS pairs at a time,
// ranks them in LDS and writes digit runs at its running positions.  16 items
// a thread keep the runs long; with few pairs, 4 spread them over more blocks.  (A
// single launch per pass with decoupled look-back took 83 us on 12.5M pairs
// and 773 on 162M, growing with the number of blocks: the chain of 256
// digits' prefixes, not memory, bounded it; count, scan and scatter take
// 7 + 8 + 43 and 99 + 8 + 541.)
constexpr int kPairThreads = 512;
constexpr int kPairWaves = kPairThreads / 64;

// Words of a block's counts: the digits of a pass of `bits` bits, 256 at least.
constexpr uint32_t digit_stride(int bits) { return bits > 8 ? 1u << bits : 256u; }
static_assert(digit_stride(kPairBits) <= (uint32_t)kPairThreads, "a thread owns at most one digit");

// Block b's share of K pairs: whole steps.
__device__ __forceinline__ void pair_share(uint32_t K, uint32_t b, uint32_t g, uint32_t step, uint32_t& begin,
                                           uint32_t& end) {
  const uint32_t per = div_up(div_up(K, step), g) * step;
  begin = (uint32_t)min((uint64_t)K, (uint64_t)b * per);
  end = (uint32_t)min((uint64_t)K, (uint64_t)begin + per);
}

// counts[block][S] of the digit at `shift` of the block's share.
template <typename TT, uint32_t S>
__global__ void __launch_bounds__(kPairThreads)
k_pair_count(const TT* __restrict__ tiles, const uint32_t* __restrict__ counters, uint32_t cap, uint32_t step,
             int shift, uint32_t mask, uint32_t* __restrict__ counts) {
  // eight counters per digit, by lane: the second pass meets runs of few
  // digits (one view's tile rows), whose additions would queue on one word
  constexpr uint32_t kRep = 8;
  __shared__ uint32_t lh[S * kRep];
  const int t = threadIdx.x;
  for (int i = t; i < (int)(S * kRep); i += kPairThreads) lh[i] = 0;
  __syncthreads();
  const uint32_t rep = (uint32_t)t % kRep;
  const uint32_t K = min(counters[kCntPairs], cap);
  uint32_t begin, end;
  pair_share(K, blockIdx.x, gridDim.x, step, begin, end);
  // lanes take consecutive pairs: in emission order their tiles are
  // consecutive too, and the additions fall in different banks
  constexpr uint32_t kAhead = 8;  // loads in flight per thread
  uint32_t k = begin + (uint32_t)t;
  for (; (uint64_t)k + (kAhead - 1) * kPairThreads < end; k += kAhead * kPairThreads) {
    TT q[kAhead];
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) q[u] = tiles[k + u * kPairThreads];
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) atomicAdd(&lh[(((uint32_t)q[u] >> shift) & mask) * kRep + rep], 1u);
  }
  for (; k < end; k += kPairThreads) atomicAdd(&lh[(((uint32_t)tiles[k] >> shift) & mask) * kRep + rep], 1u);
  __syncthreads();
  if (t < (int)S) {
    uint32_t c = 0;
#pragma unroll
    for (uint32_t r = 0; r < kRep; ++r) c += lh[t * kRep + r];
    counts[(size_t)blockIdx.x * S + t] = c;
  }
}

// counts[b][d] becomes the count of digit d in the blocks before b, total[d]
// the digit's count.  A block takes four digits, 256 threads per digit split
// the g blocks.
template <uint32_t S>
__global__ void __launch_bounds__(1024)
k_pair_scan(uint32_t* __restrict__ counts, uint32_t g, uint32_t* __restrict__ total) {
  __shared__ uint32_t s_w[16];
  const uint32_t t = threadIdx.x, d = blockIdx.x * 4u + (t >> 8), q = t & 255u;
  const int lane = t & 63, wave = t >> 6;
  const uint32_t per = div_up(g, 256u), b0 = min(g, q * per), b1 = min(g, b0 + per);
  uint32_t sum = 0;
  for (uint32_t b = b0; b < b1; ++b) sum += counts[(size_t)b * S + d];
  const uint32_t inc = wave_scan_add(sum);
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  uint32_t run = inc - sum, all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t c = s_w[(wave & ~3) + w];
    if (w < (wave & 3)) run += c;
    all += c;
  }
  for (uint32_t b = b0; b < b1; ++b) {
    const uint32_t c = counts[(size_t)b * S + d];
    counts[(size_t)b * S + d] = run;
    run += c;
  }
  if (q == 0) total[d] = all;
}

// The scatter: the digit at `shift` (`mask`: at most BITS bits).  total null:
// the counts of the (at most kScanInline) blocks are as counted, and each
// block adds up those before it by itself, which on few pairs costs less
// than the scan's launch.
constexpr uint32_t kScanInline = 64;

template <typename TT, int BITS, int kPairItems>
__global__ void __launch_bounds__(kPairThreads, 4)
k_pair_pass(const TT* __restrict__ tin, TT* __restrict__ tout, const uint32_t* __restrict__ rin,
            uint32_t* __restrict__ rout, const uint32_t* __restrict__ counters, uint32_t cap,
            const uint32_t* __restrict__ before, const uint32_t* __restrict__ total, int shift, uint32_t mask,
            uint32_t* __restrict__ sel_out, uint32_t sel, uint32_t* __restrict__ err) {
  constexpr uint32_t D = 1u << BITS, S = digit_stride(BITS), kStep = kPairThreads * kPairItems;
  __shared__ uint16_t wave_cnt[kPairWaves][D];
  __shared__ uint32_t s_global[D];
  __shared__ uint32_t s_w[S / 64];
  __shared__ TT s_tile[kStep];
  __shared__ uint32_t s_rec[kStep];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (sel_out && blockIdx.x == 0 && t == 0) *sel_out = sel;
  const uint32_t K = min(counters[kCntPairs], cap);
  uint32_t begin, end;
  pair_share(K, blockIdx.x, gridDim.x, kStep, begin, end);
  if (begin >= end) return;
  // thread t < D: where the block's next item of digit t goes
  uint32_t next = 0;
  {
    uint32_t c = 0, inc = 0, bef = 0;
    if (t < (int)S) {
      if (total) {
        c = total[t];
        bef = before[(size_t)blockIdx.x * S + t];
      } else {
        for (uint32_t b = 0; b < gridDim.x; b += 8) {
          uint32_t x[8];
#pragma unroll
          for (uint32_t u = 0; u < 8; ++u) x[u] = b + u < gridDim.x ? before[(size_t)(b + u) * S + t] : 0u;
#pragma unroll
          for (uint32_t u = 0; u < 8; ++u) {
            c += x[u];
            bef += b + u < blockIdx.x ? x[u] : 0u;
          }
        }
      }
      inc = wave_scan_add(c);
      if (lane == 63) s_w[wave] = inc;
    }
    __syncthreads();
    if (t < (int)S) {
      next = inc - c + bef;
      for (int w = 0; w < wave; ++w) next += s_w[w];
    }
  }
  // a pair's tile, and above it (2-byte tiles) or beside it its rank
  uint32_t til[kPairItems], rec[kPairItems], rnk[sizeof(TT) == 2 ? 1 : kPairItems];
  const uint32_t wbase = (uint32_t)wave * (kPairItems * 64) + (uint32_t)lane;
  for (uint32_t base = begin; base < end; base += kStep) {
#pragma unroll
    for (int r = 0; r < kPairItems; ++r) {
      const uint32_t i = min(base + wbase + r * 64, end - 1u);  // (branch-free)
      til[r] = (uint32_t)tin[i];
      rec[r] = rin[i];
    }
    for (int i = t; i < (int)(kPairWaves * D / 2); i += kPairThreads)
      reinterpret_cast<uint32_t*>(&wave_cnt[0][0])[i] = 0;
    __syncthreads();  // (and the previous step's LDS is read)
#pragma unroll
    for (int r = 0; r < kPairItems; ++r) {
      const bool ok = base + wbase + r * 64 < end;
      const uint32_t d = (til[r] >> shift) & mask;
      const uint64_t peers = match_digit<BITS>(d, ok);
      const uint64_t front = peers & ord_lanes_below();
      uint32_t pre = 0;
      if (ok) pre = wave_cnt[wave][d];
      __builtin_amdgcn_wave_barrier();
      if (ok && front == 0) wave_cnt[wave][d] = (uint16_t)(pre + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
      const uint32_t rank = pre + (uint32_t)__popcll(front);
      if constexpr (sizeof(TT) == 2) til[r] |= rank << 16;
      else rnk[r] = rank;
    }
    __syncthreads();
    // thread t < D: digit t's place in the block, wave by wave
    uint32_t cw[kPairWaves], cnt = 0, inc = 0;
    if (t < (int)S) {
      if (t < (int)D) {
#pragma unroll
        for (int w = 0; w < kPairWaves; ++w) cw[w] = wave_cnt[w][t];
#pragma unroll
        for (int w = 0; w < kPairWaves; ++w) cnt += cw[w];
      }
      inc = wave_scan_add(cnt);
      if (lane == 63) s_w[wave] = inc;
    }
    __syncthreads();
    if (t < (int)D) {
      uint32_t o = inc - cnt;
      for (int w = 0; w < wave; ++w) o += s_w[w];
      s_global[t] = next - o;  // of an item at LDS position p: p + s_global
      next += cnt;
#pragma unroll
      for (int w = 0; w < kPairWaves; ++w) {
        wave_cnt[w][t] = (uint16_t)o;
        o += cw[w];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPairItems; ++r)
      if (base + wbase + r * 64 < end) {
        const uint32_t tile = sizeof(TT) == 2 ? til[r] & 0xFFFFu : til[r];
        const uint32_t rank = sizeof(TT) == 2 ? til[r] >> 16 : rnk[sizeof(TT) == 2 ? 0 : r];
        const uint32_t pos = wave_cnt[wave][(tile >> shift) & mask] + rank;
        s_tile[pos] = (TT)tile;
        s_rec[pos] = rec[r];
      }
    __syncthreads();
    const uint32_t n_items = min(end - base, kStep);
    for (uint32_t i = t; i < n_items; i += kPairThreads) {
      const uint32_t tile = s_tile[i];
      const uint32_t dst = s_global[(tile >> shift) & mask] + i;
      if (dst < K) {
        tout[dst] = (TT)tile;
        rout[dst] = s_rec[i];
      } else {
        atomicOr(err, 2u);  // inconsistent counts: never write out of range
      }
    }
  }
}

// The tiles' runs in the grouped pairs (ranges zero on entry).  A block takes
// a contiguous share; a thread takes 16 bytes of tiles at a time, four such
// loads in flight, and writes the run ends it sees - none where the last
// pair's tile is that of the pair before the first, the tiles ascending.
template <typename TT>
__global__ void __launch_bounds__(256)
k_tile_runs(const TT* __restrict__ tiles, uint32_t* __restrict__ counters, uint32_t cap, uint32_t n_tiles,
            uint32_t* __restrict__ ranges) {
  constexpr uint32_t kItems = 16 / sizeof(TT), kAhead = 4, kRow = 256 * kItems;
  const uint32_t K = min(counters[kCntPairs], cap);
  const uint64_t share = ((uint64_t)div_up(K, gridDim.x) + kRow * kAhead - 1) / (kRow * kAhead) * (kRow * kAhead);
  const uint64_t begin = blockIdx.x * share, end = min((uint64_t)K, begin + share);
  auto boundary = [&](uint32_t prev, uint32_t tile, uint32_t k) {
    if (tile < n_tiles) ranges[2 * (size_t)tile] = k;
    else atomicOr(&counters[kCntError], 4u);
    if (prev < n_tiles) ranges[2 * (size_t)prev + 1] = k;
  };
  auto item = [](const uint4& q, uint32_t u) -> uint32_t {
    const uint32_t w = sizeof(TT) == 2 ? (u >> 1) : u;
    const uint32_t x = w == 0 ? q.x : w == 1 ? q.y : w == 2 ? q.z : q.w;
    return sizeof(TT) == 2 ? (x >> (16 * (u & 1))) & 0xFFFFu : x;
  };
  uint64_t base = begin;
  for (; base + kRow * kAhead <= end; base += kRow * kAhead) {
    uint4 q[kAhead];
    uint32_t prev[kAhead];
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
      const uint64_t k0 = base + u * kRow + threadIdx.x * kItems;
      q[u] = *reinterpret_cast<const uint4*>(tiles + k0);
      prev[u] = k0 ? (uint32_t)tiles[k0 - 1] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
      if (item(q[u], kItems - 1) == prev[u]) continue;
      const uint32_t k0 = (uint32_t)(base + u * kRow + threadIdx.x * kItems);
      uint32_t p = prev[u];
#pragma unroll
      for (uint32_t x = 0; x < kItems; ++x) {
        const uint32_t tile = item(q[u], x);
        if (tile != p) boundary(p, tile, k0 + x);
        p = tile;
      }
    }
  }
  for (uint64_t k = base + threadIdx.x; k < end; k += 256) {
    const uint32_t tile = tiles[k], p = k ? (uint32_t)tiles[k - 1] : 0xFFFFFFFFu;
    if (tile != p) boundary(p, tile, (uint32_t)k);
  }
  if (end == K && begin < end && threadIdx.x == 0) {  // the last run's end
    const uint32_t tile = tiles[K - 1];
    if (tile < n_tiles) ranges[2 * (size_t)tile + 1] = K;
  }
}

int device_cus();

namespace {
template <typename TT, int BITS, int ITEMS>
void pair_pass_bits(uint32_t g, const TT* tin, TT* tout, const uint32_t* rin, uint32_t* rout, const OrderBufs& o,
                    int shift, uint32_t mask, uint32_t* sel_out, uint32_t sel, hipStream_t s) {
  constexpr uint32_t S = digit_stride(BITS);
  hipLaunchKernelGGL((k_pair_count<TT, S>), dim3(g), dim3(kPairThreads), 0, s, tin, o.counters, o.cap,
                     (uint32_t)(kPairThreads * ITEMS), shift, mask, o.pair_counts);
  uint32_t* total = g > kScanInline ? o.pair_counts + (size_t)S * g : nullptr;
  if (total) hipLaunchKernelGGL(k_pair_scan<S>, dim3(S / 4), dim3(1024), 0, s, o.pair_counts, g, total);
  hipLaunchKernelGGL((k_pair_pass<TT, BITS, ITEMS>), dim3(g), dim3(kPairThreads), 0, s, tin, tout, rin, rout,
                     o.counters, o.cap, o.pair_counts, total, shift, mask, sel_out, sel, o.counters + kCntError);
}

template <typename TT, int ITEMS>
void pair_pass(int bits, uint32_t g, const TT* tin, TT* tout, const uint32_t* rin, uint32_t* rout,
               const OrderBufs& o, int shift, uint32_t* sel_out, uint32_t sel, hipStream_t s) {
  const uint32_t mask = (1u << bits) - 1u;
  const auto pass = bits <= 6   ? pair_pass_bits<TT, 6, ITEMS>
                    : bits == 7 ? pair_pass_bits<TT, 7, ITEMS>
                    : bits == 8 ? pair_pass_bits<TT, 8, ITEMS>
                                : pair_pass_bits<TT, sizeof(TT) == 2 ? 8 : kPairBits, ITEMS>;
  pass(g, tin, tout, rin, rout, o, shift, mask, sel_out, sel, s);
}

template <typename TT>
hipError_t order_pairs(const OrderBufs& o, hipStream_t s) {
  const uint32_t g = pair_pass_blocks(o.cap);
  int bits, np;
  tile_passes(o.n_tiles, &bits, &np);
  TT* tiles[2] = {reinterpret_cast<TT*>(o.tile_a), reinterpret_cast<TT*>(o.tile_b)};
  uint32_t* recs[2] = {o.rec_a, o.rec_b};
  const auto emit = o.seq_tile == kEmitTile ? k_emit<TT, (int)kEmitTile / kEmitThreads>
                                            : k_emit<TT, (int)kEmitTileSmall / kEmitThreads>;
  hipLaunchKernelGGL(emit, dim3(o.seq_blocks), dim3(kEmitThreads), 0, s, o.views, o.n_views, o.vals_a,
                     o.vals_b, o.unit, o.boxes, o.box4, o.counters, o.cap, tiles[0], recs[0], o.emit_status, &o.tickets[4]);
  const auto pass = pair_step(o.cap) == kPairStep ? pair_pass<TT, (int)kPairStep / kPairThreads>
                                                  : pair_pass<TT, (int)kPairStepSmall / kPairThreads>;
  for (int p = 0; p < np; ++p)
    pass(bits, g, tiles[p & 1], tiles[(p + 1) & 1], recs[p & 1], recs[(p + 1) & 1], o, p * bits,
                  p == np - 1 ? o.sel : nullptr, (uint32_t)(np & 1), s);
  const uint32_t rg = std::min(div_up(o.cap, 256u * 8u * 4u), 2048u);
  hipLaunchKernelGGL(k_tile_runs<TT>, dim3(std::max(rg, 1u)), dim3(256), 0, s, tiles[np & 1], o.counters, o.cap,
                     o.n_tiles, o.ranges);
  return hipGetLastError();
}
}  // namespace

// Digits of the tile grouping: np passes of `bits` bits each (the last may
// see fewer).  Nine bits where they save a pass: 44M pairs of 70560 tiles took
// 3 x (168 us + 49 of counting) with six, 2 x (221 + 51) with nine.
void tile_passes(uint32_t n_tiles, int* bits, int* np) {
  int b = 1;
  while (b < 32 && (1ull << b) < n_tiles) ++b;
  *np = b <= 2 * kPairBits ? (b + 7) / 8 - (b > 16) : (b + 7) / 8;
  *bits = (b + *np - 1) / *np;
}

// Blocks of a tile-digit pass: two per compute unit, at most one per step.
uint32_t pair_pass_blocks(uint32_t cap) {
  return std::min(div_up(cap > 0 ? cap : 1u, pair_step(cap)), kPairBlocks);
}

// The scan of the tile counts (offsets, the pair count) with the record
// sort's digit counts.  Small units need no counts.
hipError_t launch_order_scan(const OrderBufs& o, const uint32_t* n_tiles, uint32_t* offsets, uint64_t* scan_status,
                             uint32_t* scan_ticket, uint32_t n_rec, hipStream_t s) {
  // (the scan's blocks look back along a chain: few long ones above 4M
  // records, 166 -> 135 us at 32M with the digit counts beside it)
  const bool big = n_rec > (1u << 22);
  const uint32_t n_scan = div_up(n_rec + 1, (uint32_t)kRecThreads * (big ? 64u : (uint32_t)kScanItems));
  const uint32_t n_hist = o.small ? 0u : std::min(o.rec_blocks, 2u * (uint32_t)device_cus());
  hipLaunchKernelGGL(big ? k_scan_hist<64> : k_scan_hist<kScanItems>, dim3(n_scan + n_hist), dim3(kRecThreads), 0, s,
                     o.views, o.n_views, o.keys_a, o.rec_blocks, o.rec_hist, n_scan, n_tiles, n_rec, offsets,
                     scan_status, scan_ticket, o.counters, o.cap, o.rec_tile);
  return hipGetLastError();
}

// Records and pairs of every view in order, after launch_order_scan; the
// look-back words, tickets, counts and unit words are zero on entry.
hipError_t launch_order(const OrderBufs& o, hipStream_t s) {
  if (o.small) {
    hipLaunchKernelGGL(k_rec_small, dim3(o.n_views), dim3(kSmallThreads), 0, s, o.views, o.keys_a, o.keys_b, o.vals_b,
                       o.unit);
  } else if (o.rec_blocks > 0) {
    uint32_t* err = o.counters + kCntError;
    for (int p = 0; p < kRecPasses; ++p) {
      uint32_t* st = o.rec_status + (size_t)p * o.rec_blocks * 256;
      const bool big = o.rec_tile == kRecTile;
      const auto pass = p == 0 ? (big ? k_rec_pass<true, 16> : k_rec_pass<true, 8>)
                               : (big ? k_rec_pass<false, 16> : k_rec_pass<false, 8>);
      hipLaunchKernelGGL(pass, dim3(o.rec_blocks), dim3(kRecThreads), 0, s, o.views, o.n_views, o.keys_a, o.keys_b,
                         o.vals_a, o.vals_b, o.rec_hist, st, &o.tickets[p], o.unit, &o.tickets[5], err,
                         p);
    }
  }
  if (o.seq_blocks == 0) return hipGetLastError();
  return o.n_tiles <= 65536u ? order_pairs<uint16_t>(o, s) : order_pairs<uint32_t>(o, s);
}

// ---------------------------------------------------------------- inspection
// Copies of what the order-first path does not keep: tile boxes, keys in
// record order, sorted keys.
__device__ __forceinline__ int view_of_rec(const ViewD* __restrict__ views, int n_views, uint32_t r) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].rec_off <= r) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ void __launch_bounds__(256)
k_debug_emit(OrderBufs o, uint32_t n_rec, const float* __restrict__ records, const uint32_t* __restrict__ offsets,
             uint4* __restrict__ tile_box, uint64_t* __restrict__ keys_emit, uint32_t* __restrict__ vals_emit,
             uint32_t* __restrict__ depth_emit) {
  const uint32_t s = blockIdx.x * 256u + threadIdx.x;
  if (s >= n_rec) return;
  const int v = view_of_rec(o.views, o.n_views, s);
  const ViewD& V = o.views[v];
  const int lead = V.sort_mode == kSortFollow ? (int)V.sort_lead : v;
  const ViewD& L = o.views[lead];
  const uint32_t p = s - V.rec_off;
  if (p >= o.unit[2 * lead]) return;
  const bool side = o.unit[2 * lead + 1] != 0;
  const uint32_t rec = V.rec_off + ((side ? o.vals_b : o.vals_a)[L.sort_off + p] - L.rec_off);
  const uint32_t key = (side ? o.keys_b : o.keys_a)[L.sort_off + p];
  const uint2 bx = load_box(o.boxes, rec, o.box4);
  const uint32_t w = bx.y & 0xFFFFu, h = bx.y >> 16, tx = (uint32_t)V.tiles_x;
  if (w * h == 0) return;
  const uint32_t first = V.tile_off + (bx.x >> 16) * tx + (bx.x & 0xFFFFu);
  if (tile_box)
    tile_box[rec] = make_uint4(first, bx.y, __float_as_uint(records[(size_t)rec * kRecordFloats + 9]), tx);
  const uint32_t e0 = offsets[rec];
  for (uint32_t j = 0; j < w * h; ++j) {
    const uint32_t e = e0 + j;
    if (e >= o.cap) break;
    if (keys_emit) keys_emit[e] = ((uint64_t)(first + j / w * tx + j % w) << 32) | key;
    if (vals_emit) vals_emit[e] = rec;
    depth_emit[e] = key;
  }
}

template <typename TT>
__global__ void __launch_bounds__(256)
k_debug_sorted(OrderBufs o, const TT* __restrict__ tiles, const uint32_t* __restrict__ recs,
               const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ depth_emit,
               uint64_t* __restrict__ keys_sorted) {
  const uint32_t K = min(o.counters[kCntPairs], o.cap);
  const uint32_t k = blockIdx.x * 256u + threadIdx.x;
  if (k >= K) return;
  const uint32_t tile = tiles[k], rec = recs[k];
  const ViewD& V = o.views[view_of_rec(o.views, o.n_views, rec)];
  const uint2 bx = load_box(o.boxes, rec, o.box4);
  const uint32_t tx = (uint32_t)V.tiles_x, local = tile - V.tile_off;
  const uint32_t e = offsets[rec] + (local / tx - (bx.x >> 16)) * (bx.y & 0xFFFFu) + (local % tx - (bx.x & 0xFFFFu));
  keys_sorted[k] = ((uint64_t)tile << 32) | (e < o.cap ? depth_emit[e] : 0u);
}

// After launch_order, for inspection: any output may be null.
hipError_t launch_order_debug(const OrderBufs& o, uint32_t n_rec, const float* records, const uint32_t* offsets,
                              uint32_t* tile_box, uint64_t* keys_emit, uint32_t* vals_emit, uint64_t* keys_sorted,
                              hipStream_t s) {
  if (n_rec == 0 || o.cap == 0) return hipSuccess;
  int bits, np;
  tile_passes(o.n_tiles, &bits, &np);
  void* tiles = (np & 1) ? o.tile_b : o.tile_a;
  uint32_t* depth = reinterpret_cast<uint32_t*>((np & 1) ? o.tile_a : o.tile_b);  // free once the grouping is done
  hipLaunchKernelGGL(k_debug_emit, dim3(div_up(n_rec, 256u)), dim3(256), 0, s, o, n_rec, records, offsets,
                     reinterpret_cast<uint4*>(tile_box), keys_emit, vals_emit, depth);
  if (keys_sorted) {
    const uint32_t* recs = (np & 1) ? o.rec_b : o.rec_a;
    const dim3 grid(div_up(o.cap, 256u));
    if (o.n_tiles <= 65536u)
      hipLaunchKernelGGL(k_debug_sorted<uint16_t>, grid, dim3(256), 0, s, o, static_cast<const uint16_t*>(tiles), recs,
                         offsets, depth, keys_sorted);
    else
      hipLaunchKernelGGL(k_debug_sorted<uint32_t>, grid, dim3(256), 0, s, o, static_cast<const uint32_t*>(tiles), recs,
                         offsets, depth, keys_sorted);
  }
  return hipGetLastError();
}

}  // namespace gsr
