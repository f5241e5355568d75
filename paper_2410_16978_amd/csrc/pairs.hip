// Integer stages between projection and blending: exclusive scan of the
// per-record tile counts, duplication into (tile << 32 | depth bits, record)
// pairs in emission order, and per-tile [start, end) ranges of the sorted
// pairs.
#include "common.hpp"
#include "scan.hpp"

namespace gsr {

// ---------------------------------------------------------------- scan
__global__ void __launch_bounds__(kScanThreads)
k_scan(const uint32_t* __restrict__ in, uint32_t n, uint32_t* __restrict__ out, uint64_t* __restrict__ status,
       uint32_t* __restrict__ ticket, uint32_t* __restrict__ counters, uint32_t pair_capacity) {
  scan_block<kScanThreads, kScanItems>(in, n, out, status, ticket, counters, pair_capacity, gridDim.x);
}

uint32_t scan_tiles(uint32_t n) { return div_up(n + 1, (uint32_t)kScanTile); }

// status: scan_tiles(n) zeroed words; ticket: a zeroed counter.
hipError_t launch_scan(const uint32_t* in, uint32_t* out, uint64_t* status, uint32_t* ticket, uint32_t n,
                       uint32_t* counters, uint32_t pair_capacity, hipStream_t s) {
  hipLaunchKernelGGL(k_scan, dim3(scan_tiles(n)), dim3(kScanThreads), 0, s, in, n, out, status, ticket, counters,
                     pair_capacity);
  return hipGetLastError();
}

// ---------------------------------------------------------------- duplicate
// Each wave takes 64 consecutive records, whose pairs form one contiguous
// emission range (offsets is their exclusive scan), and writes that range
// with its lanes striding over the pairs: lane i writes pair base + i,
// finding the record that owns it by a binary search over the wave's
// offsets.  A record's tiles are row-major in its box.  Writes are
// coalesced and a large splat's pairs spread over the wave instead of one
// lane.  Pairs at or beyond min(capacity, counters[pairs]) are dropped (the
// overflow flag or the batch status already records it).  The sort carries
// each pair's emission index as its value; rec_of[e] keeps the record of
// emission index e.
template <bool BY_BOX>
__global__ void __launch_bounds__(256)
k_duplicate(const uint32_t* __restrict__ n_tiles, const uint32_t* __restrict__ offsets,
            const uint4* __restrict__ tile_box, uint32_t n_rec, const uint32_t* __restrict__ counters,
            uint32_t pair_capacity, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
            uint32_t* __restrict__ rec_of, BoxSource src) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const uint32_t lim = min(pair_capacity, counters[kCntPairs]);
  const bool valid = r < n_rec;
  const uint32_t cnt = valid ? n_tiles[r] : 0u;
  const uint32_t off = valid ? offsets[r] : 0xFFFFFFFFu;  // invalid lanes never own a pair
  uint4 tb = make_uint4(0u, 0u, 0u, 0u);
  if (cnt) {
    if (BY_BOX) {
      const uint2 q = load_box(src.boxes, r, src.box4);
      tb = make_uint4(r / src.n * src.tiles_per_view + (q.x >> 16) * src.tiles_x + (q.x & 0xFFFFu), q.y, src.depth[r],
                      src.tiles_x);
    } else {
      tb = tile_box[r];
    }
  }
  uint32_t end = valid ? off + cnt : 0u;
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) end = max(end, (uint32_t)__shfl_xor((int)end, s, 64));
  const uint32_t w0 = (uint32_t)__shfl((int)off, 0, 64);
  const uint32_t w1 = min(end, lim);
  const uint32_t r0 = r - (uint32_t)lane;
  for (uint32_t base = w0; base < w1; base += 64) {
    const uint32_t e = base + (uint32_t)lane;
    // last lane whose offset is <= e (zero-count records share the next offset)
    int lo = 0;
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) {
      const uint32_t o = (uint32_t)__shfl((int)off, lo + st, 64);
      if (o <= e) lo += st;
    }
    const uint32_t o = (uint32_t)__shfl((int)off, lo, 64);
    const uint32_t bx = (uint32_t)__shfl((int)tb.x, lo, 64);
    const uint32_t by = (uint32_t)__shfl((int)tb.y, lo, 64);
    const uint32_t bz = (uint32_t)__shfl((int)tb.z, lo, 64);
    const uint32_t bw = (uint32_t)__shfl((int)tb.w, lo, 64);
    if (e < w1) {
      const uint32_t j = e - o;
      const uint32_t w = max(by & 0xFFFFu, 1u);
      uint32_t dy;
      if (j < (1u << 24)) {  // float quotient, corrected to floor(j / w)
        dy = (uint32_t)((float)j / (float)w);
        if (dy * w > j) --dy;
        if ((dy + 1) * w <= j) ++dy;
      } else {
        dy = j / w;
      }
      const uint32_t tile = bx + dy * bw + (j - dy * w);
      keys[e] = ((uint64_t)tile << 32) | bz;
      vals[e] = e;
      rec_of[e] = r0 + (uint32_t)lo;
    }
  }
}

hipError_t launch_duplicate(const uint32_t* n_tiles, const uint32_t* offsets, const uint4* tile_box,
                            uint32_t n_rec, const uint32_t* counters, uint32_t pair_capacity,
                            uint64_t* keys, uint32_t* vals, uint32_t* rec_of, const BoxSource& src, hipStream_t s) {
  if (n_rec == 0) return hipSuccess;
  hipLaunchKernelGGL(src.boxes ? k_duplicate<true> : k_duplicate<false>, dim3(div_up(n_rec, 256u)), dim3(256), 0, s,
                     n_tiles, offsets, tile_box, n_rec, counters, pair_capacity, keys, vals, rec_of, src);
  return hipGetLastError();
}

// ---------------------------------------------------------------- ranges
__global__ void __launch_bounds__(256)
k_ranges(const uint64_t* __restrict__ keys_a, const uint64_t* __restrict__ keys_b,
         const uint32_t* __restrict__ sel, uint32_t* __restrict__ counters, uint32_t pair_capacity,
         uint32_t total_tiles, uint32_t* __restrict__ ranges) {
  const uint32_t K = min(counters[kCntPairs], pair_capacity);
  const uint64_t* keys = (*sel == 0) ? keys_a : keys_b;
  for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x) {
    const uint32_t t = (uint32_t)(keys[k] >> 32);
    if (t >= total_tiles) {
      atomicOr(&counters[kCntError], 4u);
      continue;
    }
    if (k == 0 || (uint32_t)(keys[k - 1] >> 32) != t) ranges[2 * t] = k;
    if (k + 1 == K || (uint32_t)(keys[k + 1] >> 32) != t) ranges[2 * t + 1] = k + 1;
  }
}

hipError_t launch_ranges(const uint64_t* keys_a, const uint64_t* keys_b, const uint32_t* sel,
                         uint32_t* counters, uint32_t pair_capacity, uint32_t total_tiles, uint32_t* ranges,
                         hipStream_t s) {
  if (pair_capacity == 0) return hipSuccess;
  uint32_t grid = div_up(pair_capacity, 256u);
  if (grid > 8192) grid = 8192;
  hipLaunchKernelGGL(k_ranges, dim3(grid), dim3(256), 0, s, keys_a, keys_b, sel, counters, pair_capacity,
                     total_tiles, ranges);
  return hipGetLastError();
}

// ---------------------------------------------------------------- tile order
// Tiles grouped by pair count into kTileClasses classes (largest first,
// empty tiles last), so that the forward blend starts its longest tiles
// first.  One block per 1024
// tiles: class counts per block (ballots), one addition per class and
// block reserves the block's slots in the class list.  The order within a
// class depends on the order the blocks run, which changes no result.

__global__ void __launch_bounds__(1024)
k_tile_order(const uint32_t* __restrict__ ranges, uint32_t n_tiles, uint32_t* __restrict__ class_count,
             uint32_t* __restrict__ class_list) {
  __shared__ uint32_t wc[16][kTileClasses];
  __shared__ uint32_t base[kTileClasses];
  const uint32_t t = blockIdx.x * 1024u + threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t n = 0;
  if (t < n_tiles) {
    const uint32_t s0 = ranges[2 * t], s1 = ranges[2 * t + 1];
    n = s1 > s0 ? s1 - s0 : 0u;
  }
  const uint32_t c = t < n_tiles ? tile_class(n) : kTileClasses;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t rank = 0;
#pragma unroll
  for (uint32_t k = 0; k < kTileClasses; ++k) {
    const uint64_t m = __ballot(c == k);
    if (c == k) rank = (uint32_t)__popcll(m & below);
    if (lane == 0) wc[wave][k] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  if (threadIdx.x < kTileClasses) {
    uint32_t tot = 0;
    for (int w = 0; w < 16; ++w) tot += wc[w][threadIdx.x];
    base[threadIdx.x] = tot ? atomicAdd(&class_count[threadIdx.x], tot) : 0u;
  }
  __syncthreads();
  if (c < kTileClasses) {
    uint32_t pos = base[c] + rank;
    for (int w = 0; w < wave; ++w) pos += wc[w][c];
    if (pos < n_tiles) class_list[(size_t)c * n_tiles + pos] = t;
  }
}

hipError_t launch_tile_order(const uint32_t* ranges, uint32_t n_tiles, uint32_t* class_count,
                             uint32_t* class_list, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_order, dim3(div_up(n_tiles, 1024u)), dim3(1024), 0, s, ranges, n_tiles, class_count,
                     class_list);
  return hipGetLastError();
}

// ---------------------------------------------------------------- batch status
// Requests own contiguous record ranges [req_rec[q], req_rec[q+1]), so their
// pairs are contiguous in emission order.  A request whose pairs end beyond
// the capacity is marked GSR_ENOSPACE (-2) (a suffix of the requests) and the
// pair count is cut to the end of the last request that fits, so that only
// whole requests are duplicated, sorted and blended.
__global__ void k_batch_status(const uint32_t* __restrict__ req_rec, int n_req,
                               const uint32_t* __restrict__ offsets, uint32_t pair_capacity,
                               uint32_t* __restrict__ counters, int32_t* __restrict__ req_status) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  uint32_t k_fit = 0;
  for (int q = 0; q < n_req; ++q) {
    const uint32_t end = offsets[req_rec[q + 1]];
    const bool fits = end <= pair_capacity;
    req_status[q] = fits ? 0 : -2;
    if (fits) k_fit = end;
  }
  counters[kCntPairs] = k_fit;
  counters[kCntOverflow] = 0;
}

// After a batch: a device-side error anywhere in the call (the sort's or the
// scan's bounded waits, inconsistent offsets) marks every request
// GSR_EDEVICE (-4), so no image of a faulty sort is reported as good.
__global__ void k_batch_error(const uint32_t* __restrict__ counters, int n_req, int32_t* __restrict__ req_status) {
  if (counters[kCntError] == 0u) return;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n_req; q += gridDim.x * blockDim.x) req_status[q] = -4;
}

hipError_t launch_batch_error(const uint32_t* counters, int n_req, int32_t* req_status, hipStream_t s) {
  if (n_req <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_error, dim3(1), dim3(256), 0, s, counters, n_req, req_status);
  return hipGetLastError();
}

hipError_t launch_batch_status(const uint32_t* req_rec, int n_req, const uint32_t* offsets,
                               uint32_t pair_capacity, uint32_t* counters, int32_t* req_status,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_batch_status, dim3(1), dim3(64), 0, s, req_rec, n_req, offsets, pair_capacity,
                     counters, req_status);
  return hipGetLastError();
}

}  // namespace gsr
