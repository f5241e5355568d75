// Exclusive scan of the per-record tile counts, as a block's share of a
// launch (shared by the scan's own kernel and the one that also counts the
// record sort's digits).
#pragma once
#include "common.hpp"

namespace gsr {

// Block-wide exclusive scan of one value below 2^38 per thread.  The wave
// scans it in two parts of 26 and 12 bits, whose sums stay in 32.
template <int THREADS>
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t x, uint64_t* lds_waves, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t lo = wave_scan_add((uint32_t)x & ((1u << 26) - 1u)), hi = wave_scan_add((uint32_t)(x >> 26));
  const uint64_t inc = (uint64_t)lo + ((uint64_t)hi << 26);
  if (lane == 63) lds_waves[wave] = inc;
  __syncthreads();
  uint64_t wave_off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    const uint64_t c = lds_waves[w];
    if (w < wave) wave_off += c;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return wave_off + inc - x;
}

// Single pass with decoupled look-back: blocks take their tile index from a
// ticket (so a block only waits for blocks already running), publish the
// tile's total, and the first wave looks back over 64 predecessors at a time
// for the nearest inclusive prefix.  Status words: flag in the top 2 bits,
// 62-bit value.  The last tile writes the total K and the capacity check to
// counters.  Sums are of 64 bits (a block's 32768 records of 2^17 tiles each
// pass 2^32); an offset or a count beyond 32 bits is written as 2^32 - 1,
// which is beyond every capacity.
constexpr uint64_t kScanAgg = 1ull << 62;
constexpr uint64_t kScanIncl = 2ull << 62;
constexpr uint64_t kScanValue = (1ull << 62) - 1;
constexpr uint32_t kScanSpinLimit = 1u << 22;

// nb: the blocks of the launch that scan, THREADS ITEMS records each.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void scan_block(const uint32_t* __restrict__ in, uint32_t n, uint32_t* __restrict__ out,
                                           uint64_t* __restrict__ status, uint32_t* __restrict__ ticket,
                                           uint32_t* __restrict__ counters, uint32_t pair_capacity, uint32_t nb) {
  static_assert(ITEMS <= 64, "a thread's sum stays below 2^38");
  __shared__ uint64_t lds[THREADS / 64];
  __shared__ uint32_t s_bid;
  __shared__ uint64_t s_excl;
  if (threadIdx.x == 0) s_bid = atomicAdd(ticket, 1u);
  __syncthreads();
  const uint32_t bid = s_bid;
  // thread t owns ITEMS consecutive items
  const uint32_t base = bid * (uint32_t)(THREADS * ITEMS) + threadIdx.x * ITEMS;
  uint32_t v[ITEMS];
  if (base + ITEMS <= n) {
    const uint4* in4 = reinterpret_cast<const uint4*>(in + base);  // 64-byte aligned run
#pragma unroll
    for (int k = 0; k < ITEMS / 4; ++k) {
      const uint4 q = in4[k];
      v[4 * k] = q.x;
      v[4 * k + 1] = q.y;
      v[4 * k + 2] = q.z;
      v[4 * k + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) v[k] = (base + k < n) ? in[base + k] : 0u;
  }
  uint32_t lo = 0, hi = 0;  // in halves (64-bit additions took 70 registers more)
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    lo += v[k] & 0xFFFFu;
    hi += v[k] >> 16;
  }
  uint64_t total;
  const uint64_t local = block_exclusive_scan<THREADS>(lo + ((uint64_t)hi << 16), lds, &total);
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    if (lane == 0)
      __hip_atomic_store(&status[bid], (bid == 0 ? kScanIncl : kScanAgg) | total, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    uint64_t excl = 0;
    if (bid > 0) {
      int j = (int)bid - 1;  // window [j - 63, j]
      uint32_t spins = 0;
      for (;;) {
        const int idx = j - lane;
        const uint64_t sv =
            idx >= 0 ? __hip_atomic_load(&status[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kScanIncl;
        const uint64_t flag = sv & ~kScanValue;
        const uint64_t ready = __ballot(flag != 0);
        const uint64_t incl = __ballot(flag == kScanIncl);
        // lanes up to the first inclusive one, all ready: sum them
        const int first_incl = incl ? __builtin_ctzll(incl) : 64;
        const uint64_t need = first_incl < 63 ? ((2ull << first_incl) - 1) : ~0ull;
        if ((ready & need) != need) {
          if (++spins > kScanSpinLimit) {
            if (lane == 0) atomicOr(&counters[kCntError], 16u);
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        uint64_t x = (lane <= first_incl && idx >= 0) ? (sv & kScanValue) : 0ull;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        excl += x;
        if (first_incl < 64) break;
        j -= 64;
      }
      if (lane == 0)
        __hip_atomic_store(&status[bid], kScanIncl | ((excl + total) & kScanValue), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) {
      s_excl = excl;
      if (bid == nb - 1) {
        const uint64_t K = excl + total;
        counters[kCntPairs] = K > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)K;
        if (K > pair_capacity) atomicOr(&counters[kCntOverflow], 1u);  // sticky until the caller checks
      }
    }
  }
  __syncthreads();
  // (saturating: past 2^32 - 1 the offsets stay there)
  uint32_t run = (uint32_t)min(s_excl + local, (uint64_t)0xFFFFFFFFull);
  if (base + ITEMS <= n && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    uint4* out4 = reinterpret_cast<uint4*>(out + base);
#pragma unroll
    for (int k = 0; k < ITEMS / 4; ++k) {
      uint4 q;
      q.x = run;
      run = __builtin_elementwise_add_sat(run, v[4 * k]);
      q.y = run;
      run = __builtin_elementwise_add_sat(run, v[4 * k + 1]);
      q.z = run;
      run = __builtin_elementwise_add_sat(run, v[4 * k + 2]);
      q.w = run;
      run = __builtin_elementwise_add_sat(run, v[4 * k + 3]);
      out4[k] = q;
    }
  } else {
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      if (base + k < n) out[base + k] = run;
      run = __builtin_elementwise_add_sat(run, v[k]);
    }
  }
  // out[n] = total, written by the thread that owns the end
  if (base <= n && n < base + ITEMS) out[n] = run;
}

}  // namespace gsr
