// Device helpers of the kernels that scatter words into a tensor list
// (apply.hip, leb128.hip).
#pragma once

#include "delta_internal.h"

namespace aurora {

// A value every lane of the wavefront holds alike, in scalar registers.
__device__ __forceinline__ uint64_t run_uniform(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// A scattered word: streamed past the caches and, kThrough, written through
// to memory at once ("nt sc1": non-temporal, system scope), so that the words
// reach the memory in the order in which they leave.  A 1 / 2% delta over
// 4.02 G words takes 1260 / 1951 us with it, 1290 / 1990 without.
// The tensor addresses of the multi-tensor kernels come from a table in
// memory, so the store names the global segment itself (a flat store would
// also count against the LDS wait counter).
template <bool kThrough>
__device__ __forceinline__ void store_word(uint16_t* p, uint16_t v) {
  if (kThrough)
    asm volatile("global_store_short %0, %1, off sc1 nt" ::"v"(p), "v"((uint32_t)v) : "memory");
  else
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) uint16_t*)p);
}

// Block b of n in the order in which XCD x takes the x-th eighth.
__device__ __forceinline__ uint64_t xcd_block(uint64_t b, uint64_t n) {
  const uint64_t x = b % 8, q = b / 8, per = n / 8, rem = n % 8;
  return x * per + (x < rem ? x : rem) + q;
}

// Global index -> (tensor, local index) over T tensors with bases[0..T]
// (bases[t] = first global index of tensor t, bases[T] = total).
__device__ __forceinline__ uint32_t find_tensor(const uint64_t* bases, uint32_t T, uint64_t g) {
  uint32_t lo = 0, hi = T;   // answer in [lo, hi): bases[lo] <= g < bases[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (bases[mid] <= g) lo = mid; else hi = mid;
  }
  return lo;
}

// The tensor of a wavefront's first entry, found by the whole wavefront: for
// up to 64 R tensors every lane holds R bases, loaded before the entry is
// known, and the bases at or below it are counted (otherwise, and with R =
// 0, a search).  A search of dependent loads in every wavefront costs more
// than its few entries have to hide it: the scatter of a 1% delta over 8.19 G
// words in 399 tensors takes 2.92 ms with it (192 threads a workgroup) and
// 2.52 without.
template <int R>
struct WaveBases {
  uint64_t b[R > 0 ? R : 1];
  __device__ __forceinline__ WaveBases(const uint64_t* bases, uint32_t T) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t p = 64 * r + (threadIdx.x & 63);
      b[r] = p < T ? bases[p] : ~0ull;
    }
  }
  __device__ __forceinline__ uint32_t tensor(const uint64_t* bases, uint32_t T,
                                             uint64_t first) const {
    uint32_t t = 0;
    if (R > 0 && T <= 64 * R) {
      uint32_t c = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) c += (uint32_t)__builtin_popcountll(__ballot(b[r] <= first));
      if (c > T) c = T;   // an entry past every list
      t = c ? c - 1 : 0;
    } else {
      t = find_tensor(bases, T, first);
    }
    return __builtin_amdgcn_readfirstlane(t);
  }
};

}  // namespace aurora
