// The stable sort of a small input by one work-group, in LDS.
#pragma once

#include "common.hpp"

namespace ka {

template <int kBlock>
struct LdsSort {
  static constexpr int kWaves = kBlock / 64;
  __align__(16) uint16_t cnt[kWaves][256];  // per-wave digit counts, then each wave's start of each digit
  uint32_t scan[kWaves], k_or[kWaves], k_and[kWaves];
};

// n <= kBlock * kItems values (n > 0): element i's value (its bits in mask) and
// row i are put in order of value, equal values in row order, into store; wave w
// owns 64 kItems consecutive elements.  8-bit digits over the bits that differ
// between the values at all, ranked inside each wave by ballots; about 1.2 us a
// digit at kItems = 1.  Returns the OR of the values, all their bits.  Ends with
// a barrier.
template <int kBlock, int kItems, class Store>
__device__ __forceinline__ uint32_t lds_sort(const uint32_t* __restrict__ values, uint32_t n, const Store& store,
                                             LdsSort<kBlock>& S, uint32_t mask = ~0u) {
  constexpr int kWaves = kBlock / 64;
  static_assert(kBlock >= 256, "one work-item per digit");
  const uint32_t tid = threadIdx.x, w = tid / 64, lane = lane_id();
  const uint32_t i0 = w * 64 * kItems + lane;  // elements i0 + 64 i
  uint32_t key[kItems], row[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    row[i] = i0 + 64 * i;
    key[i] = row[i] < n ? values[row[i]] : 0u;
  }
  uint32_t o = 0, a = ~0u;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    o |= key[i];
    if (row[i] < n) a &= key[i];
    key[i] &= mask;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    o |= (uint32_t)__shfl_xor((int)o, off);
    a &= (uint32_t)__shfl_xor((int)a, off);
  }
  if (lane == 0) {
    S.k_or[w] = o;
    S.k_and[w] = a;
  }
  __syncthreads();
  o = 0, a = ~0u;
#pragma unroll
  for (int ww = 0; ww < kWaves; ++ww) {
    o |= S.k_or[ww];
    a &= S.k_and[ww];
  }
  const uint32_t diff = (uint32_t)__builtin_amdgcn_readfirstlane((int)((o ^ a) & mask));  // bits in which values differ
  const uint32_t lo = diff ? (uint32_t)__builtin_ctz(diff) : 32u, hi = diff ? 32u - (uint32_t)__builtin_clz(diff) : 0u;
  if (!diff) {  // all values equal: in order already
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (row[i] < n) store.put(row[i], key[i], row[i]);
  }
  for (uint32_t shift = lo; shift < hi; shift += 8) {
    for (int i = tid; i < kWaves * 256 / 2; i += kBlock) reinterpret_cast<uint32_t*>(&S.cnt[0][0])[i] = 0u;
    if (shift != lo) {  // what the pass before has placed
#pragma unroll
      for (int i = 0; i < kItems; ++i)
        if (i0 + 64 * i < n) store.get(i0 + 64 * i, key[i], row[i]);
    }
    __syncthreads();
    uint32_t rank[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const bool valid = i0 + 64 * i < n;
      const uint32_t d = (key[i] >> shift) & 255u;
      uint32_t dl = 0, dh = 0;
      differing_lanes<0>(d, dl, dh);
      differing_lanes<2>(d, dl, dh);
      differing_lanes<4>(d, dl, dh);
      differing_lanes<6>(d, dl, dh);
      const uint64_t peers = __builtin_amdgcn_ballot_w64(valid) & ~(((uint64_t)dh << 32) | dl);
      rank[i] = 0;
      if (valid) {
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
        const uint32_t old = S.cnt[w][d];
        if (below == 0) S.cnt[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
        rank[i] = old + below;
      }
    }
    __syncthreads();
    uint32_t cnt[kWaves], total = 0, all;
    if (tid < 256) {
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) {
        cnt[ww] = total;
        total += S.cnt[ww][tid];
      }
    }
    const uint32_t start = block_excl_scan<kBlock>(total, S.scan, &all);
    if (tid < 256) {
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) S.cnt[ww][tid] = (uint16_t)(start + cnt[ww]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (i0 + 64 * i < n) store.put(S.cnt[w][(key[i] >> shift) & 255u] + rank[i], key[i], row[i]);
    __syncthreads();
  }
  __syncthreads();
  return o;
}

}  // namespace ka
