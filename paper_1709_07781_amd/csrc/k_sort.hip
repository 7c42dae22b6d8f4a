// Stable LSB radix sort of (uint32 key, uint32 row) pairs by key -- parts 1
// and 2 of the WAH index build (Sec. 4.1: tag every value with its input
// position, then sort by value; Sec. 4.2 sorts with a radix sort).
//
// Up to four passes of 8-bit digits (or, for values known to be below 2^16, one
// or two of 2 to 8 bits), each a count of every tile and a scatter; no
// work-group waits for another one:
//  * the count (one work-group per tile) writes the tile's digit counts as a row
//    of uint16; the pass-0 instance for any uint32 keys also records the OR and
//    the AND of the tile's keys, from which the sort plan is formed: a pass whose
//    digit is the same in every key (equal in the OR and the AND) is the identity
//    of a stable sort and is skipped, so 16-bit keys cost two passes;
//  * inputs of few tiles: every scatter work-group adds up the rows before its
//    own, and all of them for the digits' totals, while its keys are on their
//    way; more tiles: k_rows_scan first forms the digits' totals and, down every
//    column, the rows' prefixes;
//  * the scatter (one work-group per tile) ranks its keys by digit inside
//    each wave -- the lanes holding the same digit are found by OR-ing each
//    lane's bit into a per-digit mask in LDS (8-bit digits; digits 0 and 1 by a
//    ballot each) or with one ballot per digit bit (narrower digits), and a
//    key's rank is the number of such lanes below it plus the wave's earlier
//    count of that digit, so equal keys keep their order -- reorders the tile by
//    digit in LDS and writes each digit's run to its place, consecutive
//    work-items writing consecutive addresses.
// Tiles are taken in an XCD-aware order (see xcd_tile).
// The first active pass reads the input (and makes row ids 0..n-1 when no rows
// are given), later ones read the previous active pass's output, and the last
// active pass writes the caller's buffers.  A batch of requests is sorted inside
// every request (the segmented sort below).
#include <algorithm>
#include <cstddef>
#include <type_traits>

#include "common.hpp"

namespace ka {
namespace {

constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;
constexpr int kPasses = 32 / kRadixBits;

#ifndef KA_XCD_MAP
#define KA_XCD_MAP 1
#endif
// Tile shapes (work-items x keys per work-item of the scatter), chosen per
// launch: variant 0 is the default, the others are candidates for autotuning.
// (Persistent scatters that load the next tile into a second register set
// while ranking the current one ran 35-60% slower at every shape: the extra
// registers cost more occupancy than the prefetch saves.)
struct SortShape {
  int block, items;
};
constexpr SortShape kShapes[] = {{1024, 8}, {512, 16}, {512, 8}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

}  // namespace

// The sort plan, written between the first count and the first scatter.
struct SortPlan {
  uint32_t active;               // bit p: pass p moves data
  uint32_t keys_or;              // OR of all keys
};
static_assert(sizeof(SortPlan) <= kSortPlanBytes, "plan storage");

namespace {

struct PassBuffers {
  const uint32_t* keys_in;
  const uint32_t* rows_in;  // null: rows are positions 0..n-1
  uint32_t* keys_a;         // caller's output (written by the last active pass)
  uint32_t* rows_a;
  uint32_t* keys_b;         // scratch ping-pong buffer
  uint32_t* rows_b;
};

// Source and destination of one pass; keys are uint32, or uint16 in the
// narrow-key sort.
template <class SK, class DK>
struct PassIoT {
  // uint32 values in, uint16 keys out: the first pass, whose rows are positions
  static constexpr bool kPacked = sizeof(SK) == 4 && sizeof(DK) == 2;
  const SK* src_keys;
  const uint32_t* src_rows;
  DK* dst_keys;
  uint32_t* dst_rows;
  bool implicit_rows;
  uint32_t row_origin = 0;  // implicit rows: position - row_origin
  uint32_t key_or = 0;      // keys written as (key & key_and) | key_or (kTag scatters only)
  uint32_t key_and = ~0u;
};
using PassIo = PassIoT<uint32_t, uint32_t>;

// Source and destination of pass `pass` under the plan's active mask: the
// last active pass writes buffer a, the one before it b, and so on.
__device__ __forceinline__ PassIo pass_io(const PassBuffers& buf, uint32_t active, uint32_t pass) {
  const uint32_t later = (uint32_t)__popc(active >> pass);  // active passes from this one on
  const bool first = (active & ((1u << pass) - 1)) == 0;
  PassIo io;
  io.dst_keys = (later & 1u) ? buf.keys_a : buf.keys_b;
  io.dst_rows = (later & 1u) ? buf.rows_a : buf.rows_b;
  io.src_keys = first ? buf.keys_in : (((later + 1) & 1u) ? buf.keys_a : buf.keys_b);
  io.src_rows = first ? buf.rows_in : (((later + 1) & 1u) ? buf.rows_a : buf.rows_b);
  io.implicit_rows = first && buf.rows_in == nullptr;
  return io;
}

// LDS add of 1 to bin d by every active lane, aggregated over lanes that share
// a bin: in each of kRounds rounds the first remaining lane's bin takes the
// count of all remaining lanes with that bin in one add; the lanes left after
// the rounds add 1 each.  One round suits keys in input order (a second round
// in the first pass cost +9 us on Zipf keys); the later passes count in
// registers instead (upsweep_tile with kRounds < 0).
template <int kRounds>
__device__ __forceinline__ void lds_add_aggregated(uint32_t* bins, uint32_t d, bool valid) {
  uint64_t rest = __ballot(valid);
#pragma unroll
  for (int round = 0; round < kRounds; ++round) {
    if (!rest) return;
    const uint32_t first_lane = (uint32_t)__builtin_ctzll(rest);
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)first_lane);
    const uint64_t same = __ballot(d == d0) & rest;
    if (lane_id() == first_lane) atomicAdd(&bins[d0], (uint32_t)__popcll(same));
    rest &= ~same;
  }
  if ((rest >> lane_id()) & 1ull) atomicAdd(&bins[d], 1u);
}

// Tile of work-group b under an XCD-aware order.  Work-groups are dispatched
// round-robin over the 8 XCDs (b mod 8), each with its own L2; this gives XCD x
// the contiguous tile range [x*q + min(x, r), ...) of q or q + 1 tiles (q =
// ntiles / 8, r = ntiles mod 8), so neighbouring tiles -- whose output runs meet
// in the same cache lines -- are handled by the same L2.  A bijection on
// [0, ntiles) for every ntiles.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t ntiles) {
#if KA_XCD_MAP
  const uint32_t x = b & 7u, i = b >> 3, q = ntiles >> 3, r = ntiles & 7u;
  return x * q + min(x, r) + i;
#else
  (void)ntiles;
  return b;
#endif
}

// Elements of tile `tile` (kTile each) out of n: n_cap, or the count *d_n
// written on the device by an earlier stage (grids are then sized by the
// capacity and the tiles past the count are empty).
__device__ __forceinline__ uint32_t tile_len(uint32_t tile, uint32_t kTile, uint32_t n_cap, const uint64_t* d_n) {
  const uint32_t n = (uint32_t)device_count(n_cap, d_n), base = tile * kTile;
  return base < n ? min(kTile, n - base) : 0u;
}

// ---------------------------------------------------------------------------------
// upsweep: digit counts of one tile
// ---------------------------------------------------------------------------------
constexpr int kUpBlock = kRadix;  // one work-item per digit when the counts are written

// All of a work-item's loads are issued before the first key is counted; with
// kOrAnd the OR and the AND of the tile's keys are written too.
// The tile is keys[base, base + len); store(d, c) gets digit d's count: rows[tile][d],
// or the segmented sort's table.
template <int kBlock, int kTile, int kRounds, bool kOrAnd, class SK, class Store>
__device__ __forceinline__ void upsweep_tile(const SK* __restrict__ keys, uint32_t shift, uint32_t base, uint32_t len,
                                             Store&& store, uint32_t tile, uint32_t* __restrict__ orand,
                                             uint32_t mask = kRadix - 1) {
  constexpr int kUpWaves = kBlock / 64;
  constexpr int kUpVecs = kTile / 4 / kBlock;  // 4-key loads per work-item
  constexpr uintptr_t kAlign = 15;  // 16-byte loads
  __shared__ uint32_t s_hist[kUpWaves][kRadix];
  __shared__ uint32_t s_or[kUpWaves], s_and[kUpWaves];
  const uint32_t tid = threadIdx.x, w = tid / 64;

  // Key 4 (j * kBlock + tid) + c of the tile in k[j][c] (uint16 keys of a full
  // tile: key 8 (j/2 * kBlock + tid) + 4 (j mod 2) + c).
  uint32_t k[kUpVecs][4];
  if (len == (uint32_t)kTile && (reinterpret_cast<uintptr_t>(keys + base) & kAlign) == 0) {
    if constexpr (sizeof(SK) == 2 && kUpVecs % 2 == 0) {
      // uint16 keys: 8 per 16-byte load (which keys a work-item holds does not
      // change the counts); half the loads of 8-byte ones: 40.5 -> 35.9 us for
      // the second pass over 2^26 keys
#pragma unroll
      for (int j = 0; j < kUpVecs / 2; ++j) {
        const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(keys + base) + j * kBlock + tid);
        k[2 * j][0] = a.x & 0xFFFFu, k[2 * j][1] = a.x >> 16, k[2 * j][2] = a.y & 0xFFFFu, k[2 * j][3] = a.y >> 16;
        k[2 * j + 1][0] = a.z & 0xFFFFu, k[2 * j + 1][1] = a.z >> 16;
        k[2 * j + 1][2] = a.w & 0xFFFFu, k[2 * j + 1][3] = a.w >> 16;
      }
    } else {
#pragma unroll
      for (int j = 0; j < kUpVecs; ++j) load_key4(keys + base, (uint64_t)j * kBlock + tid, k[j]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < kUpVecs; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t e = 4 * (j * kBlock + tid) + c;
        k[j][c] = e < len ? (uint32_t)keys[base + e] : 0u;
      }
  }
  for (int i = tid; i < kUpWaves * kRadix; i += kBlock) (&s_hist[0][0])[i] = 0;
  __syncthreads();
  uint32_t kor = 0, kand = ~0u;
  // kRounds < 0: two digits are counted in registers -- 0 and the digit of the
  // wave's first key -- and every other key adds 1 in LDS.  After the first
  // pass of an LSD sort a tile's keys share their low digit and the next digit
  // is concentrated in few values, the most often 0 for small values or else
  // likely the first key's; the aggregated adds' ballots and lane reads cost
  // more there (measured on 16-bit Zipf keys: 62 -> 42 us; uniform keys 51 ->
  // 44 us).
  uint32_t c0 = 0, ch = 0;
  // Clustered keys (most work-items' four neighbouring keys share a digit): a
  // work-item's four are added as one, and the wave's equal digits in one add each.
  const uint32_t da = (k[0][0] >> shift) & mask, db = (k[0][3] >> shift) & mask;
  const uint32_t df = (uint32_t)__builtin_amdgcn_readfirstlane((int)da);
  bool clustered = __popcll(__ballot(da == db)) >= 48 && len == (uint32_t)kTile;  // uniform over the wave
  if (kRounds < 0)  // not those that sit in the two digits counted in registers
    clustered = clustered && __popcll(__ballot(da == df || da == 0u)) < 40;
  if (clustered) {
#pragma unroll
    for (int j = 0; j < kUpVecs; ++j) {
      uint32_t d[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        d[c] = (k[j][c] >> shift) & mask;
        if (kOrAnd) {
          kor |= k[j][c];
          kand &= k[j][c];
        }
      }
      const bool same = d[0] == d[1] && d[0] == d[2] && d[0] == d[3];
      uint64_t rest = __ballot(same);
      for (int round = 0; round < 3 && rest; ++round) {
        const uint32_t first_lane = (uint32_t)__builtin_ctzll(rest);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d[0], (int)first_lane);
        const uint64_t eq = __ballot(same && d[0] == d0);
        if (lane_id() == first_lane) atomicAdd(&s_hist[w][d0], 4u * (uint32_t)__popcll(eq));
        rest &= ~eq;
      }
      if ((rest >> lane_id()) & 1ull)
        atomicAdd(&s_hist[w][d[0]], 4u);
      else if (!same)
#pragma unroll
        for (int c = 0; c < 4; ++c) atomicAdd(&s_hist[w][d[c]], 1u);
    }
  }
  const uint32_t hot = (uint32_t)__builtin_amdgcn_readfirstlane((int)((k[0][0] >> shift) & mask));
  if (!clustered) {
#pragma unroll
    for (int j = 0; j < kUpVecs; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool valid = 4 * (j * kBlock + tid) + c < len;
        if (kRounds < 0) {
          const uint32_t d = (k[j][c] >> shift) & mask;
          if (valid) {
            if (d == hot)
              ++ch;
            else if (d == 0)
              ++c0;
            else
              atomicAdd(&s_hist[w][d], 1u);
          }
        } else {
          lds_add_aggregated<(kRounds < 0 ? 0 : kRounds)>(s_hist[w], (k[j][c] >> shift) & mask, valid);
        }
        if (kOrAnd && valid) {
          kor |= k[j][c];
          kand &= k[j][c];
        }
      }
  }
  if (kRounds < 0 && !clustered) {
    const uint32_t z = wave_sum(c0), h = wave_sum(ch);
    if (lane_id() == 0) {
      if (z) atomicAdd(&s_hist[w][0], z);
      if (h) atomicAdd(&s_hist[w][hot], h);
    }
  }
  if (kOrAnd) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      kor |= (uint32_t)__shfl_xor((int)kor, off);
      kand &= (uint32_t)__shfl_xor((int)kand, off);
    }
    if (lane_id() == 0) {
      s_or[w] = kor;
      s_and[w] = kand;
    }
  }
  __syncthreads();
  if (kBlock == kRadix || tid < (uint32_t)kRadix) {
    uint32_t c = 0;
#pragma unroll
    for (int ww = 0; ww < kUpWaves; ++ww) c += s_hist[ww][tid];
    store(tid, c);
  }
  if (kOrAnd && tid == 0) {
    uint32_t o = 0, a = ~0u;
#pragma unroll
    for (int ww = 0; ww < kUpWaves; ++ww) {
      o |= s_or[ww];
      a &= s_and[ww];
    }
    orand[2 * tile] = o;
    orand[2 * tile + 1] = a;
  }
}

// The look-back words of the encoder that follows the sort, zeroed by the
// sort's first launch (work-group b takes words b, b + grid, ...).
__device__ __forceinline__ void clear_words(const ClearWords& cw) {
  if (threadIdx.x == 0)
    for (uint32_t i = blockIdx.x; i < cw.count; i += gridDim.x) cw.p[kLbSpread * i] = 0ull;
}

// Passes that move data: those whose digit is not the same in every key, i.e.
// differs between the OR and the AND of the keys (all keys equal: one pass
// still moves them).
__device__ __forceinline__ uint32_t active_passes(uint32_t keys_or, uint32_t keys_and) {
  const uint32_t diff = keys_or ^ keys_and;
  uint32_t act = 0;
#pragma unroll
  for (int p = 0; p < kPasses; ++p)
    if ((diff >> (p * kRadixBits)) & (kRadix - 1)) act |= 1u << p;
  return act ? act : 1u << (kPasses - 1);
}

// OR and AND over the tiles' (OR, AND) pairs, in every work-item; s_or and
// s_and: kBlock / 64 words each.
template <int kBlock>
__device__ __forceinline__ void block_or_and(const uint32_t* __restrict__ orand, uint32_t ntiles, uint32_t* s_or,
                                             uint32_t* s_and, uint32_t* keys_or, uint32_t* keys_and) {
  uint32_t o = 0, a = ~0u;
  for (uint32_t t = threadIdx.x; t < ntiles; t += kBlock) {
    o |= orand[2 * t];
    a &= orand[2 * t + 1];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    o |= (uint32_t)__shfl_xor((int)o, off);
    a &= (uint32_t)__shfl_xor((int)a, off);
  }
  if (lane_id() == 0) {
    s_or[threadIdx.x / 64] = o;
    s_and[threadIdx.x / 64] = a;
  }
  __syncthreads();
  o = 0, a = ~0u;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) {
    o |= s_or[w];
    a &= s_and[w];
  }
  *keys_or = o;
  *keys_and = a;
}

// ---------------------------------------------------------------------------------
// scatter: one tile, ranked in LDS, written to its offsets
// ---------------------------------------------------------------------------------
// kPacked (the first pass over values of at most 16 bits): an element is
// reordered as one word, its key and its place in the tile, from which the row
// follows; half the LDS traffic and conflicts of (key, row) pairs: 178 -> 162 us
// for 2^26 Zipf values, 96 -> 86 for a batch of 2.8 10^7.  (512 x 16 work-groups,
// of which four then fit a CU: 193 us, the ranking's 16 steps are too long.
// Stores by 32-bit offsets: no change.)
template <int kBlock, int kItems, bool kPacked = false>
struct ScatterLds {
  static constexpr int kWaves = kBlock / 64;
  static constexpr int kTile = kBlock * kItems;
  static constexpr int kBytes = kPacked ? 4 * kTile : 8 * kTile;
  static constexpr int kMaskBytes = 8 * kWaves * kRadix;
  // reorder buffer (the rank masks before)
  __align__(16) unsigned char kr[kBytes > kMaskBytes ? kBytes : kMaskBytes];
  __device__ __forceinline__ uint2* pairs() { return reinterpret_cast<uint2*>(kr); }
  __device__ __forceinline__ uint32_t* words() { return reinterpret_cast<uint32_t*>(kr); }
  uint16_t wcnt[kWaves][kRadix];  // per-wave digit counts, then each wave's start of each digit in the tile
  uint32_t dbase[kRadix];         // global start minus tile-local start
  uint32_t before[kRadix];        // tile rows: digit counts of the tiles before this one
  uint32_t from[kRadix];          // and of this one and the later ones
  uint32_t scan[kWaves], scan2[kWaves];
};

// Where a scatter's starts come from: sums of the rows by every work-group
// (kSum), whose traffic out of L2 is tiles^2 * digits * 2 bytes, or the rows'
// prefixes (kScanned), one launch more a pass.
enum Starts { kGiven, kSum, kScanned };
// k_rows_scan writes the prefix of every kRowGroup-th row, and a scatter
// work-group adds the up to three rows after it to that (uint16 loads that
// arrive behind its keys): at 8192 tiles the scatters took 162 + 176 / 158 + 177 /
// 167 + 183 us with 1 / 4 / 8 rows, the scan the least with 4 or more.
constexpr uint32_t kRowGroup = 4;
// Scanned rows are stored by groups of kRowGroup, four digits of each row beside
// those of the next one: the place of digit d in the row of tile `tile`.
__device__ __forceinline__ uint32_t grouped_digit(uint32_t tile, uint32_t d) {
  return d / 4u * (4u * kRowGroup) + tile % kRowGroup * 4u + d % 4u;
}

// The tile's keys and rows: wave w owns 64*kItems consecutive elements, lane
// l the elements w*64*kItems + i*64 + l.
template <int kBlock, int kItems, class IO>
__device__ __forceinline__ void scatter_load(const IO& io, uint32_t base, uint32_t tile_n,
                                             uint32_t (&key)[kItems], uint32_t (&row)[kItems]) {
  constexpr int kTile = kBlock * kItems;
  const uint32_t w = threadIdx.x / 64, lane = lane_id();
  const uint32_t wbase = w * 64 * kItems;
  if (tile_n == (uint32_t)kTile) {  // uniform: every load of a full tile is issued unconditionally
#pragma unroll
    for (int i = 0; i < kItems; ++i) key[i] = __builtin_nontemporal_load(io.src_keys + base + wbase + i * 64 + lane);
    if (IO::kPacked) {
#pragma unroll
      for (int i = 0; i < kItems; ++i) row[i] = 0u;  // made when written
    } else if (io.implicit_rows) {
#pragma unroll
      for (int i = 0; i < kItems; ++i) row[i] = base + wbase + i * 64 + lane - io.row_origin;
    } else {
#pragma unroll
      for (int i = 0; i < kItems; ++i)
        row[i] = __builtin_nontemporal_load(io.src_rows + base + wbase + i * 64 + lane);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const uint32_t local = wbase + i * 64 + lane;
      const uint32_t g = base + local;
      const bool valid = local < tile_n;
      key[i] = valid ? (uint32_t)io.src_keys[g] : 0u;
      row[i] = valid ? (io.implicit_rows ? g - io.row_origin : io.src_rows[g]) : 0u;
    }
  }
}

// Where a tile's runs go, from tile rows (see k_radix_count_fixed): T rows of counts,
// this tile's is row `tile`; `origin` is the first position of all.
struct TileRows {
  const uint16_t* rows = nullptr;
  uint32_t T = 0, tile = 0, origin = 0;
  uint32_t before = 0, total = 0;  // kScanned: of digit threadIdx.x, in the tiles before this one and in all
};

// Adds the rows' counts to before and from (LDS, zeroed): a wave reads 512
// bytes of rows at a time.
template <int kBlock, int kBits, class Lds>
__device__ __forceinline__ void add_rows(const TileRows& tr, Lds& L) {
  constexpr uint32_t kD = 1u << kBits, kWaves = kBlock / 64;
  constexpr uint32_t kLanes = kD / 4, kRowsPer = 64 / kLanes;  // lanes per row, rows per wave and step
  const uint32_t w = threadIdx.x / 64, lane = lane_id();
  const uint32_t col = lane % kLanes, sub = lane / kLanes;
  uint32_t bef[4] = {0, 0, 0, 0}, aft[4] = {0, 0, 0, 0};
  const uint2* src = reinterpret_cast<const uint2*>(tr.rows) + col;
#pragma unroll 4
  for (uint32_t r0 = w * kRowsPer; r0 < tr.T; r0 += kWaves * kRowsPer) {
    const uint32_t r = r0 + sub;
    uint2 v = make_uint2(0u, 0u);
    if (r < tr.T) v = src[(uint64_t)r * kLanes];
    const uint32_t c[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
    const bool b = r < tr.tile;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bef[i] += b ? c[i] : 0u;
      aft[i] += b ? 0u : c[i];
    }
  }
#pragma unroll
  for (uint32_t off = kLanes; off < 64; off <<= 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bef[i] += (uint32_t)__shfl_xor((int)bef[i], (int)off);
      aft[i] += (uint32_t)__shfl_xor((int)aft[i], (int)off);
    }
  }
  if (lane < kLanes && w * kRowsPer < tr.T) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      atomicAdd(&L.before[4 * col + i], bef[i]);
      atomicAdd(&L.from[4 * col + i], aft[i]);
    }
  }
}

// Ranks, reorders and writes one tile whose keys and rows are in registers
// (their loads may still be in flight); dstart = the table entry of digit
// threadIdx.x for this tile.  Starts and ends with a barrier.  With kCheck a
// key at or above 2^check_shift sets *reject to 1.  With kFull the tile is
// full (tile_n = kBlock * kItems) and no element is checked against tile_n.
// io.kPacked: no rows are given, an element's row is its position less
// io.row_origin, `base` the tile's first.
// kStarts (see Starts): kGiven uses dstart; kSum adds up the tile rows while the
// keys are on their way, beside the ranking; kScanned has the sums in tr.
template <int kBlock, int kItems, bool kCheck = false, bool kTag = false, int kBits = kRadixBits, bool kFull = false,
          int kStarts = 0, class IO>
__device__ __forceinline__ void scatter_tile(ScatterLds<kBlock, kItems, IO::kPacked>& L, const IO& io, uint32_t base,
                                             uint32_t shift,
                                             uint32_t tile_n, uint32_t dstart, const uint32_t (&key)[kItems],
                                             const uint32_t (&row)[kItems], uint32_t check_shift = 32,
                                             uint32_t* reject = nullptr, const TileRows& tr = {}) {
  constexpr int kWaves = kBlock / 64;
  static_assert(kBits >= 2 && kBits <= kRadixBits && kBits % 2 == 0, "digit widths 2, 4, 6, 8");
  constexpr uint32_t kMask = (1u << kBits) - 1u;
  const uint32_t tid = threadIdx.x, w = tid / 64, lane = lane_id();
  const uint32_t wbase = w * 64 * kItems;
  for (int i = tid; i < kWaves * kRadix; i += kBlock) (&L.wcnt[0][0])[i] = 0;
  // 8-bit digits: per-wave digit masks, in the reorder buffer (unused until
  // the reorder).
  constexpr bool kMaskRank = kBits == kRadixBits;
  uint64_t* dmask = reinterpret_cast<uint64_t*>(&L.kr[0]) + w * kRadix;
  if (kMaskRank)
    for (int j = lane; j < kRadix; j += 64) dmask[j] = 0ull;
  if (kStarts == kSum && tid < kRadix) L.before[tid] = L.from[tid] = 0u;
  __syncthreads();
  if (kStarts == kSum) add_rows<kBlock, kBits>(tr, L);
  uint32_t before = tr.before;
  if (kStarts == kScanned && tid < (1u << kBits)) {  // the rows between the scanned one and this tile's
#pragma unroll
    for (uint32_t r = 0; r + 1 < kRowGroup; ++r)
      if (r < tr.T) before += tr.rows[grouped_digit(r, tid)];
  }

  // ---- rank inside the wave: peers = lanes with the same digit ----------------
  // 8-bit digits: digits 0 and 1, the most frequent ones on small values, by
  // one ballot each; every other digit by its mask: the lanes holding it OR
  // their bits into it, read it back and clear it (three LDS operations of the
  // one wave, executed in order; OR commutes, so the mask is exact whatever
  // order the lanes are served in).  That costs fewer instructions than a
  // ballot per digit bit (≈30 per key), and the scatter is bound by
  // instruction issue: 347 -> 330 us per 2^26 pair sort over 16-bit Zipf keys,
  // the same on uniform ones (ballots for digit 0 alone: 334 us; for 0..3:
  // 340 us).  Narrower digits take the ballots (3 rounds for 6 bits), which are
  // cheaper there: the batched build's 6-bit passes ran 1.3% slower with the
  // masks.
  const uint64_t mybit = 1ull << lane;
  // Clustered keys: many lanes that OR one mask are served one by one (6,000,011
  // clustered 16-bit values: 35 us a pass, 21 with the digits of runs taken by
  // ballot).  Seen by the wave's first step, whose first lane's digit then fills
  // a quarter of the wave or more; a step of theirs takes two digits, its first
  // lane's and the next one's, by ballot as well.  (Two loops: a branch in every
  // step of one cost random keys 2% of the pass.)
  uint32_t rank[kItems];
  auto rank_step = [&](int i, bool clustered) __attribute__((always_inline)) {
    const bool valid = (kFull || wbase + i * 64 + lane < tile_n);
    const uint32_t d = (key[i] >> shift) & kMask;
    uint32_t r = 0;
    uint64_t peers;
    if (kMaskRank) {
      const uint64_t b0 = __builtin_amdgcn_ballot_w64(valid && d == 0u);
      const uint64_t b1 = __builtin_amdgcn_ballot_w64(valid && d == 1u);
      peers = d == 0u ? b0 : b1;
      bool masked = valid && d > 1u;
      if (clustered) {
        const uint32_t df = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const uint64_t bf = __builtin_amdgcn_ballot_w64(valid && d == df);
        uint64_t rest = __builtin_amdgcn_ballot_w64(masked) & ~bf;
        if (d == df) peers = bf;
        if (rest) {
          const uint32_t dn = (uint32_t)__builtin_amdgcn_readlane((int)d, (int)__builtin_ctzll(rest));
          const uint64_t bn = __builtin_amdgcn_ballot_w64(valid && d == dn);
          if (d == dn) peers = bn;
          rest &= ~bn;
        }
        masked = (rest >> lane) & 1ull;
      }
      if (masked) {
        __hip_atomic_fetch_or(&dmask[d], mybit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        peers = __hip_atomic_load(&dmask[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        __hip_atomic_store(&dmask[d], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
    } else {
      // the valid lanes whose digit equals this lane's, i.e. that differ from
      // it in no digit bit (kBits / 2 bit pairs)
      uint32_t diff_lo = 0, diff_hi = 0;
      differing_lanes<0>(d, diff_lo, diff_hi);
      if (kBits > 2) differing_lanes<2>(d, diff_lo, diff_hi);
      if (kBits > 4) differing_lanes<4>(d, diff_lo, diff_hi);
      peers = __builtin_amdgcn_ballot_w64(valid) & ~(((uint64_t)diff_hi << 32) | diff_lo);
    }
    if (valid) {
      const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
      const uint32_t old = L.wcnt[w][d];
      if (below == 0) L.wcnt[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
      r = old + below;
    }
    rank[i] = r;
  };
  bool clustered = false;
  if (kMaskRank) {
    const uint32_t d0 = (key[0] >> shift) & kMask, df = (uint32_t)__builtin_amdgcn_readfirstlane((int)d0);
    clustered = df > 1u && __popcll(__builtin_amdgcn_ballot_w64(d0 == df)) >= 16;  // uniform
  }
  if (kMaskRank && clustered) {
#pragma unroll
    for (int i = 0; i < kItems; ++i) rank_step(i, true);
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) rank_step(i, false);
  }
  if (kCheck) {
    uint32_t over = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      over |= ((kFull || wbase + i * 64 + lane < tile_n)) ? key[i] >> check_shift : 0u;
    if (__ballot(over != 0u) && lane == 0) *reject = 1u;
  }
  __syncthreads();

  // ---- per digit: tile-local offsets and global destinations ------------------
  uint32_t tile_count = 0;
  if (tid < kRadix) {
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      const uint32_t c = L.wcnt[ww][tid];
      L.wcnt[ww][tid] = (uint16_t)tile_count;
      tile_count += c;
    }
  }
  uint32_t total;
  if (kStarts != kGiven) {  // the digits' starts: their totals scanned, then this tile's share of its digit
    uint32_t bef = before, all = tr.total;
    if (kStarts == kSum) {
      bef = tid < (1u << kBits) ? L.before[tid] : 0u;
      all = bef + (tid < (1u << kBits) ? L.from[tid] : 0u);
    }
    dstart = tr.origin + bef + block_excl_scan<kBlock>(all, L.scan2, &total);
  }
  const uint32_t loff = block_excl_scan<kBlock>(tid < kRadix ? tile_count : 0u, L.scan, &total);
  // Each wave's start of each digit in the tile: the digit's tile-local start
  // added to its per-wave offsets here, once per (wave, digit), so the reorder
  // reads one LDS word per key instead of two (2^26 Zipf sort: -5 us).
  if (tid < kRadix) {
    L.dbase[tid] = dstart - loff;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) L.wcnt[ww][tid] = (uint16_t)(L.wcnt[ww][tid] + loff);
  }
  __syncthreads();

  // ---- reorder the tile by digit in LDS ---------------------------------------
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    if ((kFull || wbase + i * 64 + lane < tile_n)) {
      const uint32_t d = (key[i] >> shift) & kMask;
      const uint32_t pos = L.wcnt[w][d] + rank[i];
      if (IO::kPacked)
        L.words()[pos] = key[i] << 16 | (wbase + i * 64 + lane);  // a key above 16 bits voids the result
      else
        L.pairs()[pos] = make_uint2(key[i], row[i]);
    }
  }
  __syncthreads();

  // ---- write each digit's run to its global place ------------------------------
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const uint32_t p = i * kBlock + tid;
    if (kFull || p < tile_n) {
      uint32_t k, r;
      if (IO::kPacked) {
        const uint32_t v = L.words()[p];
        k = v >> 16;
        r = base - io.row_origin + (v & 0xFFFFu);
      } else {
        const uint2 v = L.pairs()[p];
        k = v.x;
        r = v.y;
      }
      const uint32_t g = L.dbase[(k >> shift) & kMask] + p;
      io.dst_keys[g] = (std::remove_pointer_t<decltype(io.dst_keys)>)(kTag ? (k & io.key_and) | io.key_or : k);
      io.dst_rows[g] = r;
    }
  }
  __syncthreads();  // the LDS buffers are free again
}

// ---------------------------------------------------------------------------------
// the kernels of a pass
// ---------------------------------------------------------------------------------
// Column prefixes of the rows: pre[t / kRowGroup][d] = the counts of digit d in
// the tiles before t, totals[d] those in all T.  Bound by latency, and with many
// tiles by the work-items' scattered loads: a work-group takes 4 kCols digits, a
// work-item four of them in a kChunks-th part of the groups -- two 16-byte loads
// a group -- which it adds up, the sums are scanned over the parts in LDS, and it
// writes its prefixes, from the groups it holds (the first kHeld) or reads again.
// With rows one after the other (an 8-byte load a row) 8192 tiles took 12.8 us
// instead of 6.8, and any other number 0.2 to 2 us more.
// With plan a skipped pass leaves at once; with plan_out (the first pass)
// work-group 0 forms the plan from the tiles' OR and AND.
// Against a digit-major table (a strided write by every count, a look-back scan
// of 256 entries per tile, a gather by every scatter, a launch for the plan), us
// of kernels a request: 4,200,000 values of 12 bits 81.5 -> 74.5, of 31 bits 181.9
// -> 172.5; 2^24 of 12 bits 182.0 -> 174.8; 2^26 of 16 bits 689 -> 671 (counts
// 51.1 + 42.1 -> 45.4 + 35.8, scan 7.0 -> 6.8, scatters 162.7 + 180.0 -> 156.9 +
// 179.4).
template <int kBits, int kCols>
__global__ __launch_bounds__(1024) void k_rows_scan(const uint16_t* __restrict__ rows, uint32_t T,
                                                    uint32_t* __restrict__ pre, uint32_t* __restrict__ totals,
                                                    const SortPlan* __restrict__ plan, uint32_t pass,
                                                    const uint32_t* __restrict__ orand, SortPlan* __restrict__ plan_out) {
  constexpr uint32_t kD = 1u << kBits, kChunks = 1024 / kCols, kGroups = kD / 4 / kCols, kHeld = 2;
  __shared__ uint32_t s_sum[4 * kCols][kChunks];
  __shared__ uint32_t s_or[16], s_and[16];
  const uint32_t tid = threadIdx.x, w = tid / 64, lane = lane_id();
  if (plan && !((plan->active >> pass) & 1u)) return;
  if (plan_out && blockIdx.x == 0) {
    uint32_t o, a;
    block_or_and<1024>(orand, T, s_or, s_and, &o, &a);
    if (tid == 0) {
      plan_out->active = active_passes(o, a);
      plan_out->keys_or = o;
    }
  }
  // work-groups of one XCD take neighbouring digits, so that they share lines in its L2
  const uint32_t wg = kGroups >= 8 ? blockIdx.x % 8 * (kGroups / 8) + blockIdx.x / 8 : blockIdx.x;
  const uint32_t c = tid % kCols, chunk = tid / kCols, col = wg * kCols + c;
  const uint32_t G = (T + kRowGroup - 1) / kRowGroup, per = (G + kChunks - 1) / kChunks;
  const uint32_t g0 = min(G, chunk * per), g1 = min(G, g0 + per);
  const u32x4* src = reinterpret_cast<const u32x4*>(rows) + 2 * col;
  // the sums over a group's rows, digits packed in pairs (four counts of up to 8192 in 16 bits)
  const auto load = [&](uint32_t g) {
    u32x4 lo = src[(uint64_t)g * (kD / 2)], hi = src[(uint64_t)g * (kD / 2) + 1];
    if (g == G - 1) {  // the last group: rows from T on don't exist
      const uint32_t left = T - g * kRowGroup;
      if (left < 2) lo.z = lo.w = 0u;
      if (left < 3) hi.x = hi.y = 0u;
      if (left < 4) hi.z = hi.w = 0u;
    }
    return make_uint2(lo.x + lo.z + hi.x + hi.z, lo.y + lo.w + hi.y + hi.w);
  };
  uint32_t sum[4] = {0, 0, 0, 0};
  uint2 held[kHeld];
#pragma unroll
  for (uint32_t i = 0; i < kHeld; ++i) held[i] = g0 + i < g1 ? load(g0 + i) : make_uint2(0u, 0u);
#pragma unroll
  for (uint32_t i = 0; i < kHeld; ++i) {
    const uint2 v = held[i];
    sum[0] += v.x & 0xFFFFu, sum[1] += v.x >> 16, sum[2] += v.y & 0xFFFFu, sum[3] += v.y >> 16;
  }
#pragma unroll 4
  for (uint32_t g = g0 + kHeld; g < g1; ++g) {
    const uint2 v = load(g);
    sum[0] += v.x & 0xFFFFu, sum[1] += v.x >> 16, sum[2] += v.y & 0xFFFFu, sum[3] += v.y >> 16;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s_sum[4 * c + i][chunk] = sum[i];
  __syncthreads();
  if (w < 4 * kCols) {  // a wave per digit
    constexpr uint32_t kLane = kChunks / 64;
    uint32_t x[kLane], t = 0;
#pragma unroll
    for (uint32_t i = 0; i < kLane; ++i) {
      x[i] = t;
      t += s_sum[w][lane * kLane + i];
    }
    const uint32_t inc = wave_incl_scan(t);
#pragma unroll
    for (uint32_t i = 0; i < kLane; ++i) s_sum[w][lane * kLane + i] = inc - t + x[i];
    if (lane == 63) totals[wg * 4 * kCols + w] = inc;
  }
  __syncthreads();
  u32x4 run;
  run.x = s_sum[4 * c][chunk], run.y = s_sum[4 * c + 1][chunk];
  run.z = s_sum[4 * c + 2][chunk], run.w = s_sum[4 * c + 3][chunk];
  u32x4* dst = reinterpret_cast<u32x4*>(pre) + col;
#pragma unroll
  for (uint32_t i = 0; i < kHeld; ++i) {
    const uint2 v = held[i];
    if (g0 + i < g1) dst[(uint64_t)(g0 + i) * (kD / 4)] = run;
    run.x += v.x & 0xFFFFu, run.y += v.x >> 16, run.z += v.y & 0xFFFFu, run.w += v.y >> 16;
  }
#pragma unroll 4
  for (uint32_t g = g0 + kHeld; g < g1; ++g) {
    const uint2 v = load(g);
    dst[(uint64_t)g * (kD / 4)] = run;
    run.x += v.x & 0xFFFFu, run.y += v.x >> 16, run.z += v.y & 0xFFFFu, run.w += v.y >> 16;
  }
}

// A pass's rows and, with kScanned, their prefixes and totals.
struct RowTable {
  const uint16_t* rows;
  const uint32_t *pre, *totals;
};

// This tile's part of it.
template <int kStarts, int kBits>
__device__ __forceinline__ TileRows tile_rows(const RowTable& rt, uint32_t ntiles, uint32_t tile) {
  if (kStarts == kSum) return TileRows{rt.rows, ntiles, tile, 0u, 0u, 0u};
  const uint32_t group = tile / kRowGroup;
  TileRows tr{rt.rows + ((uint64_t)group * kRowGroup << kBits), tile % kRowGroup, tile, 0u, 0u, 0u};
  if (threadIdx.x < (1u << kBits)) {
    tr.before = rt.pre[((uint64_t)group << kBits) + threadIdx.x];
    tr.total = rt.totals[threadIdx.x];
  }
  return tr;
}

// Counts of one tile into its row.  The first pass also zeroes the encoder's
// look-back words and *reject, and (kOrAnd) records the OR and AND of the
// tile's keys.
template <int kBlock, int kItems, int kRounds, bool kGrouped, class SK>
__global__ __launch_bounds__(kBlock) void k_radix_count_fixed(const SK* __restrict__ keys, uint16_t* __restrict__ rows,
                                                       uint32_t shift, uint32_t bits, uint32_t n_cap, uint32_t ntiles,
                                                       uint32_t* __restrict__ reject,
                                                       const uint64_t* __restrict__ d_n, ClearWords cw) {
  constexpr int kTile = kBlock * kItems;
  clear_words(cw);
  if (reject && blockIdx.x == 0 && threadIdx.x == 0) *reject = 0u;
  const uint32_t tile = xcd_tile(blockIdx.x, ntiles);
  uint16_t* const row = rows + ((uint64_t)(kGrouped ? tile / kRowGroup * kRowGroup : tile) << bits);
  upsweep_tile<kBlock, kTile, kRounds, false>(
      keys, shift, tile * kTile, tile_len(tile, kTile, n_cap, d_n),
      [&](uint32_t d, uint32_t c) {
        if (d >> bits == 0u) row[kGrouped ? grouped_digit(tile, d) : d] = (uint16_t)c;
      },
      tile, nullptr, (1u << bits) - 1u);
}

template <int kBlock, int kItems, int kStarts, bool kCheck, int kBits, class SK, class DK>
__global__ __launch_bounds__(kBlock, 8) void k_radix_scatter_fixed(PassIoT<SK, DK> io, RowTable rt,
                                                         uint32_t shift, uint32_t n_cap, uint32_t ntiles,
                                                         uint32_t check_shift, uint32_t* __restrict__ reject,
                                                         const uint64_t* __restrict__ d_n) {
  constexpr int kTile = kBlock * kItems;
  __shared__ ScatterLds<kBlock, kItems, PassIoT<SK, DK>::kPacked> L;
  const uint32_t tile = xcd_tile(blockIdx.x, ntiles);
  const uint32_t base = tile * kTile;
  const uint32_t tile_n = tile_len(tile, kTile, n_cap, d_n);
  if (tile_n == 0) return;  // past a device-resident count
  const TileRows tr = tile_rows<kStarts, kBits>(rt, ntiles, tile);
  uint32_t key[kItems], row[kItems];
  scatter_load<kBlock, kItems>(io, base, tile_n, key, row);
  if (tile_n == (uint32_t)kTile)  // uniform: a full tile checks no element against its length
    scatter_tile<kBlock, kItems, kCheck, false, kBits, true, kStarts>(L, io, base, shift, tile_n, 0u, key, row, check_shift,
                                                                   reject, tr);
  else
    scatter_tile<kBlock, kItems, kCheck, false, kBits, false, kStarts>(L, io, base, shift, tile_n, 0u, key, row, check_shift,
                                                                    reject, tr);
}

// Plan-driven passes over uint32 keys (8-bit digits).  With kSum the first
// scatter forms the plan from the tiles' OR and AND in every work-group, and
// work-group 0 stores it for the later launches.
template <bool kFirst, int kBlock, int kItems, bool kGrouped>
__global__ __launch_bounds__(kBlock) void k_radix_count(PassBuffers buf, const SortPlan* __restrict__ plan,
                                                            uint16_t* __restrict__ rows, uint32_t* __restrict__ orand,
                                                            uint32_t pass, uint32_t n_cap, uint32_t ntiles,
                                                            const uint64_t* __restrict__ d_n, ClearWords cw) {
  constexpr int kTile = kBlock * kItems;
  const uint32_t* keys = buf.keys_in;
  if (kFirst) clear_words(cw);
  if (!kFirst) {
    const uint32_t active = plan->active;
    if (!((active >> pass) & 1u)) return;  // uniform over the grid
    keys = pass_io(buf, active, pass).src_keys;
  }
  const uint32_t tile = xcd_tile(blockIdx.x, ntiles);
  uint16_t* const row = rows + (uint64_t)(kGrouped ? tile / kRowGroup * kRowGroup : tile) * kRadix;
  upsweep_tile<kBlock, kTile, kFirst ? 1 : -1, kFirst>(
      keys, pass * kRadixBits, tile * kTile, tile_len(tile, kTile, n_cap, d_n),
      [&](uint32_t d, uint32_t c) { row[kGrouped ? grouped_digit(tile, d) : d] = (uint16_t)c; }, tile, orand);
}

template <bool kFirst, int kStarts, int kBlock, int kItems>
__global__ __launch_bounds__(kBlock, kItems <= 8 ? 8 : 4) void k_radix_scatter(
    PassBuffers buf, SortPlan* __restrict__ plan, RowTable rt, const uint32_t* __restrict__ orand, uint32_t pass,
    uint32_t n_cap, uint32_t ntiles, const uint64_t* __restrict__ d_n) {
  constexpr int kTile = kBlock * kItems;
  __shared__ ScatterLds<kBlock, kItems> L;
  uint32_t active;
  if (kFirst && kStarts == kSum) {
    uint32_t o, a;
    block_or_and<kBlock>(orand, ntiles, L.scan, reinterpret_cast<uint32_t*>(&L.kr[0]), &o, &a);
    active = active_passes(o, a);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      plan->active = active;
      plan->keys_or = o;
    }
    __syncthreads();  // L is free again
  } else {
    active = plan->active;
  }
  if (!((active >> pass) & 1u)) return;
  const PassIo io = pass_io(buf, active, pass);
  const uint32_t tile = xcd_tile(blockIdx.x, ntiles);
  const uint32_t base = tile * kTile;
  const uint32_t tile_n = tile_len(tile, kTile, n_cap, d_n);
  if (tile_n == 0) return;  // past a device-resident count
  const TileRows tr = tile_rows<kStarts, kRadixBits>(rt, ntiles, tile);
  uint32_t key[kItems], row[kItems];
  scatter_load<kBlock, kItems>(io, base, tile_n, key, row);
  if (tile_n == (uint32_t)kTile)
    scatter_tile<kBlock, kItems, false, false, kRadixBits, true, kStarts>(L, io, base, pass * kRadixBits, tile_n, 0u, key, row,
                                                                       32u, nullptr, tr);
  else
    scatter_tile<kBlock, kItems, false, false, kRadixBits, false, kStarts>(L, io, base, pass * kRadixBits, tile_n, 0u, key, row,
                                                                        32u, nullptr, tr);
}

}  // namespace

namespace {

// ---------------------------------------------------------------------------------
// the segmented sort: a batch of requests, keys sorted inside each request
// ---------------------------------------------------------------------------------
// Request j owns positions [req_off[j], req_off[j+1]); its tiles are its
// positions cut at the multiples of kTile, so tile l of request j covers
// [max(req_off[j], (c0 + l) kTile), min(req_off[j+1], (c0 + l + 1) kTile)) with
// c0 = req_off[j] / kTile (whole tiles stay aligned).  tile_base[j] is the
// number of tiles of the requests before j, tile_req[t] the request of tile t
// (~0 from the last tile on; looking it up by search in every work-group and
// launch took 9 dependent loads of 192 requests).  The digit counts are kept
//  * as a table, request j's at 256 tile_base[j] + d ntiles_j + l: scanned in
//    that order, each entry is the position in the batch of the tile's first
//    key with digit d, and no key leaves its request; or
//  * as rows (see k_radix_count_fixed), of which a tile sums its own request's, in
//    batches of few tiles or of requests of few (see seg_sort).
// Rows are made relative to the request's first position; the last pass writes
// the key tagged with its request (j << value_bits | key), which is what the
// encoder and the per-request split read.
template <int kTile>
__device__ __forceinline__ uint32_t request_tiles(const uint32_t* __restrict__ req_off, uint32_t j) {
  const uint32_t r0 = req_off[j], r1 = req_off[j + 1];
  return r1 > r0 ? (r1 + (uint32_t)kTile - 1u) / (uint32_t)kTile - r0 / (uint32_t)kTile : 0u;
}

// The layout of up to kSegLayoutMax requests by one work-group: tile_base,
// tile_req (ub entries), the table's length, the cleared flags.  One launch for
// three, but its waves take the requests in turn: us a batch of 12-bit values by
// three launches / by this one, 192 requests of 20,000 values 118 / 113, 512 of
// 1100 89 / 84, 1024 110 / 109, 2048 152 / 160 (of 5000 values 259 / 270), 4096 242
// / 269, 8192 405 / 463.
constexpr uint32_t kSegLayoutMax = 1024;
template <int kTile>
__global__ __launch_bounds__(1024) void k_seg_layout(const uint32_t* __restrict__ req_off, uint32_t nreq, uint32_t ub,
                                                     uint32_t* __restrict__ tile_base, uint32_t* __restrict__ tile_req,
                                                     uint64_t* __restrict__ tlen, uint32_t* __restrict__ bad,
                                                     uint32_t* __restrict__ req_bad) {
  static_assert(kSegLayoutMax == 1024, "a request per work-item");
  __shared__ uint32_t s_scan[16], s_base[kSegLayoutMax];
  const uint32_t tid = threadIdx.x;
  uint32_t nt = 0, all;
  if (tid < nreq) {
    nt = request_tiles<kTile>(req_off, tid);
    if (req_bad) req_bad[tid] = 0u;
  }
  const uint32_t base = block_excl_scan<1024>(nt, s_scan, &all);
  if (tid < nreq) tile_base[tid] = base;
  s_base[tid] = base;
  __syncthreads();
  for (uint32_t q = tid / 64; q < nreq; q += 16) {  // a wave per request
    const uint32_t t1 = min(q + 1 < nreq ? s_base[q + 1] : all, ub);
    for (uint32_t t = s_base[q] + lane_id(); t < t1; t += 64) tile_req[t] = q;
  }
  if (tid == 0) {
    tile_base[nreq] = all;
    *tlen = (uint64_t)kRadix * all;
    *bad = 0u;
  }
  for (uint32_t t = all + tid; t < ub; t += 1024) tile_req[t] = ~0u;
}

// The same for more requests: the tile counts (scanned by the launch between),
// then a wave per request.
template <int kTile>
__global__ __launch_bounds__(256) void k_seg_tiles(const uint32_t* __restrict__ req_off, uint32_t nreq,
                                                   uint32_t* __restrict__ ntiles) {
  for (uint32_t j = blockIdx.x * 256 + threadIdx.x; j <= nreq; j += gridDim.x * 256)
    ntiles[j] = j < nreq ? request_tiles<kTile>(req_off, j) : 0u;
}

__global__ __launch_bounds__(256) void k_seg_map(const uint32_t* __restrict__ tile_base, uint32_t nreq, uint32_t ub,
                                                 uint32_t* __restrict__ tile_req, uint64_t* __restrict__ tlen,
                                                 uint32_t* __restrict__ bad, uint32_t* __restrict__ req_bad) {
  const uint32_t first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  for (uint32_t j = first / 64; j < nreq; j += stride / 64) {
    const uint32_t t1 = min(tile_base[j + 1], ub);
    for (uint32_t t = tile_base[j] + lane_id(); t < t1; t += 64) tile_req[t] = j;
    if (req_bad && lane_id() == 0) req_bad[j] = 0u;
  }
  const uint32_t all = tile_base[nreq];
  for (uint64_t t = (uint64_t)all + first; t < ub; t += stride) tile_req[t] = ~0u;
  if (first == 0) {
    *tlen = (uint64_t)kRadix * all;
    *bad = 0u;
  }
}

struct SegTile {
  uint32_t j, l, base, len, nt;
};

// Tile t of request j.
template <int kTile>
__device__ __forceinline__ SegTile seg_tile(const uint32_t* __restrict__ req_off, const uint32_t* __restrict__ tile_base,
                                            uint32_t j, uint32_t t) {
  SegTile s;
  s.j = j;
  s.l = t - tile_base[j];
  s.nt = tile_base[j + 1] - tile_base[j];
  const uint32_t r0 = req_off[j], r1 = req_off[j + 1], c0 = r0 / (uint32_t)kTile;
  s.base = max(r0, (c0 + s.l) * (uint32_t)kTile);
  s.len = min(r1, (c0 + s.l + 1u) * (uint32_t)kTile) - s.base;
  return s;
}

// The batch's tiles on the device, and where the counts are (one of the two).
struct Segments {
  const uint32_t *req_off, *tile_base, *tile_req;
  uint32_t ub;        // tiles at most
  uint32_t* table;    // digit-major per request
  uint16_t* rows;     // 1 << bits counts per tile
};

template <int kTile, int kRounds, bool kRows, class SK>
__global__ __launch_bounds__(kUpBlock) void k_seg_count(const SK* __restrict__ keys, Segments sg, uint32_t shift,
                                                        uint32_t bits, ClearWords cw) {
  clear_words(cw);
  const uint32_t t = xcd_tile(blockIdx.x, sg.ub), j = sg.tile_req[t];
  if (j == ~0u) return;  // uniform over the work-group
  const SegTile s = seg_tile<kTile>(sg.req_off, sg.tile_base, j, t);
  uint32_t* const part = sg.table + (uint64_t)kRadix * (t - s.l) + s.l;
  uint16_t* const row = sg.rows + ((uint64_t)t << bits);
  upsweep_tile<kUpBlock, kTile, kRounds, false>(
      keys, shift, s.base, s.len,
      [&](uint32_t d, uint32_t c) {
        if (!kRows)
          part[(uint64_t)d * s.nt] = c;
        else if (d >> bits == 0u)
          row[d] = (uint16_t)c;
      },
      t, nullptr, (1u << bits) - 1u);
}

// offs: the scanned table (not with kRows).  kCheck (the first pass): a key at
// or above 2^value_bits flags its request (req_bad[j]) or, without req_bad, the
// batch (*bad).  kTag (the last pass): keys are written as j << value_bits |
// key.
template <int kBlock, int kItems, bool kCheck, bool kTag, bool kRows, int kBits, class SK, class DK>
__global__ __launch_bounds__(kBlock, 8) void k_seg_scatter(PassIoT<SK, DK> io, Segments sg,
                                                           const uint32_t* __restrict__ offs, uint32_t shift,
                                                           uint32_t value_bits, uint32_t* __restrict__ bad,
                                                           uint32_t* __restrict__ req_bad) {
  constexpr int kTile = kBlock * kItems;
  __shared__ ScatterLds<kBlock, kItems, PassIoT<SK, DK>::kPacked> L;
  const uint32_t t = xcd_tile(blockIdx.x, sg.ub), j = sg.tile_req[t];
  if (j == ~0u) return;  // uniform over the work-group
  const SegTile s = seg_tile<kTile>(sg.req_off, sg.tile_base, j, t);
  const uint32_t dstart = !kRows && threadIdx.x < kRadix
                              ? offs[(uint64_t)kRadix * (t - s.l) + (uint64_t)threadIdx.x * s.nt + s.l]
                              : 0u;
  io.row_origin = sg.req_off[j];
  if (kTag) {
    io.key_and = value_bits < 32 ? (1u << value_bits) - 1u : ~0u;
    io.key_or = value_bits < 32 ? j << value_bits : 0u;
  }
  uint32_t key[kItems], row[kItems];
  scatter_load<kBlock, kItems>(io, s.base, s.len, key, row);
  uint32_t* const flag = req_bad ? req_bad + j : bad;
  const TileRows tr{sg.rows + ((uint64_t)(t - s.l) << kBits), s.nt, s.l, io.row_origin, 0u, 0u};
  if (s.len == (uint32_t)kTile)  // uniform: a full tile checks no element against its length
    scatter_tile<kBlock, kItems, kCheck, kTag, kBits, true, kRows ? kSum : kGiven>(L, io, s.base, shift, s.len, dstart, key, row, value_bits,
                                                                   flag, tr);
  else
    scatter_tile<kBlock, kItems, kCheck, kTag, kBits, false, kRows ? kSum : kGiven>(L, io, s.base, shift, s.len, dstart, key, row, value_bits,
                                                                    flag, tr);
}

// Digits of a fixed-pass sort of values below 2^value_bits (value_bits 1..16):
// pass p ranks `bits` bits from `shift` on.  The byte split takes 8 bits, then
// the rest; the even split halves value_bits.  Widths are rounded up to even
// (the ranking takes the bits in pairs): bits above value_bits are 0 in every
// key that passes the range check, and a key that fails it is flagged and its
// result discarded, so masking them only keeps its ranks in range.
struct DigitSplit {
  uint32_t passes;
  uint32_t shift[2], bits[2];
};

DigitSplit digit_split(uint32_t value_bits, bool even) {
  auto up2 = [](uint32_t b) { return (b + 1u) & ~1u; };
  DigitSplit d{};
  d.passes = (value_bits + kRadixBits - 1) / kRadixBits;
  if (d.passes == 1) {
    d.shift[0] = 0;
    d.bits[0] = up2(value_bits);
    return d;
  }
  const uint32_t b0 = even ? up2((value_bits + 1) / 2) : (uint32_t)kRadixBits;
  d.shift[0] = 0;
  d.bits[0] = b0;
  d.shift[1] = b0;
  d.bits[1] = up2(value_bits - b0);
  return d;
}

// Scratch of a pass's rows; the prefixes too if they are scanned.
struct RowScratch {
  uint16_t* rows = nullptr;
  uint32_t *pre = nullptr, *totals = nullptr;
  bool ok = false;
  RowScratch(Env& env, uint32_t ntiles, bool scanned) {
    const uint64_t groups = ((uint64_t)ntiles + kRowGroup - 1) / kRowGroup;
    rows = static_cast<uint16_t*>(env.scratch(groups * kRowGroup * kRadix * 2));
    if (scanned) {
      pre = static_cast<uint32_t*>(env.scratch(groups * kRadix * 4));
      totals = static_cast<uint32_t*>(env.scratch(kRadix * 4));
    }
    ok = rows && (!scanned || (pre && totals));
  }
  RowTable table() const { return {rows, pre, totals}; }
};

// Beyond 2048 tiles a work-group takes 4 digits instead of 16: us with 4 / 16 digits
// of 6 bits 1024 tiles 3.9 / 4.3, 2048 4.6 / 4.8, 4096 4.9 / 5.3, 8192 7.4 / 9.5; of
// 8 bits 4.6 / 4.3, 4.6 / 4.8, 5.0 / 5.4, 7.1 / 9.1.
int scan_rows(Env& env, const RowScratch& rs, uint32_t bits, uint32_t ntiles, const SortPlan* plan, uint32_t pass,
              const uint32_t* orand, SortPlan* plan_out) {
  env.prof_begin("radix_rows_scan");
#define KA_ROWS_SCAN(B, C) \
  k_rows_scan<B, C><<<dim3((1u << B) / 4 / C), dim3(1024), 0, env.stream()>>>(rs.rows, ntiles, rs.pre, \
                                                                              rs.totals, plan, pass, orand, plan_out)
  switch (bits) {
    case 2:
      KA_ROWS_SCAN(2, 1);
      break;
    case 4:
      KA_ROWS_SCAN(4, 4);
      break;
    case 6:
      if (ntiles <= 2048)
        KA_ROWS_SCAN(6, 4);
      else
        KA_ROWS_SCAN(6, 1);
      break;
    default:
      if (ntiles <= 2048)
        KA_ROWS_SCAN(8, 4);
      else
        KA_ROWS_SCAN(8, 1);
      break;
  }
#undef KA_ROWS_SCAN
  env.prof_end("radix_rows_scan");
  return check_launch(env, "radix_rows_scan launch");
}

// One pass of the narrow-key sort.  A scanned sort's counts come from 256
// work-items a tile: they stream, where those of few tiles wait.
template <int kBlock, int kItems, int kStarts, bool kCheck, class SK, class DK>
int rows_pass16(Env& env, const PassIoT<SK, DK>& io, const RowScratch& rs, uint32_t shift, uint32_t bits, uint32_t nn,
                uint32_t ntiles, uint32_t check_shift, uint32_t* reject, const uint64_t* d_n, ClearWords cw) {
  constexpr int kCount = kStarts == kScanned ? 256 : kBlock;
  const dim3 g(ntiles), b(kBlock);
  env.prof_begin(kCheck ? "radix_upsweep0" : "radix_upsweep");
  k_radix_count_fixed<kCount, kBlock * kItems / kCount, kCheck ? 1 : -1, kStarts == kScanned, SK>
      <<<g, dim3(kCount), 0, env.stream()>>>(io.src_keys, rs.rows, shift, bits, nn, ntiles, reject, d_n, cw);
  env.prof_end(kCheck ? "radix_upsweep0" : "radix_upsweep");
  int rc = check_launch(env, "radix_count launch");
  if (rc) return rc;
  if (kStarts == kScanned && (rc = scan_rows(env, rs, bits, ntiles, nullptr, 0, nullptr, nullptr))) return rc;
  env.prof_begin("radix_scatter");
#define KA_ROWS_SCATTER(B)                                     \
  k_radix_scatter_fixed<kBlock, kItems, kStarts, kCheck, B, SK, DK>   \
      <<<g, b, 0, env.stream()>>>(io, rs.table(), shift, nn, ntiles, check_shift, reject, d_n)
  switch (bits) {
    case 2:
      KA_ROWS_SCATTER(2);
      break;
    case 4:
      KA_ROWS_SCATTER(4);
      break;
    case 6:
      KA_ROWS_SCATTER(6);
      break;
    default:
      KA_ROWS_SCATTER(8);
      break;
  }
#undef KA_ROWS_SCATTER
  env.prof_end("radix_scatter");
  return check_launch(env, "radix_scatter launch");
}

// The narrow-key sort: keys below 2^value_bits, value_bits <= 16, rows
// 0..n-1.  ceil(value_bits / 8) fixed passes (no plan, no skipped launches)
// with the even split of digit_split; from the first pass on the keys are
// stored as uint16 (6 bytes per pair instead of 8).  The first pass flags a
// key at or above 2^value_bits in *reject (cleared by its count); the sort's
// output is then unspecified.
template <int kBlock, int kItems, int kStarts>
int rows_sort16(Env& env, const uint32_t* keys, uint16_t* skeys, uint32_t* srows, uint64_t n, uint32_t value_bits,
                uint32_t* reject, const uint64_t* d_n, ClearWords cw) {
  constexpr int kTile = kBlock * kItems;
  const uint32_t ntiles = (uint32_t)((n + kTile - 1) / kTile), nn = (uint32_t)n;
  const DigitSplit ds = digit_split(value_bits, true);
  uint16_t* kb = nullptr;
  uint32_t* rb = nullptr;
  if (ds.passes > 1) {
    kb = static_cast<uint16_t*>(env.scratch(n * 2));
    rb = static_cast<uint32_t*>(env.scratch(n * 4));
    if (!kb || !rb) return env.fail(kErrOom, "radix_sort16: scratch buffers");
  }
  const RowScratch rs(env, ntiles, kStarts == kScanned);
  if (!rs.ok) return env.fail(kErrOom, "radix_sort16: digit rows");
  PassIoT<uint32_t, uint16_t> io0{keys, nullptr, ds.passes > 1 ? kb : skeys, ds.passes > 1 ? rb : srows, true};
  int rc = rows_pass16<kBlock, kItems, kStarts, true>(env, io0, rs, ds.shift[0], ds.bits[0], nn, ntiles, value_bits,
                                                      reject, d_n, cw);
  if (rc || ds.passes == 1) return rc;
  PassIoT<uint16_t, uint16_t> io1{kb, rb, skeys, srows, false};
  return rows_pass16<kBlock, kItems, kStarts, false>(env, io1, rs, ds.shift[1], ds.bits[1], nn, ntiles, 32u, nullptr,
                                                     d_n, ClearWords{});
}

// The plan-driven sort of uint32 keys.
template <int kBlock, int kItems, int kStarts>
int rows_sort32(Env& env, const uint32_t* keys, const uint32_t* rows_in, uint32_t* skeys, uint32_t* srows, uint64_t n,
                const uint64_t* d_n, ClearWords cw) {
  constexpr int kTile = kBlock * kItems, kCount = kStarts == kScanned ? 256 : kBlock;
  SortPlan* plan = reinterpret_cast<SortPlan*>(env.arena()->plan);
  const uint32_t ntiles = (uint32_t)((n + kTile - 1) / kTile), nn = (uint32_t)n;
  PassBuffers buf;
  buf.keys_in = keys;
  buf.rows_in = rows_in;
  buf.keys_a = skeys;
  buf.rows_a = srows;
  buf.keys_b = static_cast<uint32_t*>(env.scratch(n * 4));
  buf.rows_b = static_cast<uint32_t*>(env.scratch(n * 4));
  uint32_t* orand = static_cast<uint32_t*>(env.scratch((uint64_t)ntiles * 2 * 4));
  const RowScratch rs(env, ntiles, kStarts == kScanned);
  if (!buf.keys_b || !buf.rows_b || !orand || !rs.ok) return env.fail(kErrOom, "radix_sort: scratch buffers");
  const dim3 g(ntiles), b(kBlock), bc(kCount);
  for (uint32_t pass = 0; pass < (uint32_t)kPasses; ++pass) {
    const char* name = pass ? "radix_upsweep" : "radix_upsweep0";
    env.prof_begin(name);
    if (pass == 0)
      k_radix_count<true, kCount, kTile / kCount, kStarts == kScanned><<<g, bc, 0, env.stream()>>>(buf, plan, rs.rows, orand, pass, nn,
                                                                                  ntiles, d_n, cw);
    else
      k_radix_count<false, kCount, kTile / kCount, kStarts == kScanned><<<g, bc, 0, env.stream()>>>(buf, plan, rs.rows, orand, pass, nn,
                                                                                   ntiles, d_n, cw);
    env.prof_end(name);
    int rc = check_launch(env, "radix_upsweep launch");
    if (rc) return rc;
    if (kStarts == kScanned &&
        (rc = scan_rows(env, rs, kRadixBits, ntiles, pass ? plan : nullptr, pass, orand, pass ? nullptr : plan)))
      return rc;
    env.prof_begin("radix_scatter");
    if (pass == 0)
      k_radix_scatter<true, kStarts, kBlock, kItems><<<g, b, 0, env.stream()>>>(buf, plan, rs.table(), orand, pass,
                                                                                    nn, ntiles, d_n);
    else
      k_radix_scatter<false, kStarts, kBlock, kItems><<<g, b, 0, env.stream()>>>(buf, plan, rs.table(), orand, pass,
                                                                                     nn, ntiles, d_n);
    env.prof_end("radix_scatter");
    if ((rc = check_launch(env, "radix_scatter launch"))) return rc;
  }
  return kOk;
}

// Tile shape by capacity: about one tile per CU, from 1024 keys up; kNone: the
// rows are scanned.  A scan is two launches and 4 us a pass (three or more a
// request), sums by every tile grow with the square of their number.  An index
// request, us, scanned / summed: 12-bit values (6-bit digits) 2,000,000 63 / 56,
// 3,100,000 74 / 72, 4,100,000 77 / 75, 5,242,880 93 / 97; 16-bit (8-bit digits)
// 2,000,000 67 / 64, 3,100,000 83 / 84, 4,194,304 87 / 94; any uint32 2,000,000
// 125 / 120, 2,500,000 151 / 149, 3,100,000 152 / 157, 4,194,304 161 / 178.
enum class RowShape { kNone, k1024, k2048, k4096, k8192 };
constexpr uint64_t row_tiles_max(uint32_t bits) { return bits > 6 ? 352 : 512; }
RowShape row_shape(uint64_t n, uint32_t bits) {
  if (n <= 256ull * 1024) return RowShape::k1024;
  if (n <= 256ull * 2048) return RowShape::k2048;
  if (n <= 256ull * 4096) return RowShape::k4096;
  if (n <= row_tiles_max(bits) * 8192) return RowShape::k8192;
  return RowShape::kNone;
}

// One pass of the segmented sort.
template <bool kCheck, bool kTag, bool kRows, class SK, class DK>
int seg_pass(Env& env, const PassIoT<SK, DK>& io, const Segments& sg, uint32_t* offs, const uint64_t* tlen,
             uint32_t shift, uint32_t bits, uint32_t value_bits, uint32_t* bad, uint32_t* req_bad, ClearWords cw) {
  constexpr int kBlock = kShapes[0].block, kItems = kShapes[0].items, kTile = kBlock * kItems;
  env.prof_begin(kCheck ? "radix_upsweep0" : "radix_upsweep");
  k_seg_count<kTile, kCheck ? 1 : -1, kRows, SK><<<dim3(sg.ub), dim3(kUpBlock), 0, env.stream()>>>(io.src_keys, sg,
                                                                                                  shift, bits, cw);
  env.prof_end(kCheck ? "radix_upsweep0" : "radix_upsweep");
  int rc = check_launch(env, "seg_count launch");
  if (rc) return rc;
  if (!kRows && (rc = launch_exclusive_scan(env, sg.table, offs, (uint64_t)kRadix * sg.ub, tlen))) return rc;
  env.prof_begin("radix_scatter");
#define KA_SEG_SCATTER(B)                                                                                             \
  k_seg_scatter<kBlock, kItems, kCheck, kTag, kRows, B, SK, DK><<<dim3(sg.ub), dim3(kBlock), 0, env.stream()>>>(       \
      io, sg, offs, shift, value_bits, bad, req_bad)
  switch (bits) {
    case 2:
      KA_SEG_SCATTER(2);
      break;
    case 4:
      KA_SEG_SCATTER(4);
      break;
    case 6:
      KA_SEG_SCATTER(6);
      break;
    default:
      KA_SEG_SCATTER(8);
      break;
  }
#undef KA_SEG_SCATTER
  env.prof_end("radix_scatter");
  return check_launch(env, "seg_scatter launch");
}

template <bool kRows>
int seg_passes(Env& env, const uint32_t* values, const DigitSplit& ds, const Segments& sg, uint32_t* offs,
               const uint64_t* tlen, uint32_t value_bits, uint16_t* kb, uint32_t* rb, uint32_t* skeys, uint32_t* srows,
               uint32_t* bad, uint32_t* req_bad, ClearWords cw) {
  // pass 0: uint32 values in (checked), uint16 keys out -- or tagged keys if it is the only pass
  if (ds.passes == 1)
    return seg_pass<true, true, kRows>(env, PassIoT<uint32_t, uint32_t>{values, nullptr, skeys, srows, true}, sg, offs,
                                       tlen, ds.shift[0], ds.bits[0], value_bits, bad, req_bad, cw);
  const int rc =
      seg_pass<true, false, kRows>(env, PassIoT<uint32_t, uint16_t>{values, nullptr, kb, rb, true}, sg, offs, tlen,
                                   ds.shift[0], ds.bits[0], value_bits, bad, req_bad, cw);
  if (rc) return rc;
  // pass 1: uint16 keys in, tagged uint32 keys out
  return seg_pass<false, true, kRows>(env, PassIoT<uint16_t, uint32_t>{kb, rb, skeys, srows, false}, sg, offs, tlen,
                                      ds.shift[1], ds.bits[1], value_bits, bad, req_bad, ClearWords{});
}

// The segmented sort of a batch (values below 2^value_bits, value_bits <= 16):
// uint16 keys between passes, request-relative rows, tagged uint32 keys out;
// the byte or the even digit split.
int seg_sort(Env& env, const uint32_t* values, uint64_t n, const uint32_t* req_off, uint32_t nreq,
             uint32_t value_bits, uint32_t* skeys, uint32_t* srows, uint32_t* bad, uint32_t* req_bad, bool even,
             uint32_t max_req, ClearWords cw) {
  constexpr int kTile = kShapes[0].block * kShapes[0].items;
  const DigitSplit ds = digit_split(value_bits, even);
  const uint64_t ub64 = (n + kTile - 1) / kTile + nreq;  // tiles: at most one more per request
  if (ub64 >= (1ull << 31)) return env.fail(kErrArg, "segmented sort: too many tiles");
  Segments sg{};
  sg.ub = (uint32_t)ub64;
  sg.req_off = req_off;
  // Rows unless a request has too many tiles to sum (or may have, and the batch
  // has): more than 16 where the last digit has 8 bits, more than 128 below.  Us a
  // batch by the scanned table / by rows, requests of 20,000, 2^17, 2^18, 2^20 and
  // 2^21 values: 1.7 10^7 values of 12 bits 264/257, 224/218, 224/219, 224/219,
  // 225/227; of 14 bits 347/337, 237/236, 235/233, 233/232, 236/240; of 16 bits
  // 416/405, 297/298, 257/259, 241/250, 240/264; of 8 bits 187/180, 162/162,
  // 160/164, 156/164, 158/175.  3 10^6 values (366 tiles) of 16 bits 129/121,
  // 115/107, 109/102, 98/93, 97/93.
  const uint64_t row_request = (ds.bits[ds.passes - 1] > 6 ? 16ull : 128ull) * kTile;
  const bool use_rows = sg.ub <= 384 || max_req <= row_request;
  uint32_t* tile_base = static_cast<uint32_t*>(env.scratch(4ull * (nreq + 1)));
  uint32_t* tile_req = static_cast<uint32_t*>(env.scratch(4ull * sg.ub));
  uint64_t* tlen = static_cast<uint64_t*>(env.scratch(8));
  uint32_t* offs = nullptr;
  if (use_rows) {
    sg.rows = static_cast<uint16_t*>(env.scratch(2ull * kRadix * sg.ub));
  } else {
    sg.table = static_cast<uint32_t*>(env.scratch((uint64_t)kRadix * sg.ub * 4));
    offs = static_cast<uint32_t*>(env.scratch((uint64_t)kRadix * sg.ub * 4));
  }
  uint16_t* kb = ds.passes > 1 ? static_cast<uint16_t*>(env.scratch(2 * n)) : nullptr;
  uint32_t* rb = ds.passes > 1 ? static_cast<uint32_t*>(env.scratch(4 * n)) : nullptr;
  if (!tile_base || !tile_req || !tlen || (use_rows ? !sg.rows : !sg.table || !offs) || (ds.passes > 1 && (!kb || !rb)))
    return env.fail(kErrOom, "segmented sort: scratch");
  sg.tile_base = tile_base;
  sg.tile_req = tile_req;
  int rc;
  env.prof_begin("seg_tiles");
  if (nreq <= kSegLayoutMax) {
    k_seg_layout<kTile><<<dim3(1), dim3(1024), 0, env.stream()>>>(req_off, nreq, sg.ub, tile_base, tile_req, tlen, bad,
                                                                  req_bad);
    env.prof_end("seg_tiles");
    if ((rc = check_launch(env, "seg_layout launch"))) return rc;
  } else {
    uint32_t* ntiles = static_cast<uint32_t*>(env.scratch(4ull * (nreq + 1)));
    if (!ntiles) return env.fail(kErrOom, "segmented sort: scratch");
    k_seg_tiles<kTile><<<dim3(std::min<uint32_t>((nreq + 256) / 256, 1024)), dim3(256), 0, env.stream()>>>(req_off, nreq,
                                                                                                        ntiles);
    env.prof_end("seg_tiles");
    if ((rc = check_launch(env, "seg_tiles launch"))) return rc;
    if ((rc = launch_exclusive_scan(env, ntiles, tile_base, nreq + 1ull, nullptr))) return rc;
    k_seg_map<<<dim3(std::min<uint32_t>(nreq / 4 + 1, 4096)), dim3(256), 0, env.stream()>>>(tile_base, nreq, sg.ub,
                                                                                         tile_req, tlen, bad, req_bad);
    if ((rc = check_launch(env, "seg_map launch"))) return rc;
  }
  return use_rows ? seg_passes<true>(env, values, ds, sg, offs, tlen, value_bits, kb, rb, skeys, srows, bad, req_bad, cw)
                  : seg_passes<false>(env, values, ds, sg, offs, tlen, value_bits, kb, rb, skeys, srows, bad, req_bad,
                                      cw);
}

}  // namespace

int batch_variant_count() { return kNumShapes + 1; }

int launch_radix_sort_segments(Env& env, const uint32_t* values, uint64_t n, const uint32_t* req_off, uint32_t nreq,
                               uint32_t value_bits, uint32_t* skeys, uint32_t* srows, uint32_t* bad,
                               uint32_t* req_bad, bool even_split, uint32_t max_req, ClearWords cw) {
  if (n == 0) return kOk;
  if (!values || !req_off || !skeys || !srows || !bad || nreq == 0)
    return env.fail(kErrArg, "segmented sort: null buffer");
  if (value_bits == 0 || value_bits > 16) return env.fail(kErrArg, "segmented sort: value_bits must be 1..16");
  if (n >= (1ull << 31)) return env.fail(kErrArg, "segmented sort: n must be below 2^31");
  return seg_sort(env, values, n, req_off, nreq, value_bits, skeys, srows, bad, req_bad, even_split, max_req, cw);
}

const uint32_t* sort_plan_keys_or(Env& env) {
  return reinterpret_cast<const uint32_t*>(static_cast<const char*>(env.arena()->plan) + offsetof(SortPlan, keys_or));
}

int launch_radix_sort_rows16(Env& env, const uint32_t* keys, uint16_t* skeys, uint32_t* srows, uint64_t n,
                             uint32_t value_bits, uint32_t* reject, const uint64_t* d_n, ClearWords cw) {
  if (!reject) return env.fail(kErrArg, "radix_sort16: null reject flag");
  if (value_bits == 0 || value_bits > 16) return env.fail(kErrArg, "radix_sort16: value_bits must be 1..16");
  if (n == 0) return launch_fill_u32(env, reject, 1, 0);
  if (!keys || !skeys || !srows) return env.fail(kErrArg, "radix_sort16: null buffer");
  if (n >= (1ull << 31)) return env.fail(kErrArg, "radix_sort16: n must be below 2^31");
  switch (row_shape(n, digit_split(value_bits, true).bits[0])) {
    case RowShape::k1024:
      return rows_sort16<256, 4, kSum>(env, keys, skeys, srows, n, value_bits, reject, d_n, cw);
    case RowShape::k2048:
      return rows_sort16<512, 4, kSum>(env, keys, skeys, srows, n, value_bits, reject, d_n, cw);
    case RowShape::k4096:
      return rows_sort16<1024, 4, kSum>(env, keys, skeys, srows, n, value_bits, reject, d_n, cw);
    case RowShape::k8192:
      return rows_sort16<1024, 8, kSum>(env, keys, skeys, srows, n, value_bits, reject, d_n, cw);
    case RowShape::kNone:
      break;
  }
  return rows_sort16<1024, 8, kScanned>(env, keys, skeys, srows, n, value_bits, reject, d_n, cw);
}

int launch_radix_sort_pairs(Env& env, const uint32_t* keys, const uint32_t* rows, uint32_t* skeys,
                            uint32_t* srows, uint64_t n, int shape, const uint64_t* d_n, ClearWords cw) {
  if (n == 0) return kOk;
  if (!keys || !skeys || !srows) return env.fail(kErrArg, "radix_sort: null buffer");
  if (n >= (1ull << 31)) return env.fail(kErrArg, "radix_sort: n must be below 2^31");
  if (shape == 0) {
    switch (row_shape(n, kRadixBits)) {
      case RowShape::k1024:
        return rows_sort32<256, 4, kSum>(env, keys, rows, skeys, srows, n, d_n, cw);
      case RowShape::k2048:
        return rows_sort32<512, 4, kSum>(env, keys, rows, skeys, srows, n, d_n, cw);
      case RowShape::k4096:
        return rows_sort32<1024, 4, kSum>(env, keys, rows, skeys, srows, n, d_n, cw);
      case RowShape::k8192:
        return rows_sort32<1024, 8, kSum>(env, keys, rows, skeys, srows, n, d_n, cw);
      case RowShape::kNone:
        break;
    }
  }
  switch (shape) {
    case 0:
      return rows_sort32<kShapes[0].block, kShapes[0].items, kScanned>(env, keys, rows, skeys, srows, n, d_n, cw);
    case 1:
      return rows_sort32<kShapes[1].block, kShapes[1].items, kScanned>(env, keys, rows, skeys, srows, n, d_n, cw);
    case 2:
      return rows_sort32<kShapes[2].block, kShapes[2].items, kScanned>(env, keys, rows, skeys, srows, n, d_n, cw);
    default:
      return env.fail(kErrArg, "radix_sort: unknown tile shape");
  }
}

}  // namespace ka
