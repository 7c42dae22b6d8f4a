// Bitmap decoding, AND / OR of bitmaps and lookup by value -- the queries the
// index is built for (Sec. 4.1 keeps a lookup table from values to bitmaps;
// Sec. 4.2 names interactive searches and queries).  The word formats are the
// encoder's: the paper's form, canonical WAH (a run of full groups is one
// 1-fill: bits 31 and 30 set, run length in bits 29..0), PLWAH (25-bit fill
// lengths; a fill absorbs the group right after it when that differs from the
// fill's groups in one bit only: bits 29..25 = 1 + that bit's index).
//
// Decoding is a scan of the words' group counts (the look-back scan, counting
// as it loads) and a pass over tiles of groups: a tile finds its first and last
// word by a 64-way search, marks where the words between start, and a running
// maximum gives every group its word.  AND / OR decodes both bitmaps tile by
// tile in one pass, which writes the combined groups and each tile's summary,
// and encodes them in a second: what a group emits depends on it and the group
// before, a fill's length on the last non-empty group and a 1-fill's on the end
// of its run, both found in the tile or in the summaries.  Both are bound by
// latency (the search's dependent loads, about 1 us each): over 645,162 groups
// a decode takes 7 + 10 us and an OR 8 + 17 + 6 us, in two and three launches
// (both bitmaps' scans in one: 13.4 us and a launch's gap before); counting,
// scanning, searching per group, compacting and encoding through a group list
// took 27 us in three and 80 us in sixteen.
//
// Every count that depends on the data stays on the device; grids are sized
// by capacities and read the true counts there.
#include <algorithm>

#include "common.hpp"

namespace ka {
namespace {

constexpr uint32_t kFillBit = 0x80000000u;
constexpr uint32_t kOneBit = 0x40000000u;
constexpr uint32_t kFull = 0x7FFFFFFFu;
constexpr uint32_t kLen30 = 0x3FFFFFFFu;
constexpr uint32_t kLen25 = 0x1FFFFFFu;
constexpr int kBlock = 256;
constexpr uint32_t kMaxGrid = 4096;

__device__ __forceinline__ uint32_t dev_count(uint64_t cap, const uint64_t* d_n) {
  return (uint32_t)device_count(cap, d_n);
}

uint32_t grid_for(uint64_t cap) {
  const uint64_t g = (cap + kBlock - 1) / kBlock;
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(g, kMaxGrid));
}

// ---------------------------------------------------------------------------------
// tiles of groups decoded from words
// ---------------------------------------------------------------------------------
constexpr int kPer = 8;                   // consecutive groups per work-item
constexpr uint32_t kTile = kBlock * kPer;  // 2048 groups
constexpr int kWaves = kBlock / 64;

// One bitmap: m words (the count on the device) and the scan of their group counts.
struct Bitmap {
  const uint32_t* words;
  const uint32_t* start;
  uint64_t cap;
  const uint64_t* len;
  __device__ __forceinline__ uint32_t count() const { return dev_count(cap, len); }
};

// Groups that m words cover.
template <int kFmt>
__device__ __forceinline__ uint64_t total_groups(const Bitmap& b, uint32_t m) {
  return m ? (uint64_t)b.start[m - 1] + word_groups<kFmt>(b.words[m - 1]) : 0u;
}

// Last k in [0, m) with start[k] <= g, by one wave (m > 0; start[0] = 0): every
// step leaves a 64th of the range.
__device__ __forceinline__ uint32_t wave_last_start(const uint32_t* __restrict__ start, uint32_t m, uint32_t g) {
  uint32_t lo = 0, hi = m;  // start[lo] <= g < start[hi] (or hi = m)
  while (hi - lo > 1u) {
    const uint32_t step = (hi - lo + 63u) / 64u;
    const uint64_t p = (uint64_t)lo + (uint64_t)lane_id() * step;
    const bool le = p < hi && start[p < hi ? p : lo] <= g;
    const uint32_t c = (uint32_t)__popcll(__ballot(le || lane_id() == 0));
    lo += (c - 1u) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

// Group gi of the word w that starts at group s.
template <int kFmt>
__device__ __forceinline__ uint32_t group_value(uint32_t w, uint32_t s, uint32_t gi) {
  if (!(w & kFillBit)) return w;
  const bool one = (w & kOneBit) != 0u;
  const uint32_t len = kFmt == kFmtPlwah ? (w & kLen25) : (w & kLen30);
  if (gi - s < len) return one ? kFull : 0u;
  const uint32_t p = kFmt == kFmtPlwah ? (w >> kPlwahShift) & 31u : 0u;  // the absorbed group after the fill
  return one ? (kFull & ~(1u << (p - 1u))) : (1u << (p - 1u));
}

// Largest of the wave's lanes up to this one.
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t x) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, off);
    if ((int)lane_id() >= off) x = max(x, y);
  }
  return x;
}

// Largest of the work-group's work-items before this one (0 for the first) and,
// in *all, of all of them.  s_wave: kWaves words; one barrier.
__device__ __forceinline__ uint32_t block_excl_max(uint32_t x, uint32_t* s_wave, uint32_t* all) {
  const uint32_t inc = wave_incl_max(x), w = threadIdx.x / 64;
  if (lane_id() == 63) s_wave[w] = inc;
  uint32_t r = (uint32_t)__shfl_up((int)inc, 1);
  if (lane_id() == 0) r = 0;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const uint32_t m = s_wave[i];
    if (i < (int)w) r = max(r, m);
    t = max(t, m);
  }
  *all = t;
  return r;
}

// Every word after wl up to wr (the words that hold group g0 and the tile's last
// one) marks its first group in s_mark (kTile words, zeroed, a barrier since)
// with its index + 1, wl the tile's first group; words of no groups mark none.
template <int kFmt>
__device__ __forceinline__ void mark_words(const Bitmap& b, uint32_t m, uint32_t wl, uint32_t wr, uint32_t g0,
                                           uint32_t* s_mark) {
  const uint32_t tid = threadIdx.x;
  if (!m) return;
  if (tid == 0) s_mark[0] = wl + 1u;
  // kPer words per work-item and step, their loads issued together (a word
  // covers a group at least, so one step is the rule)
  for (uint64_t k0 = (uint64_t)wl + 1u + tid; k0 <= wr; k0 += kPer * kBlock) {
    uint32_t at[kPer], w[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint64_t k = k0 + (uint64_t)i * kBlock;
      at[i] = k <= wr ? b.start[k] - g0 : kTile;
      w[i] = k <= wr ? b.words[k] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (at[i] < kTile && word_groups<kFmt>(w[i])) s_mark[at[i]] = (uint32_t)k0 + i * kBlock + 1u;
  }
}

// The index + 1 of the word of each of this work-item's groups, from the marks.
__device__ __forceinline__ void marked_words(const uint32_t* s_mark, uint32_t* s_wave, uint32_t (&idx)[kPer]) {
  const u32x4* const mine = reinterpret_cast<const u32x4*>(s_mark + kPer * threadIdx.x);
  const u32x4 x = mine[0], y = mine[1];
  idx[0] = x.x, idx[1] = x.y, idx[2] = x.z, idx[3] = x.w;
  idx[4] = y.x, idx[5] = y.y, idx[6] = y.z, idx[7] = y.w;
#pragma unroll
  for (int i = 1; i < kPer; ++i) idx[i] = max(idx[i], idx[i - 1]);
  uint32_t all;
  const uint32_t before = block_excl_max(idx[kPer - 1], s_wave, &all);
#pragma unroll
  for (int i = 0; i < kPer; ++i) idx[i] = max(idx[i], before);
}

// Groups g0 + kPer tid + (0 .. kPer-1) of a bitmap in v (0 past its total and
// from ngroups on; words that cover 2^32 groups and more give unspecified ones).
template <int kFmt>
__device__ __forceinline__ void word_values(const Bitmap& b, uint64_t total, uint32_t g0, uint32_t ngroups,
                                            const uint32_t (&idx)[kPer], uint32_t (&v)[kPer]) {
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const uint32_t l = kPer * threadIdx.x + i, g = g0 + l;
    v[i] = l < ngroups - g0 && g < total ? group_value<kFmt>(b.words[idx[i] - 1u], b.start[idx[i] - 1u], g) : 0u;
  }
}

__device__ __forceinline__ void zero_marks(uint32_t* s_mark) {
  const u32x4 zero = {0u, 0u, 0u, 0u};
  u32x4* const mine = reinterpret_cast<u32x4*>(s_mark + kPer * threadIdx.x);
  mine[0] = zero;
  mine[1] = zero;
}

// This work-item's kPer words of a tile that holds n at out, in 16-byte stores
// where all exist.
__device__ __forceinline__ void store_tile(uint32_t* __restrict__ out, uint32_t n, const uint32_t (&v)[kPer]) {
  const uint32_t g = kPer * threadIdx.x;
  if (g + kPer <= n) {
    u32x4w a, c;
    a.x = v[0], a.y = v[1], a.z = v[2], a.w = v[3];
    c.x = v[4], c.y = v[5], c.z = v[6], c.w = v[7];
    *reinterpret_cast<u32x4w*>(out + g) = a;
    *reinterpret_cast<u32x4w*>(out + g + 4) = c;
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (g + i < n) out[g + i] = v[i];
  }
}

// groups[g] for g < ngroups; the output's length is ngroups, or 0 if the words
// cover more.
template <int kFmt>
__global__ __launch_bounds__(kBlock) void k_decode_expand(Bitmap b, uint32_t ngroups, uint32_t* __restrict__ groups,
                                                          uint64_t* __restrict__ len, LenHost host) {
  __shared__ __align__(16) uint32_t s_mark[kTile];
  __shared__ uint32_t s_wave[kWaves], s_at[2];
  const uint32_t m = b.count(), g0 = blockIdx.x * kTile;
  const uint64_t total = total_groups<kFmt>(b, m);
  if (blockIdx.x == 0 && threadIdx.x == 0) put_len(len, host, 0, total > ngroups ? 0u : ngroups);
  if (g0 >= ngroups) return;
  zero_marks(s_mark);
  if (m && threadIdx.x < 128) {  // wave 0: the first group's word, wave 1: the last one's
    const uint32_t w = threadIdx.x / 64;
    const uint32_t k = wave_last_start(b.start, m, w ? g0 + min(kTile, ngroups - g0) - 1u : g0);
    if (lane_id() == 0) s_at[w] = k;
  }
  __syncthreads();
  if (m) mark_words<kFmt>(b, m, s_at[0], s_at[1], g0, s_mark);
  __syncthreads();
  uint32_t idx[kPer], v[kPer];
  marked_words(s_mark, s_wave, idx);
  word_values<kFmt>(b, total, g0, ngroups, idx, v);
  store_tile(groups + g0, min(kTile, ngroups - g0), v);
}

// ---------------------------------------------------------------------------------
// AND / OR of two bitmaps and the encoding of dense groups
// ---------------------------------------------------------------------------------
// What a group x emits after the group p before it (the first group: p = 1, a
// literal of one row).
struct DenseEmits {
  bool fill, main, run;  // a 0-fill for the empty groups before it; a literal or 1-fill; main starts a run of full ones
};
template <int kFmt>
__device__ __forceinline__ DenseEmits dense_emits(uint32_t x, uint32_t p) {
  DenseEmits e;
  const bool full = kFmt != kFmtPaper && x == kFull, pfull = kFmt != kFmtPaper && p == kFull;
  e.fill = x != 0u && p == 0u;
  bool skip = full && pfull;  // inside the run's 1-fill
  if (kFmt == kFmtPlwah) {
    const uint32_t pop = (uint32_t)__popc(x);
    skip = skip || (pfull && pop == 30u);    // absorbed by the run's 1-fill
    skip = skip || (e.fill && pop == 1u);  // absorbed by its 0-fill
  }
  e.main = x != 0u && !skip;
  e.run = e.main && full;
  return e;
}

// Summary of a tile of groups: the words it emits, its last non-empty group's
// index + 1 (0: none), its leading full groups.  Of many tiles (last1 not null)
// the last two also over every 64 and every 4096 of them.
struct TileSums {
  uint32_t *words, *last, *lead;
  uint32_t *last1, *lead1, *last2, *lead2;
};
constexpr uint32_t kLevel = 64;  // entries of a level in one of the next: a wave's window

template <int kFmt, int kOutFmt>
__global__ __launch_bounds__(kBlock) void k_combine(Bitmap a, Bitmap b, uint32_t ngroups, uint32_t op,
                                                    uint32_t* __restrict__ dense, TileSums sums) {
  __shared__ __align__(16) uint32_t s_mark[2][kTile];
  __shared__ uint32_t s_wave[2][kWaves], s_at[4], s_prev[2], s_sum[kWaves];
  const uint32_t tid = threadIdx.x, ma = a.count(), mb = b.count(), g0 = blockIdx.x * kTile;
  zero_marks(s_mark[0]);
  zero_marks(s_mark[1]);
  const uint64_t ta = total_groups<kFmt>(a, ma), tb = total_groups<kFmt>(b, mb);
  {  // a wave each: the words of the tile's first and last group in a and in b
    const uint32_t w = tid / 64, lane = lane_id();
    const bool first = !(w & 1u);
    const Bitmap& t = w < 2 ? a : b;
    const uint32_t m = w < 2 ? ma : mb, last = g0 + min(kTile, ngroups - g0) - 1u;
    uint32_t k = m ? wave_last_start(t.start, m, first ? g0 - (g0 ? 1u : 0u) : last) : 0u;
    if (first) {
      if (lane == 0)  // the group before the tile
        s_prev[w / 2] = g0 && g0 - 1u < (w < 2 ? ta : tb) ? group_value<kFmt>(t.words[k], t.start[k], g0 - 1u) : 0u;
      // on to the tile's first group: one word at most, but for words of no groups
      for (uint32_t step = 64; m && step == 64;) {
        const uint64_t p = (uint64_t)k + 1u + lane;
        const uint64_t past = __ballot(!(p < m && t.start[p] <= g0));
        step = past ? (uint32_t)__builtin_ctzll(past) : 64u;
        k += step;
      }
    }
    if (lane == 0) s_at[w] = k;
  }
  __syncthreads();
  mark_words<kFmt>(a, ma, s_at[0], s_at[1], g0, s_mark[0]);
  mark_words<kFmt>(b, mb, s_at[2], s_at[3], g0, s_mark[1]);
  __syncthreads();
  uint32_t ia[kPer], ib[kPer], va[kPer], vb[kPer];
  marked_words(s_mark[0], s_wave[0], ia);
  marked_words(s_mark[1], s_wave[1], ib);
  word_values<kFmt>(a, ta, g0, ngroups, ia, va);
  word_values<kFmt>(b, tb, g0, ngroups, ib, vb);
  const uint32_t g = g0 + kPer * tid;
  uint32_t x[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) x[i] = op ? va[i] | vb[i] : va[i] & vb[i];
  store_tile(dense + g0, min(kTile, ngroups - g0), x);
  __syncthreads();
  s_mark[0][tid] = x[kPer - 1];  // the next work-item's group before its first
  __syncthreads();
  uint32_t p = 1u, words = 0, last = 0, lead = kTile;
  if (tid)
    p = s_mark[0][tid - 1];
  else if (g0)
    p = op ? s_prev[0] | s_prev[1] : s_prev[0] & s_prev[1];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const DenseEmits e = dense_emits<kOutFmt>(x[i], p);
    words += (e.fill ? 1u : 0u) + (e.main ? 1u : 0u);
    if (x[i]) last = g + i + 1u;
    if (x[i] != kFull && lead == kTile) lead = kPer * tid + i;
    p = x[i];
  }
  uint32_t last_all, nlead_all;
  (void)block_excl_max(last, s_wave[0], &last_all);
  (void)block_excl_max(kTile - lead, s_wave[1], &nlead_all);  // the smallest lead
  const uint32_t wsum = wave_sum(words);
  if (lane_id() == 0) s_sum[tid / 64] = wsum;
  __syncthreads();
  if (tid == 0) {
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) t += s_sum[i];
    sums.words[blockIdx.x] = t;
    sums.last[blockIdx.x] = last_all;
    sums.lead[blockIdx.x] = kTile - nlead_all;
  }
}

// Words of the tiles before tile t, by one wave.
__device__ __forceinline__ uint32_t wave_words_before(const uint32_t* __restrict__ words, uint32_t t) {
  uint32_t s = 0;
  for (uint32_t i = lane_id(); i < t; i += 64) s += words[i];
  return wave_sum(s);
}

// The last entry that is not 0 of v[lo .. t), or 0, by one wave.
__device__ __forceinline__ uint32_t wave_last_before(const uint32_t* __restrict__ v, uint32_t lo, uint32_t t) {
  for (int64_t j = (int64_t)t - 1; j >= (int64_t)lo; j -= 64) {
    const int64_t i = j - (int64_t)lane_id();
    const uint32_t l = i >= (int64_t)lo ? v[i] : 0u;
    const uint64_t some = __ballot(l != 0u);
    if (some) return (uint32_t)__builtin_amdgcn_readlane((int)l, (int)__builtin_ctzll(some));
  }
  return 0u;
}

// Adds the leading full groups of v[t .. end) to ext, by one wave, up to the first
// entry that is not `whole` (then true).
__device__ __forceinline__ bool wave_lead_after(const uint32_t* __restrict__ v, uint32_t t, uint32_t end,
                                                uint32_t whole, uint32_t& ext) {
  for (uint64_t j = t; j < end; j += 64) {
    const uint64_t i = j + lane_id();
    const uint32_t l = i < end ? v[i] : 0u;
    const uint64_t stop = __ballot(i < end && l != whole);
    if (stop) {
      const uint32_t at = (uint32_t)__builtin_ctzll(stop);
      ext += at * whole + (uint32_t)__builtin_amdgcn_readlane((int)l, (int)at);
      return true;
    }
    ext += (uint32_t)min((uint64_t)64, end - j) * whole;
  }
  return false;
}

// The last non-empty group before tile t (index + 1, or 0) and the full groups
// right after it, by one wave each: the tiles beside it, or up to a window of
// them, of blocks of 64 and then blocks of 4096.
__device__ __forceinline__ uint32_t wave_carry(const TileSums& sums, uint32_t t) {
  if (!sums.last1) return wave_last_before(sums.last, 0u, t);
  const uint32_t b = t / kLevel, c = b / kLevel;
  uint32_t r = wave_last_before(sums.last, b * kLevel, t);
  if (!r) r = wave_last_before(sums.last1, c * kLevel, b);
  return r ? r : wave_last_before(sums.last2, 0u, c);
}
__device__ __forceinline__ uint32_t wave_full_after(const TileSums& sums, uint32_t t, uint32_t ntiles) {
  uint32_t ext = 0;
  if (!sums.last1) {
    (void)wave_lead_after(sums.lead, t + 1u, ntiles, kTile, ext);
    return ext;
  }
  const uint32_t b = t / kLevel, c = b / kLevel;
  const uint32_t nb = (ntiles + kLevel - 1u) / kLevel, nc = (nb + kLevel - 1u) / kLevel;
  if (wave_lead_after(sums.lead, t + 1u, min(ntiles, (b + 1u) * kLevel), kTile, ext)) return ext;
  if (wave_lead_after(sums.lead1, b + 1u, min(nb, (c + 1u) * kLevel), kLevel * kTile, ext)) return ext;
  (void)wave_lead_after(sums.lead2, c + 1u, nc, kLevel * kLevel * kTile, ext);
  return ext;
}

// The upper levels of the tiles' summaries: a work-group takes 4096 tiles, a wave
// 64 at a time.
__global__ __launch_bounds__(1024) void k_tile_levels(TileSums sums, uint32_t ntiles) {
  __shared__ uint32_t s_last[kLevel], s_lead[kLevel];
  const uint32_t w = threadIdx.x / 64, lane = lane_id(), nb = (ntiles + kLevel - 1u) / kLevel;
  // (last, lead) of 64 entries; those that don't exist are empty
  const auto reduce = [&](uint32_t last, uint32_t lead, uint32_t whole, uint32_t& last_all, uint32_t& lead_all) {
    const uint64_t some = __ballot(last != 0u), stop = __ballot(lead != whole);
    last_all = some ? (uint32_t)__builtin_amdgcn_readlane((int)last, 63 - (int)__builtin_clzll(some)) : 0u;
    const uint32_t at = stop ? (uint32_t)__builtin_ctzll(stop) : 64u;
    lead_all = at * whole + (at < 64u ? (uint32_t)__builtin_amdgcn_readlane((int)lead, (int)at) : 0u);
  };
  for (uint32_t i = w; i < kLevel; i += 16) {
    const uint32_t b = blockIdx.x * kLevel + i, t = b * kLevel + lane;
    uint32_t last, lead;
    reduce(t < ntiles ? sums.last[t] : 0u, t < ntiles ? sums.lead[t] : 0u, kTile, last, lead);
    if (lane == 0) {
      s_last[i] = last;
      s_lead[i] = lead;
      if (b < nb) {
        sums.last1[b] = last;
        sums.lead1[b] = lead;
      }
    }
  }
  __syncthreads();
  if (w == 0) {
    uint32_t last, lead;
    reduce(s_last[lane], s_lead[lane], kLevel * kTile, last, lead);
    if (lane == 0) {
      sums.last2[blockIdx.x] = last;
      sums.lead2[blockIdx.x] = lead;
    }
  }
}

// The words of one tile.  first_word: the scan of the tiles' words, or null
// (every tile then adds up those before it).  The last tile writes the length:
// the words' count, or 0 if an input covers more than ngroups groups.  A fill
// beyond its length field sets *reject (given only where one can be).
template <int kFmt, int kOutFmt>
__global__ __launch_bounds__(kBlock) void k_dense_encode(Bitmap a, Bitmap b, const uint32_t* __restrict__ dense,
                                                         uint32_t ngroups, TileSums sums,
                                                         const uint32_t* __restrict__ first_word,
                                                         uint32_t* __restrict__ out, uint64_t* __restrict__ len,
                                                         LenHost host, uint32_t* __restrict__ reject) {
  __shared__ uint32_t s_words[2 * kTile];
  __shared__ uint64_t s_full[kTile / 64];  // bit i: group i of the tile is full
  __shared__ uint32_t s_last[kBlock], s_wave[kWaves], s_scan[kWaves];
  __shared__ uint32_t s_base, s_carry, s_ext;
  const uint32_t tid = threadIdx.x, tile = blockIdx.x, ntiles = gridDim.x, g0 = tile * kTile, g = g0 + kPer * tid;
  uint32_t x[kPer];
  if (g + kPer <= ngroups) {
    const u32x4w q = *reinterpret_cast<const u32x4w*>(dense + g), r = *reinterpret_cast<const u32x4w*>(dense + g + 4);
    x[0] = q.x, x[1] = q.y, x[2] = q.z, x[3] = q.w;
    x[4] = r.x, x[5] = r.y, x[6] = r.z, x[7] = r.w;
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) x[i] = g + i < ngroups ? dense[g + i] : 0u;
  }
  const uint32_t edge = tid == 0 && g0 ? dense[g0 - 1u] : 1u;
  const uint32_t w = tid / 64;
  if (w == 0) {  // the tile's first word
    const uint32_t base = first_word ? first_word[tile] : wave_words_before(sums.words, tile);
    if (lane_id() == 0) s_base = base;
  } else if (w == 1) {  // the last non-empty group before the tile
    const uint32_t carry = wave_carry(sums, tile);
    if (lane_id() == 0) s_carry = carry;
  } else if (w == 2) {  // full groups right after the tile
    const uint32_t ext = wave_full_after(sums, tile, ntiles);
    if (lane_id() == 0) s_ext = ext;
  }
  s_last[tid] = x[kPer - 1];
  uint32_t full = 0, last = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    full |= (x[i] == kFull ? 1u : 0u) << i;
    if (x[i]) last = g + i + 1u;
  }
  reinterpret_cast<uint8_t*>(s_full)[tid] = (uint8_t)full;
  __syncthreads();
  const uint32_t prev = tid ? s_last[tid - 1] : edge;
  uint32_t p = prev, words = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const DenseEmits e = dense_emits<kOutFmt>(x[i], p);
    words += (e.fill ? 1u : 0u) + (e.main ? 1u : 0u);
    p = x[i];
  }
  uint32_t total, all;
  uint32_t at = block_excl_scan<kBlock>(words, s_scan, &total);
  const uint32_t before = max(block_excl_max(last, s_wave, &all), s_carry);
  p = prev;
  uint32_t nz = before;  // index + 1 of the last non-empty group so far
  bool over = false;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const DenseEmits e = dense_emits<kOutFmt>(x[i], p);
    if (e.fill) {
      const uint32_t gap = g + i - nz;
      over = over || gap > kLen30;
      uint32_t word = kFillBit | gap;
      if (kOutFmt == kFmtPlwah && !e.main) word |= (1u + (uint32_t)__builtin_ctz(x[i])) << kPlwahShift;
      s_words[at++] = word;
    }
    if (e.main) {
      uint32_t word = x[i];
      if (e.run) {  // the run's length: to the next group that is not full
        const uint32_t l0 = kPer * tid + i;
        uint32_t j = l0 / 64u;
        uint64_t rest = ~s_full[j] & (~0ull << (l0 % 64u));
        while (!rest && ++j < kTile / 64u) rest = ~s_full[j];
        const uint32_t L = rest ? 64u * j + (uint32_t)__builtin_ctzll(rest) - l0 : kTile - l0 + s_ext;
        word = kFillBit | kOneBit | L;
        if (kOutFmt == kFmtPlwah && (uint64_t)g + i + L < ngroups) {
          const uint32_t y = dense[g + i + L];
          if (__popc(y) == 30) word |= (1u + (uint32_t)__builtin_ctz(~y & kFull)) << kPlwahShift;
        }
      }
      s_words[at++] = word;
    }
    if (x[i]) nz = g + i + 1u;
    p = x[i];
  }
  if (over && reject) *reject = 1u;
  __syncthreads();
  const uint32_t base = s_base;
  for (uint32_t i = tid; i < total; i += kBlock) out[base + i] = s_words[i];
  if (tile == ntiles - 1 && tid == 0) {
    const bool more = total_groups<kFmt>(a, a.count()) > ngroups || total_groups<kFmt>(b, b.count()) > ngroups;
    put_len(len, host, 0, more ? 0u : base + total);
  }
}

// ---------------------------------------------------------------------------------
// lookup of values in the table
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_lookup(const uint32_t* __restrict__ keys, uint64_t dcap,
                                                   const uint64_t* __restrict__ d_len,
                                                   const uint32_t* __restrict__ queries, uint32_t q_cap,
                                                   const uint64_t* __restrict__ q_len,
                                                   uint32_t* __restrict__ slots) {
  const uint32_t D = dev_count(dcap, d_len), q = dev_count(q_cap, q_len);
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < q; i += gridDim.x * kBlock) {
    const uint32_t x = queries[i];
    uint32_t lo = 0, hi = D;  // first key >= x
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2u;
      if (keys[mid] < x)
        lo = mid + 1u;
      else
        hi = mid;
    }
    slots[i] = (lo < D && keys[lo] == x) ? lo : 0xFFFFFFFFu;
  }
}

__global__ void k_set_zero_u32(uint32_t* p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0u;
}

// Voids a length (and puts it on the host) if *reject is set.
__global__ void k_void_len(uint64_t* __restrict__ len, LenHost host, const uint32_t* __restrict__ reject) {
  if (threadIdx.x == 0 && blockIdx.x == 0) put_len(len, host, 0, *reject ? 0u : *len);
}

int launch_void_len(Env& env, uint64_t* len, LenHost host, const uint32_t* reject) {
  k_void_len<<<dim3(1), dim3(64), 0, env.stream()>>>(len, host, reject);
  return check_launch(env, "void_len launch");
}

int launch_zero_u32(Env& env, uint32_t* p) {
  k_set_zero_u32<<<dim3(1), dim3(64), 0, env.stream()>>>(p);
  return check_launch(env, "zero launch");
}

// ---- host side --------------------------------------------------------------------------
// Tiles beyond which the summaries get their upper levels.  Without them a tile of
// a nearly empty or nearly full result walks over all the others; they cost a
// launch.  Us an AND of a nearly empty bitmap / an OR of full ones / an OR of two
// of literals, walking and by levels: 2^23 groups 84, 70, 93 and 74, 57, 96; 2^24
// 159, 139, 157 and 110, 82, 160; 2^27 3804, 3965, 1123 and 737, 397, 1136; at
// 2^22 the walk is as fast.
constexpr uint32_t kLevelTiles = 4096;

// A bitmap with room for the scan of its group counts.
bool make_bitmap(Env& env, const uint32_t* words, uint64_t cap, const uint64_t* len, Bitmap* out, ScanJob* job) {
  uint32_t* start = static_cast<uint32_t*>(env.scratch(4 * std::max<uint64_t>(cap, 1)));
  *out = Bitmap{words, start, cap, len};
  *job = ScanJob{words, start, cap, len};
  return start != nullptr;
}

template <int kFmt, int kOutFmt>
int combine_fmt(Env& env, const Bitmap& a, const Bitmap& b, uint32_t ngroups, uint32_t op, uint32_t* dense,
                const TileSums& sums, uint32_t* first_word, uint32_t* words, uint64_t* len, LenHost host,
                uint32_t* reject) {
  const uint32_t ntiles = (ngroups + kTile - 1) / kTile;
  const dim3 grid(ntiles), block(kBlock);
  env.prof_begin("wah_combine");
  k_combine<kFmt, kOutFmt><<<grid, block, 0, env.stream()>>>(a, b, ngroups, op, dense, sums);
  env.prof_end("wah_combine");
  int rc = check_launch(env, "combine launch");
  if (rc) return rc;
  if (first_word && (rc = launch_exclusive_scan(env, sums.words, first_word, ntiles, nullptr))) return rc;
  if (sums.last1) {
    k_tile_levels<<<dim3((ntiles + kLevel * kLevel - 1) / (kLevel * kLevel)), dim3(1024), 0, env.stream()>>>(sums, ntiles);
    if ((rc = check_launch(env, "tile_levels launch"))) return rc;
  }
  if (reject && (rc = launch_zero_u32(env, reject))) return rc;
  env.prof_begin("dense_encode");
  k_dense_encode<kFmt, kOutFmt><<<grid, block, 0, env.stream()>>>(a, b, dense, ngroups, sums, first_word, words, len,
                                                                   reject ? LenHost{} : host, reject);
  env.prof_end("dense_encode");
  if ((rc = check_launch(env, "dense_encode launch"))) return rc;
  return reject ? launch_void_len(env, len, host, reject) : kOk;
}

}  // namespace

int launch_wah_decode(Env& env, const uint32_t* words, uint64_t m_cap, const uint64_t* m_len, uint32_t fmt,
                      uint32_t ngroups, uint32_t* groups, uint64_t* len, LenHost host) {
  if (fmt > kFmtPlwah) return env.fail(kErrArg, "unknown WAH format");
  if (!len || (ngroups && !groups) || (m_cap && !words)) return env.fail(kErrArg, "wah decode: null buffer");
  Bitmap b;
  ScanJob job;
  if (!make_bitmap(env, words, m_cap, m_len, &b, &job)) return env.fail(kErrOom, "wah decode: scratch");
  const int rc = launch_exclusive_scan_groups(env, job, nullptr, fmt);
  if (rc) return rc;
  const dim3 grid(std::max<uint32_t>(1, (uint32_t)(((uint64_t)ngroups + kTile - 1) / kTile))), block(kBlock);
  env.prof_begin("wah_decode");
  switch (fmt) {
    case kFmtPaper:
      k_decode_expand<kFmtPaper><<<grid, block, 0, env.stream()>>>(b, ngroups, groups, len, host);
      break;
    case kFmtCanonical:
      k_decode_expand<kFmtCanonical><<<grid, block, 0, env.stream()>>>(b, ngroups, groups, len, host);
      break;
    default:
      k_decode_expand<kFmtPlwah><<<grid, block, 0, env.stream()>>>(b, ngroups, groups, len, host);
      break;
  }
  env.prof_end("wah_decode");
  return check_launch(env, "decode_expand launch");
}

int launch_wah_combine(Env& env, const uint32_t* a, uint64_t a_cap, const uint64_t* a_len, const uint32_t* b,
                       uint64_t b_cap, const uint64_t* b_len, uint32_t in_fmt, uint32_t ngroups, uint32_t op,
                       uint32_t out_fmt, uint32_t* words, uint64_t* len_words, LenHost host) {
  if (op > 1) return env.fail(kErrArg, "wah combine: op must be 0 (AND) or 1 (OR)");
  if (in_fmt > kFmtPlwah || out_fmt > kFmtPlwah) return env.fail(kErrArg, "unknown WAH format");
  if (!words || !len_words || (a_cap && !a) || (b_cap && !b)) return env.fail(kErrArg, "wah combine: null buffer");
  if (ngroups == 0) return launch_set_len(env, len_words, 0, host);
  const uint32_t ntiles = (ngroups + kTile - 1) / kTile;
  uint32_t* dense = static_cast<uint32_t*>(env.scratch(4ull * ngroups));
  uint32_t* sums = static_cast<uint32_t*>(env.scratch(12ull * ntiles));
  // The tiles' words are scanned in a launch of their own only where every
  // tile's own sum would read more (2048 tiles: 8 KiB a tile).
  uint32_t* first_word = ntiles > 2048 ? static_cast<uint32_t*>(env.scratch(4ull * ntiles)) : nullptr;
  TileSums ts{sums, sums + ntiles, sums + 2ull * ntiles, nullptr, nullptr, nullptr, nullptr};
  if (ntiles > kLevelTiles) {
    const uint64_t nb = (ntiles + kLevel - 1) / kLevel, nc = (nb + kLevel - 1) / kLevel;
    uint32_t* const levels = static_cast<uint32_t*>(env.scratch(8 * (nb + nc)));
    if (!levels) return env.fail(kErrOom, "wah combine: scratch");
    ts.last1 = levels, ts.lead1 = levels + nb;
    ts.last2 = levels + 2 * nb, ts.lead2 = ts.last2 + nc;
  }
  uint32_t* reject = ngroups > kLen30 ? static_cast<uint32_t*>(env.scratch(4)) : nullptr;
  if (!dense || !sums || (ntiles > 2048 && !first_word) || (ngroups > kLen30 && !reject))
    return env.fail(kErrOom, "wah combine: scratch");
  Bitmap ba, bb;
  ScanJob ja, jb;
  if (!make_bitmap(env, a, a_cap, a_len, &ba, &ja) || !make_bitmap(env, b, b_cap, b_len, &bb, &jb))
    return env.fail(kErrOom, "wah combine: scratch");
  const int rc = launch_exclusive_scan_groups(env, ja, &jb, in_fmt);
  if (rc) return rc;
#define KA_COMBINE(I, O) \
  return combine_fmt<I, O>(env, ba, bb, ngroups, op, dense, ts, first_word, words, len_words, host, reject)
#define KA_COMBINE_IN(I)                                    \
  if (out_fmt == kFmtPaper) KA_COMBINE(I, kFmtPaper);         \
  if (out_fmt == kFmtCanonical) KA_COMBINE(I, kFmtCanonical); \
  KA_COMBINE(I, kFmtPlwah)
  if (in_fmt == kFmtPaper) {
    KA_COMBINE_IN(kFmtPaper);
  }
  if (in_fmt == kFmtCanonical) {
    KA_COMBINE_IN(kFmtCanonical);
  }
  KA_COMBINE_IN(kFmtPlwah);
#undef KA_COMBINE_IN
#undef KA_COMBINE
}

int launch_wah_lookup(Env& env, const uint32_t* keys, uint64_t d_cap, const uint64_t* d_len, const uint32_t* queries,
                      uint64_t q, uint32_t* slots, const uint64_t* q_len) {
  if (q == 0) return kOk;
  if (!queries || !slots || (d_cap && !keys)) return env.fail(kErrArg, "wah lookup: null buffer");
  if (q >= (1ull << 32)) return env.fail(kErrArg, "wah lookup: too many queries");
  env.prof_begin("wah_lookup");
  k_lookup<<<dim3(grid_for(q)), dim3(kBlock), 0, env.stream()>>>(keys, d_cap, d_len, queries, (uint32_t)q, q_len,
                                                                         slots);
  env.prof_end("wah_lookup");
  return check_launch(env, "lookup launch");
}

}  // namespace ka
