// Exclusive prefix sum and stream compaction of uint32 arrays.
//
// Both are single-pass: every tile (one work-group) is reduced, publishes its
// total, finds its exclusive prefix by decoupled look-back over its
// predecessors and writes its results -- 8 bytes of HBM traffic per element
// for the scan, 4 + 4*kept for the compaction.  Tiles are numbered by
// work-group id and the look-back has a fallback (a predecessor that stays
// silent is reduced from its input by the waiting wave), so no wait depends on
// the order in which work-groups are dispatched.  The fallback reads a
// predecessor's input, which is why the input and output must not overlap.
// (Tiles numbered by a ticket counter instead cost about 8 ns per work-group,
// serialised on the counter.)  The compaction is the primitive of the
// fuseFillsLiterals step (Sec. 4.1): it removes the zero entries and keeps the
// order; its phases "count per group", "scan of the group counts" and "move
// the valid elements" run in one kernel.
//
// Tile layout: round r of lane l of wave w holds the 4 consecutive elements
// starting at tile_base + 4 (64 (w R + r) + l), so every global access is a
// coalesced 16-byte load or store, and a wave's elements are consecutive: its
// rounds' sums are carried along in a scalar, only one sum per wave goes through
// LDS, and a full tile's rounds check no end.  (Rounds over the whole
// work-group, a sum per wave and round: 229 registers for 122 in the scan.)  Us
// before / now: scans of 10^6 values 5.9 / 5.4, 8 10^6 12.1 / 10.8, 6.7 10^7 121 /
// 90; compactions of 10^6 7.4 / 6.6, 8 10^6 15.4 / 14.3, 2.4 10^7 39.7 / 33.3, 6.7
// 10^7 97 / 91 (with the cached loads of load4).
//
// The number of rounds R is chosen per launch: 8 (8192
// elements per tile) up to a capacity, where the look-back's latency dominates,
// 16 above, where fewer tiles mean fewer look-backs per byte.  Scans, us a
// request with 8 / 16 rounds: 4 10^6 values 21.4 / 21.7, 8 10^6 29.6 / 24.8, 1.6
// 10^7 43 / 37.  Compactions, whose tile is staged in LDS (32 / 64 KiB: four or
// two work-groups per CU), us of the kernel, half the values kept, all kept: 8 10^6
// 13.2 / 13.4, 15.6 / 16.6; 2.4 10^7 30.6 / 34.4, 35.6 / 39.7; 3.4 10^7 40 / 43, 52 /
// 57; 4.2 10^7 48 / 52, 76 / 70; 5 10^7 65 / 67, 88 / 85; 6.8 10^7 90 / 90, 118 /
// 111; 1.34 10^8 172 / 166, 222 / 210.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace ka {
namespace {

constexpr int kScanBlock = 256;
constexpr int kWaves = kScanBlock / 64;
constexpr int kSmallRounds = 8, kLargeRounds = 16;
constexpr uint64_t kLargeScan = 1ull << 22, kLargeCompact = 1ull << 25;  // capacities above use kLargeRounds
template <int R>
constexpr int kTileElems = kScanBlock * R * 4;

// Loads are kept in the caches (kStream: not).  The 256 MB behind the L2 hold an
// input for what reads it next: us of a scan and a compaction of the same values in
// turn, both streamed / both cached, 3 10^7 values 47 + 41 / 42 + 36, 4 10^7 79 + 52
// / 54 + 46.  Only the compactions of kLargeRounds stream: from 2^25 values on, an
// input and the up to as many values kept exceed the caches, and what a launch
// keeps isn't known before it.  Compactions alone, of the same values again, in tiles
// of 16 streamed / of 8 cached, all, half and a tenth of the values kept: 3.4 10^7
// 57, 47, 39 / 52, 40, 34; 3.8 10^7 60, 51, 43 / 67, 44, 38; 4.2 10^7 66, 55, 48 / 76,
// 48, 41; 5 10^7 76, 64, 55 / 88, 65, 48; 6.8 10^7 101, 85, 74 / 118, 90, 70.  (After
// a scan of the same half-empty values the cached ones gain more: 4 10^7 71 + 50 / 54
// + 46, 6 10^7 98 + 70 / 88 + 70.)  Stores are streamed.
template <bool kVec, bool kFull, bool kStream>
__device__ __forceinline__ void load4(const uint32_t* __restrict__ p, uint64_t e, uint64_t n, uint32_t v[4]) {
  if (kVec && (kFull || e + 4 <= n)) {
    const u32x4* const src = reinterpret_cast<const u32x4*>(p + e);
    const u32x4 q = kStream ? __builtin_nontemporal_load(src) : *src;
    v[0] = q.x;
    v[1] = q.y;
    v[2] = q.z;
    v[3] = q.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (e + j < n) ? p[e + j] : 0u;
  }
}

template <bool kVec, bool kFull = false>
__device__ __forceinline__ void store4(uint32_t* __restrict__ p, uint64_t e, uint64_t n, const uint32_t v[4]) {
  if (kVec && (kFull || e + 4 <= n)) {
    u32x4 q;
    q.x = v[0];
    q.y = v[1];
    q.z = v[2];
    q.w = v[3];
    __builtin_nontemporal_store(q, reinterpret_cast<u32x4*>(p + e));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (e + j < n) p[e + j] = v[j];
  }
}

// Exclusive prefix of each lane's round sums over (wave, round, lane) order, plus
// the tile total.  One barrier.
template <int R>
__device__ __forceinline__ void tile_scan(const uint32_t (&s)[R], uint32_t (&pre)[R], uint32_t* tile_total,
                                          uint32_t* s_wave) {
  const uint32_t w = threadIdx.x / 64;
  uint32_t run = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t inc = wave_incl_scan(s[r]);
    pre[r] = run + inc - s[r];
    run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  }
  if (lane_id() == 0) s_wave[w] = run;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const uint32_t t = s_wave[i];
    before += (i < (int)w) ? t : 0u;
    total += t;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) pre[r] += before;
  *tile_total = total;
}

// Wave 0 publishes the tile total, looks back, publishes the inclusive prefix
// and leaves the tile's exclusive prefix in *s_prefix; reduce(t) gives a
// silent predecessor's total (see lb_lookback_st).  Tile t's status word is
// lb.status[kLbSpread * t].
template <class Reduce>
__device__ __forceinline__ void tile_lookback(const LbArgs& lb, uint32_t tile, uint32_t tile_total,
                                              uint32_t* s_prefix, Reduce&& reduce) {
  if (threadIdx.x < 64) {
    uint32_t prefix = 0;
    uint64_t* slot = lb.status + (uint64_t)kLbSpread * tile;
    if (tile == 0) {
      if (threadIdx.x == 0) lb_publish(slot, tile_total, lb.epoch, kLbInclusive);
    } else {
      if (threadIdx.x == 0) lb_publish(slot, tile_total, lb.epoch, kLbAggregate);
      prefix = lb_lookback_st<kLbSpread>(lb.status, tile, LbEpoch{lb.epoch}, lb.spin_limit, reduce);
      if (threadIdx.x == 0) lb_publish(slot, prefix + tile_total, lb.epoch, kLbInclusive);
    }
    if (threadIdx.x == 0) *s_prefix = prefix;
  }
  __syncthreads();
}

// Total of tile u by one wave (every lane gets it); op maps an element to
// what it adds (itself for the scan, 1 if non-zero for the compaction).
template <int R, bool kVec, class Op>
__device__ __forceinline__ uint32_t wave_tile_total(const uint32_t* in, uint32_t u, uint64_t n, Op op) {
  const uint64_t b = (uint64_t)u * kTileElems<R>;
  uint32_t acc = 0;
#pragma unroll 4
  for (int i = 0; i < kTileElems<R> / 256; ++i) {
    uint32_t q[4];
    load4<kVec, false, false>(in, b + 4 * ((uint64_t)i * 64 + lane_id()), n, q);
    acc += op(q[0]) + op(q[1]) + op(q[2]) + op(q[3]);
  }
  return wave_sum(acc);
}

// The first of the 4 elements of round r of this work-item in its tile.
template <int R>
__device__ __forceinline__ uint32_t round_elem(int r) {
  return 4u * ((threadIdx.x / 64u * R + r) * 64u + lane_id());
}

template <int R, bool kVec, bool kStream>
__device__ __forceinline__ void load_tile(const uint32_t* __restrict__ in, uint64_t tile, uint64_t n,
                                          uint32_t (&v)[R][4]) {
  const uint64_t base = tile * kTileElems<R>;
  if (kVec && base + kTileElems<R> <= n) {  // uniform: no round checks the end
#pragma unroll
    for (int r = 0; r < R; ++r) load4<kVec, true, kStream>(in, base + round_elem<R>(r), n, v[r]);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) load4<kVec, false, kStream>(in, base + round_elem<R>(r), n, v[r]);
  }
}

// What an element adds: itself, or the groups that it covers as a word of a
// bitmap (the count fused into the scan: no array of counts).
struct AddSelf {
  static constexpr bool kSelf = true;
  __device__ __forceinline__ uint32_t operator()(uint32_t x) const { return x; }
};
template <int kFmt>
struct AddGroups {
  static constexpr bool kSelf = false;
  __device__ __forceinline__ uint32_t operator()(uint32_t x) const { return word_groups<kFmt>(x); }
};

// One tile per work-group.  The grid is the tile count of n_cap; with a
// smaller device-resident count the surplus work-groups leave at once.  kPair:
// two arrays, the second's tiles from work-group first_b on, its status words
// from there on too (two bitmaps of a 2 10^7-row column: 2 x 6.7 us and the
// gap between two launches -> 8.0 us).
// Two work-groups per CU are enough with 16 rounds (32 KB of loads each), and more
// of them spread the chip over more of the arrays: 3.3 10^7 values 51 us with
// three, 46 with two; 6.7 10^7 96 / 90.
template <int R, bool kVec, class Op, bool kPair>
__global__ __launch_bounds__(kScanBlock)
__attribute__((amdgpu_waves_per_eu(2, R == kLargeRounds ? 2 : 8))) void k_exclusive_scan_u32(ScanJob a, ScanJob b, uint32_t first_b, LbArgs lb) {
  constexpr int kTile = kTileElems<R>;
  __shared__ uint32_t s_prefix;
  __shared__ uint32_t s_wave[kWaves];
  const bool second = kPair && blockIdx.x >= first_b;
  const ScanJob job = second ? b : a;
  const uint32_t* __restrict__ in = job.in;
  uint32_t* __restrict__ out = job.out;
  const uint64_t n = device_count(job.n_cap, job.d_n);
  const uint64_t ntiles = (n + kTile - 1) / kTile;
  const uint32_t tile = second ? blockIdx.x - first_b : blockIdx.x;
  if (second) lb.status += (uint64_t)kLbSpread * first_b;
  if (tile >= ntiles) return;
  const uint64_t base = (uint64_t)tile * kTile;
  uint32_t v[R][4];
  load_tile<R, kVec, false>(in, tile, n, v);
  if (!Op::kSelf) {  // elements past the end add nothing
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[r][j] = base + round_elem<R>(r) + j < n ? Op()(v[r][j]) : 0u;
  }
  uint32_t s[R], pre[R];
#pragma unroll
  for (int r = 0; r < R; ++r) s[r] = v[r][0] + v[r][1] + v[r][2] + v[r][3];
  uint32_t total;
  tile_scan<R>(s, pre, &total, s_wave);
  tile_lookback(lb, tile, total, &s_prefix, [&](uint32_t u) {
    return wave_tile_total<R, kVec>(in, u, n, Op());  // an earlier tile: every element exists
  });
  const uint32_t tp = s_prefix;
  const auto write = [&](auto full) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      uint32_t acc = tp + pre[r], o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        o[j] = acc;
        acc += v[r][j];
      }
      store4<kVec, decltype(full)::value>(out, base + round_elem<R>(r), n, o);
    }
  };
  if (kVec && base + kTile <= n)
    write(std::true_type());
  else
    write(std::false_type());
}

// Kept elements are staged in LDS at their tile-local positions, then copied
// to out[prefix ...] with consecutive work-items writing consecutive words.
template <int R, bool kVec>
__global__ __launch_bounds__(kScanBlock) void k_compact_nonzero_u32(const uint32_t* __restrict__ in,
                                                                    uint32_t* __restrict__ out, uint64_t n_cap,
                                                                    const uint64_t* __restrict__ d_n,
                                                                    uint64_t* __restrict__ d_out_len, LenHost host, LbArgs lb) {
  constexpr int kTile = kTileElems<R>;
  __shared__ uint32_t s_prefix;
  __shared__ uint32_t s_wave[kWaves];
  __shared__ __align__(16) uint32_t s_out[kTile];
  const uint64_t n = device_count(n_cap, d_n);
  const uint64_t ntiles = (n + kTile - 1) / kTile;
  if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) put_len(d_out_len, host, 0, 0);  // empty input
  const uint32_t tile = blockIdx.x;
  if (tile >= ntiles) return;
  uint32_t v[R][4];
  load_tile<R, kVec, R == kLargeRounds>(in, tile, n, v);
  uint32_t s[R], pre[R];
#pragma unroll
  for (int r = 0; r < R; ++r) s[r] = (v[r][0] != 0) + (v[r][1] != 0) + (v[r][2] != 0) + (v[r][3] != 0);
  uint32_t total;
  tile_scan<R>(s, pre, &total, s_wave);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint32_t pos = pre[r];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (v[r][j] != 0) s_out[pos++] = v[r][j];
  }
  tile_lookback(lb, tile, total, &s_prefix, [&](uint32_t u) {  // ends with a barrier
    return wave_tile_total<R, kVec>(in, u, n, [](uint32_t x) { return x != 0 ? 1u : 0u; });
  });
  const uint64_t dst = s_prefix;
  // four kept words per work-item and step (16-byte stores at word alignment)
  const uint32_t nv = total / 4;
  for (uint32_t v = threadIdx.x; v < nv; v += kScanBlock)
    *reinterpret_cast<u32x4w*>(out + dst + 4 * v) = *reinterpret_cast<const u32x4*>(s_out + 4 * v);
  if (threadIdx.x < total - 4 * nv) out[dst + 4 * nv + threadIdx.x] = s_out[4 * nv + threadIdx.x];
  if (tile == ntiles - 1 && threadIdx.x == 0) put_len(d_out_len, host, 0, dst + total);
}

inline bool ranges_overlap(const uint32_t* a, const uint32_t* b, uint64_t n) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + 4 * n && y < x + 4 * n;
}

template <int R, class Op, bool kPair>
int scan_launch(Env& env, const ScanJob& a, const ScanJob& b) {
  const auto tiles = [](const ScanJob& j) { return (uint32_t)((j.n_cap + kTileElems<R> - 1) / kTileElems<R>); };
  const uint32_t first_b = tiles(a), grid = first_b + (kPair ? tiles(b) : 0u);
  LbArgs lb;
  if (!env.lookback((uint64_t)kLbSpread * grid, &lb))
    return env.fail(kErrOom, "exclusive_scan_u32: look-back state");
  uintptr_t at = reinterpret_cast<uintptr_t>(a.in) | reinterpret_cast<uintptr_t>(a.out);
  if (kPair) at |= reinterpret_cast<uintptr_t>(b.in) | reinterpret_cast<uintptr_t>(b.out);
  const dim3 g(grid), block(kScanBlock);
  env.prof_begin("exclusive_scan_u32");
  if ((at & 15u) == 0)
    k_exclusive_scan_u32<R, true, Op, kPair><<<g, block, 0, env.stream()>>>(a, b, first_b, lb);
  else
    k_exclusive_scan_u32<R, false, Op, kPair><<<g, block, 0, env.stream()>>>(a, b, first_b, lb);
  env.prof_end("exclusive_scan_u32");
  return check_launch(env, "exclusive_scan_u32 launch");
}

int check_scan(Env& env, const ScanJob& j) {
  if (!j.in || !j.out) return env.fail(kErrArg, "exclusive_scan_u32: null buffer");
  if (j.n_cap > 0xFFFFFFFFull) return env.fail(kErrArg, "exclusive_scan_u32: more than 2^32-1 elements");
  if (ranges_overlap(j.in, j.out, j.n_cap)) return env.fail(kErrArg, "exclusive_scan_u32: in and out overlap");
  return kOk;
}

template <class Op>
int scan_any(Env& env, const ScanJob& j) {
  if (j.n_cap == 0) return kOk;
  const int rc = check_scan(env, j);
  if (rc) return rc;
  return j.n_cap > kLargeScan ? scan_launch<kLargeRounds, Op, false>(env, j, j)
                              : scan_launch<kSmallRounds, Op, false>(env, j, j);
}

template <class Op>
int scan_pair(Env& env, const ScanJob& a, const ScanJob& b) {
  if (a.n_cap == 0) return scan_any<Op>(env, b);
  if (b.n_cap == 0) return scan_any<Op>(env, a);
  int rc = check_scan(env, a);
  if (rc || (rc = check_scan(env, b))) return rc;
  return std::max(a.n_cap, b.n_cap) > kLargeScan ? scan_launch<kLargeRounds, Op, true>(env, a, b)
                                                 : scan_launch<kSmallRounds, Op, true>(env, a, b);
}

template <class Op>
int scan_groups(Env& env, const ScanJob& a, const ScanJob* b) {
  return b ? scan_pair<Op>(env, a, *b) : scan_any<Op>(env, a);
}

}  // namespace

// in and out must not overlap.
int launch_exclusive_scan(Env& env, const uint32_t* in, uint32_t* out, uint64_t n_cap, const uint64_t* d_n) {
  return scan_any<AddSelf>(env, ScanJob{in, out, n_cap, d_n});
}

int launch_exclusive_scan_groups(Env& env, const ScanJob& a, const ScanJob* b, uint32_t fmt) {
  switch (fmt) {
    case kFmtPaper:
      return scan_groups<AddGroups<kFmtPaper>>(env, a, b);
    case kFmtCanonical:
      return scan_groups<AddGroups<kFmtCanonical>>(env, a, b);
    case kFmtPlwah:
      return scan_groups<AddGroups<kFmtPlwah>>(env, a, b);
    default:
      return env.fail(kErrArg, "unknown WAH format");
  }
}

template <int R>
static int compact_launch(Env& env, const uint32_t* in, uint32_t* out, uint64_t n_cap, const uint64_t* d_n,
                          uint64_t* d_out_len, LenHost host) {
  const uint32_t grid = (uint32_t)((n_cap + kTileElems<R> - 1) / kTileElems<R>);
  LbArgs lb;
  if (!env.lookback((uint64_t)kLbSpread * grid, &lb))
    return env.fail(kErrOom, "compact_nonzero_u32: look-back state");
  const bool vec = (reinterpret_cast<uintptr_t>(in) & 15u) == 0;
  env.prof_begin("compact_nonzero_u32");
  if (vec)
    k_compact_nonzero_u32<R, true><<<dim3(grid), dim3(kScanBlock), 0, env.stream()>>>(in, out, n_cap, d_n, d_out_len, host,
                                                                                   lb);
  else
    k_compact_nonzero_u32<R, false><<<dim3(grid), dim3(kScanBlock), 0, env.stream()>>>(in, out, n_cap, d_n, d_out_len, host,
                                                                                    lb);
  env.prof_end("compact_nonzero_u32");
  return check_launch(env, "compact_nonzero_u32 launch");
}

int launch_compact_nonzero(Env& env, const uint32_t* in, uint32_t* out, uint64_t n_cap, const uint64_t* d_n,
                           uint64_t* d_out_len, LenHost host) {
  if (!d_out_len) return env.fail(kErrArg, "compact_nonzero_u32: no length slot");
  if (n_cap == 0) return launch_set_len(env, d_out_len, 0, host);
  if (!in || !out) return env.fail(kErrArg, "compact_nonzero_u32: null buffer");
  if (n_cap > 0xFFFFFFFFull) return env.fail(kErrArg, "compact_nonzero_u32: more than 2^32-1 elements");
  if (ranges_overlap(in, out, n_cap)) return env.fail(kErrArg, "compact_nonzero_u32: in and out overlap");
  return n_cap > kLargeCompact ? compact_launch<kLargeRounds>(env, in, out, n_cap, d_n, d_out_len, host)
                               : compact_launch<kSmallRounds>(env, in, out, n_cap, d_n, d_out_len, host);
}

}  // namespace ka
