// WAH encoding of sorted (value, row) pairs -- parts 3 to 6 of the index build
// of Sec. 4.1:
//   part 3  chunk ids and literals: a group is a maximal run of equal value
//           and equal chunk id row / 31; its literal ORs 1 << (row % 31);
//   part 4  fills: the gap of empty chunks since the previous group of the
//           same value (or since chunk -1 for the value's first group);
//   part 5  fuseFillsLiterals: the fill and literal words of every group in
//           order, zero fills dropped (a stream compaction, fused here: each
//           group emits 1 or 2 words and the word positions are a prefix sum);
//   part 6  lookup table: keys[d] and offsets[d] for the first group of each
//           value, offsets[D] = W.
//
// What element e contributes depends only on e and its predecessor e - 1:
//   seg(e) = e is the first element of its value,
//   grp(e) = seg(e) or chunk(e) != chunk(e - 1)   (e starts a group),
//   gap(e) = grp(e) and the fill before e is non-zero (chunk(e) != 0 for a
//            value's first group, chunk(e) != chunk(e - 1) + 1 otherwise),
// and e emits grp(e) + gap(e) words and seg(e) values.  So the encoding is one
// single-pass kernel over tiles of 8 pairs per work-item, k_wah_write: each tile
// counts its words and values, publishes both counts, finds the counts of all
// earlier tiles by decoupled look-back (one status chain for words, one for
// values; a silent predecessor is counted from its input by the waiting wave)
// and writes its words and lookup-table entries; the last tile writes W, D,
// offsets[D] and the three output lengths.  The sorted pairs are read once.
// A group spans at most 31 sorted elements (rows are distinct), so a tile
// finishes a group that runs past its end by reading at most 30 elements
// ahead (kLook).
//
// The other word formats (canonical WAH: a run of full groups is one 1-fill;
// PLWAH: a fill also absorbs the group after it when that differs in one bit)
// come out of the same pass, because what they add is decided by a few sorted
// elements too -- rows of a value are distinct and ascending, so two elements
// of one value whose rows differ by exactly their distance enclose a full run:
//   full(e)   the group that e starts holds all 31 rows: e + 30 has the same
//             value and row(e) + 30, and e's row starts its chunk;
//   pfull(e)  the group before e's is the chunk before it and full: e - 31 has
//             the same value and starts that chunk;
//   thirty(e) the group holds 30 rows: e + 29 is in it and it is not full;
//   one(e)    it holds one row: e + 1 is not in it;
// and a run of L full groups ends where e + 31 L - 1 no longer has row(e) +
// 31 L - 1 (monotone in L: exponential, then binary search, at run starts
// only).  A group emits its fill (unless it is skipped) and its literal or
// 1-fill (unless it is skipped or absorbed); positions are the same prefix sum.  Words are staged in LDS (over the staged input, which is
// dead by then) and written out by consecutive work-items.  Sorted keys are
// uint32, or uint16 when every value is below 2^16 (the index build's
// narrow-key sort).
#include <algorithm>

#include "common.hpp"
#include "lds_sort.hpp"

namespace ka {
namespace {

// 1024 work-items x 8 elements: a tile of 8192 pairs, two work-groups of 16
// waves per CU (bound by LDS; 63 or 64 VGPRs).  The look-back's latency (a few
// device-coherent round trips, about 0.75 us each) is paid once per tile while
// the tile's work-group waits, and the LDS sweeps stall on bank conflicts:
// twice the waves of 512 x 16 hide both better, 206 -> 181 us on 2^26 Zipf
// pairs and 324 -> 225 us on uniform 16-bit ones (the batched build of 4096
// requests: +0.8%).  Tiles of 4096 pairs paid the look-back twice as often
// (244 against 228 us at 512 x 16); 16384-pair tiles (one work-group per CU)
// took 308 us.
constexpr int kEncBlock = 1024;
constexpr int kEncItems = 8;
constexpr int kVecs = kEncItems / 4;  // 16-byte loads per work-item and array
constexpr int kLook = 32;             // >= 30 elements of look-ahead
constexpr uint32_t kGroupRows = 31;
constexpr uint32_t kFill = 0x80000000u;
constexpr uint32_t kOnes = 0x40000000u;      // fill bit of a 1-fill

// Padded LDS index: four spare words after every 64 elements.  Groups of 4
// elements stay 16-byte aligned, so the tile is staged with conflict-free
// 16-byte writes (work-item t writes elements 4t..4t+3); a work-item reads its
// 8 consecutive elements with two 16-byte reads, and the 16 work-items served
// together (starting 32 bytes apart, plus 16 after every eighth) cover all 64
// banks once.
__device__ __forceinline__ uint32_t pidx(uint32_t i) { return i + 4 * (i >> 6); }
static_assert(kEncItems == 8, "one padded run of 8 elements per work-item");

// LDS of one tile of kBlock * kEncItems pairs.
template <int kBlock, int kFmt>
struct EncLds {
  static constexpr int kTile = kBlock * kEncItems;
  static constexpr int kStage = kTile + kLook;  // staged elements (the look-behind is kept apart)
  static constexpr int kPadded = kStage + 4 * (kStage / 64) + 4;
  static constexpr int kBehind = kFmt == kFmtPaper ? 1 : 32;  // elements base - kBehind .. base - 1
  static_assert(2 * kTile <= 2 * kPadded, "word staging fits over the input staging");
  __align__(16) uint32_t mem[2 * kPadded];  // keys, rows; then the tile's words
  uint32_t bk[kBehind], br[kBehind];
  uint32_t scan[kBlock / 64];
  uint32_t pre[2];
};

// Tile elements in registers: slot (j, c) of work-item tid holds element
// b + 4 (j * kBlock + tid) + c (0 beyond len).
template <int kBlock, bool kVec, class KeyT>
__device__ __forceinline__ void load_pairs(const KeyT* __restrict__ skeys, const uint32_t* __restrict__ srows,
                                           uint32_t b, uint32_t len, uint32_t tid, uint32_t (&vk)[kVecs][4],
                                           uint32_t (&vr)[kVecs][4]) {
  if (kVec && len == (uint32_t)(kBlock * kEncItems)) {
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
      const uint32_t q = j * kBlock + tid;
      load_key4(skeys + b, q, vk[j]);
      const u32x4 c = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(srows + b) + q);
      vr[j][0] = c.x, vr[j][1] = c.y, vr[j][2] = c.z, vr[j][3] = c.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < kVecs; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t i = 4 * (j * kBlock + tid) + c;
        vk[j][c] = i < len ? (uint32_t)skeys[b + i] : 0u;
        vr[j][c] = i < len ? srows[b + i] : 0u;
      }
  }
}

// Rows of a batch of requests sorted together are batch positions; the row
// inside the request is the position minus the request's first position,
// found from the request id in the key's high bits (key >> req_shift).
struct BatchRows {
  const uint32_t* req_base;  // null: rows are used as they are
  uint32_t req_shift;
  __device__ __forceinline__ uint32_t local(uint32_t key, uint32_t row) const {
    return req_base ? row - req_base[req_shift < 32 ? key >> req_shift : 0u] : row;
  }
};

// What the element with key k and row r emits whose predecessor has key kp and
// row rp (first: no predecessor).  at(d, k, r) tells whether the element d
// places further on (back for a negative d) exists and has key k and row r;
// in_group(d, k, c) whether it exists and has key k and chunk c.
struct Emits {
  bool seg, grp;    // starts a value, a group
  bool fill, main;  // a fill word (the gap's 0-fill), a literal or 1-fill word
  bool full;        // main is the 1-fill of the run that starts here
};

template <int kFmt, class At, class InGroup>
__device__ __forceinline__ Emits element_emits(uint32_t k, uint32_t c, uint32_t bit, uint32_t kp, uint32_t cp,
                                               bool first, At&& at, InGroup&& in_group) {
  Emits e;
  e.seg = first || k != kp;
  e.grp = e.seg || c != cp;
  e.fill = e.grp && (e.seg ? c != 0u : c != cp + 1u);
  e.main = e.grp;
  e.full = false;
  if (kFmt != kFmtPaper && e.grp) {
    e.full = bit == 0u && at(30, k, c * kGroupRows + 30u);
    // the group before is the chunk before (then there is no gap) and full
    const bool pfull = !e.seg && c == cp + 1u && at(-31, k, cp * kGroupRows);
    bool skip = e.full && pfull;  // inside the run's 1-fill
    if (kFmt == kFmtPlwah) {
      skip = skip || (pfull && !e.full && in_group(29, k, c));  // 30 rows: absorbed by the run's 1-fill
      if (e.fill && !in_group(1, k, c)) e.main = false;         // one row: absorbed by its 0-fill
    }
    if (skip) e.main = false;
    e.full = e.full && e.main;
  }
  return e;
}

// Words and values that tile u emits, counted from its input by one wave --
// the look-back's fallback for a predecessor that has not published yet.  Lane
// l takes consecutive elements.
template <int kTile, int kFmt, class KeyT>
__device__ LbPairSum wave_tile_count(const KeyT* __restrict__ skeys, const uint32_t* __restrict__ srows, uint32_t n,
                                     uint32_t u, BatchRows br) {
  constexpr uint32_t kPer = kTile / 64;
  const uint32_t b = u * kTile;
  const uint32_t end = min(b + (uint32_t)kTile, n);
  const uint32_t e0 = b + lane_id() * kPer;
  uint32_t nw = 0, ns = 0;
  if (e0 < end) {
    uint32_t kp = 0, rp = 0;
    if (e0 > 0) {
      kp = skeys[e0 - 1];
      rp = br.local(kp, srows[e0 - 1]);
    }
    const uint32_t e1 = min(e0 + kPer, end);
#pragma unroll 1
    for (uint32_t e = e0; e < e1; ++e) {
      const uint32_t k = skeys[e], r = br.local(k, srows[e]), c = r / kGroupRows;
      auto exists = [&](int d) { return d < 0 ? e >= (uint32_t)-d : e + (uint32_t)d < n; };
      const Emits m = element_emits<kFmt>(
          k, c, r - c * kGroupRows, kp, rp / kGroupRows, e == 0,
          [&](int d, uint32_t kk, uint32_t rr) { return exists(d) && skeys[e + d] == kk && srows[e + d] == rr; },
          [&](int d, uint32_t kk, uint32_t cc) {
            return exists(d) && skeys[e + d] == kk && srows[e + d] / kGroupRows == cc;
          });
      nw += (m.fill ? 1u : 0u) + (m.main ? 1u : 0u);
      ns += m.seg ? 1u : 0u;
      kp = k;
      rp = r;
    }
  }
  return {wave_sum(nw), wave_sum(ns)};
}

// An empty input's index, D = 0, W = 0, offsets = [0], by one work-item.
__device__ __forceinline__ void write_empty_index(const IndexOut& out) {
  out.offsets[0] = 0;
  put_len(out.len_keys, out.host, 0, 0);
  put_len(out.len_offsets, out.host, 1, 1);
  put_len(out.len_words, out.host, 2, 0);
}

__global__ void k_wah_empty(IndexOut out) {
  if (threadIdx.x == 0) write_empty_index(out);
}

// Rejection of the whole input, decided by earlier kernels: the encoding is
// void when (*flag >> shift) != 0 (a value at or above 2^shift), and every
// output length is then 0.
struct Reject {
  const uint32_t* flag;  // null: never
  uint32_t shift;
  __device__ __forceinline__ bool operator()() const { return flag && shift < 32 && (*flag >> shift) != 0u; }
};

constexpr int kSmallBlock = 1024;  // the work-group that sorts and encodes a small input

// Pairs at their padded places in the encoder's stage.
struct StagedPairs {
  uint32_t *k, *r;
  __device__ __forceinline__ void put(uint32_t i, uint32_t key, uint32_t row) const {
    k[pidx(i)] = key;
    r[pidx(i)] = row;
  }
  __device__ __forceinline__ void get(uint32_t i, uint32_t& key, uint32_t& row) const {
    key = k[pidx(i)];
    row = r[pidx(i)];
  }
};

// ---------------------------------------------------------------------------------
// write: literals, fills and lookup-table entries of one tile
// ---------------------------------------------------------------------------------
// The other formats take 59 to 75 VGPRs in work-groups of 256 and 512 (6 or 7
// waves per SIMD), and a small input's sort 65 to 81 in its one of 1024: held to
// 64 they spill.
// One work-group per tile; status[kLbSpread * tile] is the tile's (words, values)
// look-back word, zeroed before the launch.
//
// kSort > 0: the one work-group sorts the input itself, at most 1024 * kSort
// values (skeys; no rows, no status), and the index is whole after this launch.
// A small request is latency: eight launches of one or a few work-groups each
// (two passes of count, scan and scatter, then clear and encode) and the gaps
// between them took 56 us of a request of 777 values.
template <int kBlock, int kFmt, bool kVec, int kSort, class KeyT>
__global__ __launch_bounds__(kBlock, kFmt == kFmtPaper && !kSort ? 8 : 4) void k_wah_write(const KeyT* __restrict__ skeys,
                                                         const uint32_t* __restrict__ srows, uint32_t n_cap,
                                                         const uint64_t* __restrict__ d_n,
                                                         uint64_t* __restrict__ status, uint32_t spin_limit,
                                                         IndexOut out, BatchRows br, Reject rej) {
  constexpr int kTile = EncLds<kBlock, kFmt>::kTile, kBehind = EncLds<kBlock, kFmt>::kBehind;
  __shared__ EncLds<kBlock, kFmt> L;
  uint32_t* s_k = L.mem;
  uint32_t* s_r = L.mem + EncLds<kBlock, kFmt>::kPadded;
  uint32_t* s_words = L.mem;  // after the literals are built
  const uint32_t tid = threadIdx.x, tile = blockIdx.x;
  const uint32_t base = tile * kTile;
  // n_cap pairs, or the count written on the device by an earlier stage: the
  // grid then covers the capacity and the tiles past the count leave at once
  // (tile 0 of an empty input writes the empty index).
  const uint32_t n = (uint32_t)device_count(n_cap, d_n);
  if (base >= n) {
    if (tile == 0 && tid == 0) write_empty_index(out);
    return;
  }
  uint32_t small_or = 0;
  const uint32_t tile_n = min((uint32_t)kTile, n - base);
  const uint32_t avail = min((uint32_t)(kTile + kLook), n - base);  // readable from base on

  if constexpr (kSort > 0) {
    __shared__ LdsSort<kBlock> S;
    small_or = lds_sort<kBlock, kSort>(skeys, n, StagedPairs{s_k, s_r}, S);
  }
  // ---- stage elements base .. base+kTile+kLook-1 into slots 0.. ---------------
  // Work-items 64.. also load the look-ahead (slots kTile ..) and the kBehind
  // elements before base.
  if constexpr (kSort == 0) {
    uint32_t vk[kVecs][4], vr[kVecs][4];
    load_pairs<kBlock, kVec>(skeys, srows, base, tile_n, tid, vk, vr);
    const bool extra = tid >= 64 && tid < 64 + kLook + kBehind;
    const bool behind = tid >= 64 + kLook;
    const int64_t g = behind ? (int64_t)base - kBehind + (tid - 64 - kLook) : (int64_t)base + kTile + (tid - 64);
    uint32_t xk = 0, xr = 0;
    if (extra) {
      const bool ok = g >= 0 && g < (int64_t)n;
      xk = ok ? (uint32_t)skeys[g] : 0u;
      xr = ok ? br.local(xk, srows[g]) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
      const uint32_t sl = pidx(4 * (j * kBlock + tid));
      u32x4 k4, r4;
      k4.x = vk[j][0], k4.y = vk[j][1], k4.z = vk[j][2], k4.w = vk[j][3];
      r4.x = br.local(vk[j][0], vr[j][0]), r4.y = br.local(vk[j][1], vr[j][1]);
      r4.z = br.local(vk[j][2], vr[j][2]), r4.w = br.local(vk[j][3], vr[j][3]);
      *reinterpret_cast<u32x4*>(s_k + sl) = k4;
      *reinterpret_cast<u32x4*>(s_r + sl) = r4;
    }
    if (extra) {
      if (behind) {
        L.bk[tid - 64 - kLook] = xk;
        L.br[tid - 64 - kLook] = xr;
      } else {
        const uint32_t sl = pidx((uint32_t)(kTile + (tid - 64)));
        s_k[sl] = xk;
        s_r[sl] = xr;
      }
    }
    __syncthreads();
  }

  // ---- this work-item's kEncItems consecutive elements, in registers: key, the
  // row's group (row / 31) and its bit inside the group; elements past the
  // tile's end get bit 31, which no literal keeps --------------------------------
  const uint32_t e0 = tid * kEncItems;
  const uint32_t nvalid = e0 < tile_n ? min(tile_n - e0, (uint32_t)kEncItems) : 0u;
  const uint32_t valid = nvalid >= 32u ? ~0u : (1u << nvalid) - 1u;  // bit i: element i exists
  uint32_t key[kEncItems], grp_of[kEncItems], bit_of[kEncItems];
#pragma unroll
  for (int q = 0; q < kEncItems / 4; ++q) {
    const u32x4 k4 = *reinterpret_cast<const u32x4*>(s_k + pidx(e0) + 4 * q);
    const u32x4 r4 = *reinterpret_cast<const u32x4*>(s_r + pidx(e0) + 4 * q);
    const uint32_t kk[4] = {k4.x, k4.y, k4.z, k4.w}, rr[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = 4 * q + c;
      key[i] = kk[c];
      grp_of[i] = rr[c] / kGroupRows;
      bit_of[i] = (valid >> i) & 1u ? rr[c] - grp_of[i] * kGroupRows : 31u;
    }
  }
  // The element before this work-item's first: the previous work-item's last
  // (a shuffle; lane 0 reads it from LDS: the wave before, or the look-behind).
  const uint32_t lane = lane_id();
  uint32_t kprev = (uint32_t)__shfl_up((int)key[kEncItems - 1], 1);
  uint32_t cprev = (uint32_t)__shfl_up((int)grp_of[kEncItems - 1], 1);
  if (lane == 0) {
    constexpr int kLast = EncLds<kBlock, kFmt>::kBehind - 1;
    kprev = tid ? s_k[pidx(e0 - 1)] : L.bk[kLast];
    cprev = (tid ? s_r[pidx(e0 - 1)] : L.br[kLast]) / kGroupRows;
  }

  // ---- group and value heads, words and values emitted ------------------------------
  // bit i: element i starts a group / a value / has a fill word / a literal or
  // 1-fill word (the paper's form: every head has one)
  uint32_t heads = 0, segs = 0, gaps = 0, mains = 0;
  uint32_t run_i = kEncItems;  // the element whose word is a 1-fill: full groups are 31 elements apart, so one at most
  const bool first_of_input = base + e0 == 0u;  // this work-item's element 0 is the input's first
#pragma unroll
  for (int i = 0; i < kEncItems; ++i) {
    const uint32_t x = e0 + i;
    // keys and rows by tile-local position, from the look-behind to the look-ahead
    auto key_at = [&](int d) { return d < 0 && x < (uint32_t)-d ? L.bk[(32 + x + d) & 31] : s_k[pidx(x + d)]; };
    auto row_at = [&](int d) { return d < 0 && x < (uint32_t)-d ? L.br[(32 + x + d) & 31] : s_r[pidx(x + d)]; };
    auto exists = [&](int d) { return d < 0 ? base + x >= (uint32_t)-d : x + (uint32_t)d < avail; };
    const Emits m = element_emits<kFmt>(
        key[i], grp_of[i], bit_of[i], i ? key[i - 1] : kprev, i ? grp_of[i - 1] : cprev, i == 0 && first_of_input,
        [&](int d, uint32_t kk, uint32_t rr) { return exists(d) && key_at(d) == kk && row_at(d) == rr; },
        [&](int d, uint32_t kk, uint32_t cc) {
          return exists(d) && key_at(d) == kk && row_at(d) / kGroupRows == cc;
        });
    heads |= (uint32_t)m.grp << i;
    segs |= (uint32_t)m.seg << i;
    gaps |= (uint32_t)m.fill << i;
    if (kFmt != kFmtPaper) {
      mains |= (uint32_t)m.main << i;
      if (m.full && ((valid >> i) & 1u)) run_i = i;
    }
  }
  heads &= valid;
  segs &= valid;
  gaps &= valid;
  mains = kFmt == kFmtPaper ? heads : mains & valid;
  const uint32_t nw = (uint32_t)__popc(mains) + (uint32_t)__popc(gaps);
  const uint32_t ns = (uint32_t)__popc(segs);
  // Both counts in one scan: words in the low half, values in the high half
  // (a tile emits at most 2 * kTile words and kTile values).
  uint32_t packed_total;
  const uint32_t packed_pre = block_excl_scan<kBlock>((ns << 16) | nw, L.scan, &packed_total);
  const uint32_t tile_nw = packed_total & 0xFFFFu, tile_ns = packed_total >> 16;

  // ---- publish the tile's counts at once: successors find them while this
  // tile builds its words --------------------------------------------------------------
  if (!kSort && tid == 0)
    lb_publish_raw(status + kLbSpread * tile,
                   lb_pack_pair(tile_nw, tile_ns, tile == 0 ? kLbInclusive : kLbAggregate));

  // ---- the last group may run past this work-item's elements (at most 30
  // further elements): collect its bits now.  They are the elements of the next
  // work-items before their first group head ("lead"): a group holds at most 31
  // elements, so it reaches at most four work-items further, and the fourth
  // one has a head.  Shuffles within the wave; the wave's last four lanes read
  // ahead in LDS (the next wave's elements, or the look-ahead).  Lanes with
  // invalid elements have no head and no lead bits, which ends a group at the
  // tile's (and the input's) end.
  const uint32_t lead_n = heads ? (uint32_t)__builtin_ctz(heads) : (uint32_t)kEncItems;
  uint32_t lead = 0;
#pragma unroll
  for (int i = 0; i < kEncItems; ++i)
    if ((uint32_t)i < lead_n) lead |= (1u << bit_of[i]) & ~kFill;  // bit 31 marks invalid elements
  const uint32_t lead1 = (uint32_t)__shfl_down((int)lead, 1), lead2 = (uint32_t)__shfl_down((int)lead, 2);
  const uint32_t lead3 = (uint32_t)__shfl_down((int)lead, 3), lead4 = (uint32_t)__shfl_down((int)lead, 4);
  const uint32_t nh = heads == 0u ? 1u : 0u;
  const uint32_t nohead1 = (uint32_t)__shfl_down((int)nh, 1), nohead2 = (uint32_t)__shfl_down((int)nh, 2);
  const uint32_t nohead3 = (uint32_t)__shfl_down((int)nh, 3);
  uint32_t tail = 0;
  if (e0 + kEncItems <= tile_n) {
    if (lane < 60) {
      tail = lead1 | (nohead1 ? (lead2 | (nohead2 ? (lead3 | (nohead3 ? lead4 : 0u)) : 0u)) : 0u);
    } else {
      const uint32_t kl = key[kEncItems - 1], cl = grp_of[kEncItems - 1];
      for (uint32_t j = e0 + kEncItems; j < avail; ++j) {
        const uint32_t kj = s_k[pidx(j)];
        const uint32_t rj = s_r[pidx(j)];
        const uint32_t cj = rj / kGroupRows;
        if (kj != kl || cj != cl) break;
        tail |= 1u << (rj - cj * kGroupRows);
      }
    }
  }

  // ---- a run of full groups starts here: its length, and the group that its
  // 1-fill absorbs.  Elements of the stage from LDS, later ones from memory. ---------
  uint32_t run_word = 0;
  if (kFmt != kFmtPaper && run_i < (uint32_t)kEncItems) {
    const uint32_t x = e0 + run_i;
    auto key_at = [&](uint32_t j) { return j < avail ? s_k[pidx(j)] : (uint32_t)skeys[base + j]; };
    auto row_at = [&](uint32_t j) { return j < avail ? s_r[pidx(j)] : srows[base + j]; };
    const uint32_t k0 = key_at(x), r0 = row_at(x);
    auto ok = [&](uint32_t len) {  // elements x .. x + 31 len - 1 are len full groups
      const uint64_t d = 31ull * len - 1ull;
      if (d >= n - base - x) return false;
      return key_at(x + (uint32_t)d) == k0 && row_at(x + (uint32_t)d) == r0 + (uint32_t)d;
    };
    uint32_t lo = 1, step = 1;  // ok(lo) holds
    while (ok(lo + step)) {
      lo += step;
      step <<= 1;
    }
    uint32_t hi = lo + step;  // ok(hi) fails
    while (hi - lo > 1u) {
      const uint32_t mid = lo + (hi - lo) / 2u;
      if (ok(mid))
        lo = mid;
      else
        hi = mid;
    }
    run_word = kFill | kOnes | lo;
    if (kFmt == kFmtPlwah) {
      const uint32_t j0 = x + kGroupRows * lo, c1 = r0 / kGroupRows + lo;  // the group after the run
      if (base + j0 + 29u < n && key_at(j0 + 29u) == k0 && row_at(j0 + 29u) / kGroupRows == c1) {  // 30 rows
        uint32_t a = 0, b = 30;  // its first a rows are the chunk's first a rows
        while (a < b) {
          const uint32_t mid = (a + b) / 2u;
          if (row_at(j0 + mid) == c1 * kGroupRows + mid)
            a = mid + 1u;
          else
            b = mid;
        }
        run_word |= (1u + a) << kPlwahShift;  // the missing row's bit
      }
    }
  }
  __syncthreads();  // the staged input is dead from here on

  // ---- one backward sweep: literals (OR of the group's bits) and fills, placed in
  // LDS from the end of this work-item's words --------------------------------------
  const uint32_t wbeg = packed_pre & 0xFFFFu;  // this work-item's first word in the tile
  {
    uint32_t w = wbeg + nw;  // one past this work-item's last word
    uint32_t acc = tail;
#pragma unroll
    for (int i = kEncItems - 1; i >= 0; --i) {
      acc |= 1u << bit_of[i];
      if ((heads >> i) & 1u) {
        if (kFmt == kFmtPaper || ((mains >> i) & 1u))
          s_words[--w] = kFmt != kFmtPaper && (uint32_t)i == run_i
                             ? run_word
                             : acc & ~kFill;  // drops the bit 31 of elements past the tile's end
        acc = 0;
        if ((gaps >> i) & 1u) {
          const uint32_t cp = i ? grp_of[i - 1] : cprev;
          uint32_t word = kFill | (((segs >> i) & 1u) ? grp_of[i] : grp_of[i] - cp - 1u);
          if (kFmt == kFmtPlwah && !((mains >> i) & 1u)) word |= (1u + bit_of[i]) << kPlwahShift;
          s_words[--w] = word;
        }
      }
    }
  }

  // ---- the tile's first word and value: look back over the earlier tiles (wave 0)
  if (tid < 64) {
    LbPairSum pre{0u, 0u};
    if (!kSort && tile > 0) {
      pre = lb_lookback_st<kLbSpread>(status, tile, LbPair{}, spin_limit, [&](uint32_t u) {
        return wave_tile_count<kTile, kFmt>(skeys, srows, n, u, br);
      });
      if (tid == 0)
        lb_publish_raw(status + kLbSpread * tile, lb_pack_pair(pre.a + tile_nw, pre.b + tile_ns, kLbInclusive));
    }
    if (tid == 0) {
      L.pre[0] = pre.a;
      L.pre[1] = pre.b;
    }
  }
  __syncthreads();
  const uint32_t wpre = L.pre[0], dpre = L.pre[1];

  // ---- words, then the lookup-table entries of the values starting here ----------------
  // Four words per work-item and step: an aligned 16-byte LDS read and a
  // 16-byte global store at word alignment (wpre is any word): a quarter of the
  // store instructions of word-sized stores (204 against 215 us per 2^26
  // Zipf pairs).
  {
    const uint32_t nv = tile_nw / 4;
    for (uint32_t v = tid; v < nv; v += kBlock)
      *reinterpret_cast<u32x4w*>(out.words + wpre + 4 * v) = *reinterpret_cast<const u32x4*>(s_words + 4 * v);
    if (tid < tile_nw - 4 * nv) out.words[wpre + 4 * nv + tid] = s_words[4 * nv + tid];
  }
  if (segs) {
    const uint32_t ls = packed_pre >> 16;  // tile-local index of this work-item's first value
#pragma unroll
    for (int i = 0; i < kEncItems; ++i) {
      if ((segs >> i) & 1u) {
        const uint32_t below = (1u << i) - 1u;
        const uint32_t d = dpre + ls + (uint32_t)__popc(segs & below);
        out.keys[d] = key[i];
        out.offsets[d] = wpre + wbeg + (uint32_t)__popc(mains & below) + (uint32_t)__popc(gaps & below);
      }
    }
  }
  if (base + tile_n == n && tid == 0) {  // the last tile: totals and lengths
    const uint32_t D = dpre + tile_ns, W = wpre + tile_nw;
    out.offsets[D] = W;
    const bool void_ = kSort ? rej.shift < 32 && (small_or >> rej.shift) != 0u : rej();
    put_len(out.len_keys, out.host, 0, void_ ? 0u : D);
    put_len(out.len_offsets, out.host, 1, void_ ? 0u : (uint64_t)D + 1);
    put_len(out.len_words, out.host, 2, void_ ? 0u : W);
  }
}

// Zeroes the encoder's status words (ntiles of them, kLbSpread apart) before
// the write kernel.
__global__ void k_wah_clear(uint64_t* __restrict__ status, uint32_t ntiles) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ntiles) status[kLbSpread * i] = 0ull;
}

// Work-items of the encoder's work-groups by capacity: tiles small enough for
// about one per CU; the other formats, whose registers allow one work-group of
// 1024 per CU, stay at 512.
uint32_t enc_block(uint64_t n, uint32_t format) {
  return n <= 256ull * 2048 ? 256u : n <= 256ull * 4096 || format != kFmtPaper ? 512u : (uint32_t)kEncBlock;
}

uint32_t enc_tiles(uint64_t n, uint32_t format) {
  const uint64_t tile = (uint64_t)enc_block(n, format) * kEncItems;
  return (uint32_t)((n + tile - 1) / tile);
}

template <int kBlock, int kFmt, class KeyT>
int encode_block(Env& env, const KeyT* skeys, const uint32_t* srows, uint32_t n, const IndexOut& out,
                 const EncodeOpts& opt) {
  const uint32_t ntiles = enc_tiles(n, kFmt);
  // The (words, values) chain has no epoch: its own status words, zeroed by the
  // sort before it or here.
  uint64_t* status = opt.cleared.p;
  if (!status) {
    const ClearWords cw = wah_status(env, n, kFmt);
    if (!cw.p) return env.fail(kErrOom, "wah encoder: look-back status words");
    status = cw.p;
    k_wah_clear<<<dim3((ntiles + 255) / 256), dim3(256), 0, env.stream()>>>(status, ntiles);
    const int rc = check_launch(env, "wah_clear launch");
    if (rc) return rc;
  } else if (opt.cleared.count < ntiles) {
    return env.fail(kErrArg, "wah encoder: too few look-back status words");
  }
  constexpr uintptr_t kKeyAlign = sizeof(KeyT) == 4 ? 15u : 7u;
  const bool vec = ((reinterpret_cast<uintptr_t>(skeys) & kKeyAlign) | (reinterpret_cast<uintptr_t>(srows) & 15u)) == 0;
  const BatchRows br{opt.req_base, opt.req_shift};
  const Reject rej{opt.reject_flag, opt.reject_shift};
  env.prof_begin("wah_write");
  if (vec)
    k_wah_write<kBlock, kFmt, true, 0, KeyT><<<dim3(ntiles), dim3(kBlock), 0, env.stream()>>>(
        skeys, srows, n, opt.d_n, status, env.spin_limit(), out, br, rej);
  else
    k_wah_write<kBlock, kFmt, false, 0, KeyT><<<dim3(ntiles), dim3(kBlock), 0, env.stream()>>>(
        skeys, srows, n, opt.d_n, status, env.spin_limit(), out, br, rej);
  env.prof_end("wah_write");
  return check_launch(env, "wah_write launch");
}

template <int kFmt, class KeyT>
int encode_fmt(Env& env, const KeyT* skeys, const uint32_t* srows, uint32_t n, const IndexOut& out,
               const EncodeOpts& opt) {
  const uint32_t block = enc_block(n, kFmt);
  if (block == 256u) return encode_block<256, kFmt>(env, skeys, srows, n, out, opt);
  if constexpr (kFmt == kFmtPaper)
    if (block == (uint32_t)kEncBlock) return encode_block<kEncBlock, kFmt>(env, skeys, srows, n, out, opt);
  return encode_block<512, kFmt>(env, skeys, srows, n, out, opt);
}

template <int kFmt>
void small_fmt(Env& env, const uint32_t* values, uint32_t n, const IndexOut& out, const EncodeOpts& opt,
               const Reject& rej) {
  static_assert(kSmallIndexMax == kSmallBlock * 8, "the largest small input fills the work-group");
  const dim3 g(1), b(kSmallBlock);
#define KA_SMALL(I)                                                                                          \
  k_wah_write<kSmallBlock, kFmt, false, I, uint32_t><<<g, b, 0, env.stream()>>>(values, nullptr, n, opt.d_n, \
                                                                                 nullptr, 0u, out, BatchRows{}, rej)
  // values per work-item of the sort: each costs a ranking step in every pass
  if (n <= 1024)
    KA_SMALL(1);
  else if (n <= 2048)
    KA_SMALL(2);
  else if (n <= 4096)
    KA_SMALL(4);
  else
    KA_SMALL(8);
#undef KA_SMALL
}

template <class KeyT>
int encode_impl(Env& env, const KeyT* skeys, const uint32_t* srows, uint64_t n, const IndexOut& out,
                const EncodeOpts& opt) {
  if (!out.offsets || !out.len_keys || !out.len_offsets || !out.len_words)
    return env.fail(kErrArg, "wah encoder: null output");
  if (n >= (1ull << 30)) return env.fail(kErrArg, "wah encoder: n must be below 2^30");
  if (n && (!skeys || !srows || !out.keys || !out.words)) return env.fail(kErrArg, "wah encoder: null buffer");
  if (n == 0) {
    k_wah_empty<<<dim3(1), dim3(64), 0, env.stream()>>>(out);
    return check_launch(env, "wah_empty launch");
  }
  switch (opt.format) {
    case kFmtPaper:
      return encode_fmt<kFmtPaper>(env, skeys, srows, (uint32_t)n, out, opt);
    case kFmtCanonical:
      return encode_fmt<kFmtCanonical>(env, skeys, srows, (uint32_t)n, out, opt);
    case kFmtPlwah:
      return encode_fmt<kFmtPlwah>(env, skeys, srows, (uint32_t)n, out, opt);
    default:
      return env.fail(kErrArg, "unknown WAH format");
  }
}

}  // namespace

ClearWords wah_status(Env& env, uint64_t n, uint32_t format) {
  ClearWords cw;
  cw.count = enc_tiles(n, format);
  cw.p = static_cast<uint64_t*>(env.scratch(8ull * kLbSpread * std::max<uint32_t>(cw.count, 1)));
  return cw;
}

int launch_wah_encode(Env& env, const uint32_t* skeys, const uint32_t* srows, uint64_t n, const IndexOut& out,
                      const EncodeOpts& opt) {
  return encode_impl(env, skeys, srows, n, out, opt);
}

int launch_wah_small(Env& env, const uint32_t* values, uint64_t n, uint32_t value_bits, const IndexOut& out,
                     const EncodeOpts& opt) {
  if (!values || !out.keys || !out.offsets || !out.words || !out.len_keys || !out.len_offsets || !out.len_words)
    return env.fail(kErrArg, "wah index: null buffer");
  if (n == 0 || n > kSmallIndexMax) return env.fail(kErrArg, "wah index: not a small input");
  const Reject rej{nullptr, value_bits >= 1 && value_bits <= 31 ? value_bits : 32u};
  env.prof_begin("wah_small");
  switch (opt.format) {
    case kFmtPaper:
      small_fmt<kFmtPaper>(env, values, (uint32_t)n, out, opt, rej);
      break;
    case kFmtCanonical:
      small_fmt<kFmtCanonical>(env, values, (uint32_t)n, out, opt, rej);
      break;
    case kFmtPlwah:
      small_fmt<kFmtPlwah>(env, values, (uint32_t)n, out, opt, rej);
      break;
    default:
      return env.fail(kErrArg, "unknown WAH format");
  }
  env.prof_end("wah_small");
  return check_launch(env, "wah_small launch");
}

int launch_wah_encode16(Env& env, const uint16_t* skeys, const uint32_t* srows, uint64_t n, const IndexOut& out,
                        const EncodeOpts& opt) {
  return encode_impl(env, skeys, srows, n, out, opt);
}

}  // namespace ka
