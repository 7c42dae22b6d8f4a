// ka_wah_index_noalloc: the composed index build (radix sort of (value, row)
// pairs, then the WAH encoder) for callers that cannot allocate device memory.
//
// Every scratch buffer the kernels need -- the sorted pairs, the sort's
// ping-pong pair, its digit rows and plan, the encoder's look-back words -- is
// carved out of one file-scope device array, `scratch`, whose device address is
// looked up once per device.  Nothing here calls hipMalloc, hipFree, hipMemset or
// any other allocating routine; the kernels are the same ones ka_wah_index
// launches.  The array keeps the contents of the last call: the look-back words
// are zeroed by the sort's first launch, and every other region is fully written
// before it is read.  Calls that overlap on one device (different streams, or
// threads without ordering) share the array and race.
#include <mutex>

#include "runtime_internal.hpp"

namespace ka {
namespace {

constexpr uint64_t kAlign = 256;
constexpr uint64_t kMaxN = KA_NOALLOC_MAX_N;
constexpr uint64_t kPairBytes = kMaxN * 4;  // one uint32 array of kMaxN elements
// Tiles of a launch: at most 512 where tiles are sized to the input, else 8192 values each.
constexpr uint64_t kTiles = (kMaxN / 8192 > 512 ? kMaxN / 8192 : 512) + 4;
constexpr uint64_t kRowBytes = kTiles * 256 * (2 + 1) + 256 * 4;  // digit rows, their prefixes (a fourth of them), totals
constexpr uint64_t kOrAndBytes = kTiles * 8;
constexpr uint64_t kEncStatusBytes = kTiles * 8 * kLbSpread;  // encoder status slots
constexpr uint64_t kScratchBytes =
    kSortPlanBytes + 4 * kPairBytes + kRowBytes + kOrAndBytes + kEncStatusBytes + 16 * kAlign;

__device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of `scratch` on each device, looked up on the first call with
// that device current.
constexpr int kMaxDevices = 64;
std::mutex g_mu;
void* g_scratch[kMaxDevices] = {};

int scratch_address(int dev, void** out) {
  if (dev < 0 || dev >= kMaxDevices) return set_error(KA_E_DEVICE, "device ordinal beyond the supported count");
  std::lock_guard<std::mutex> g(g_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_error(KA_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return KA_OK;
}

// Launch environment over the static array: scratch by bump allocation.  No
// kernel of this path looks back by epochs, so there are no such words.
class NoAllocEnv final : public Env {
 public:
  NoAllocEnv(char* base, hipStream_t s) : base_(base), s_(s) {
    arena_.plan = base_;
    used_ = kSortPlanBytes;
  }
  hipStream_t stream() override { return s_; }
  void* scratch(uint64_t bytes) override {
    const uint64_t at = (used_ + kAlign - 1) / kAlign * kAlign;
    if (at + bytes > kScratchBytes) return nullptr;
    used_ = at + bytes;
    return base_ + at;
  }
  bool lookback(uint64_t, LbArgs*) override { return false; }
  LookbackArena* arena() override { return &arena_; }
  void prof_begin(const char*) override {}
  void prof_end(const char*) override {}
  int fail(int code, const char* msg) override { return set_error(code, msg); }

 private:
  char* base_;
  hipStream_t s_;
  uint64_t used_ = 0;
  LookbackArena arena_;
};

}  // namespace
}  // namespace ka

using namespace ka;

extern "C" KA_API int ka_wah_index_noalloc(const uint32_t* values, uint64_t n, uint32_t* keys, uint32_t* offsets,
                                           uint32_t* words, uint64_t* lengths, void* stream) {
  try {
    if (!offsets || !lengths || (n && (!values || !keys || !words))) return set_error(KA_E_ARG, "null argument");
    if (n > kMaxN)
      return set_error(KA_E_ARG, "ka_wah_index_noalloc: n exceeds KA_NOALLOC_MAX_N (the static scratch size)");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return set_error(KA_E_DEVICE, "no current HIP device");
    void* base = nullptr;
    int rc = scratch_address(dev, &base);
    if (rc) return rc;
    NoAllocEnv env(static_cast<char*>(base), static_cast<hipStream_t>(stream));
    const IndexOut out{keys, offsets, words, lengths, lengths + 1, lengths + 2, {}};
    if (n == 0) return launch_wah_encode(env, nullptr, nullptr, 0, out);
    if (n <= kSmallIndexMax) return launch_wah_small(env, values, n, 0, out);
    EncodeOpts opt;
    opt.cleared = wah_status(env, n);
    uint32_t* skeys = static_cast<uint32_t*>(env.scratch(4 * n));
    uint32_t* srows = static_cast<uint32_t*>(env.scratch(4 * n));
    if (!opt.cleared.p || !skeys || !srows) return set_error(KA_E_ARG, "ka_wah_index_noalloc: scratch exhausted");
    if ((rc = launch_radix_sort_pairs(env, values, nullptr, skeys, srows, n, 0, nullptr, opt.cleared))) return rc;
    return launch_wah_encode(env, skeys, srows, n, out, opt);
  } catch (...) {
    return set_error(KA_E_DEVICE, "unexpected internal error");
  }
}
