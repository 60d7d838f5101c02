// Host side of the OptCC executor on one MI355X (gfx950, CDNA4): argument
// checks, the choice of the kernel, the per-device plan tables of the general
// kernel and launches.  Whole AllReduces: optcc_chain.hpp and
// optcc_server_chain.hpp; everything else: optcc_kernels.hpp; each instantiated
// per element type in its own .hip files.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "optcc_internal.hpp"
#include "optcc_launch.hpp"

namespace optcc {
namespace {

using namespace kern;

// The plan's host tile table for tiles of tile_elems elements: tile_elems-
// element pieces of every segment's ring part and P2P chunk, built once per
// tile length.  The caller holds pl.mu; the vector lives as long as the plan.
const std::vector<TileDesc> &host_tiles(const optcc_plan_t &pl, int tile_elems) {
  auto it = pl.host_tiles.find(tile_elems);
  if (it != pl.host_tiles.end()) return it->second;
  std::vector<TileDesc> &tiles = pl.host_tiles[tile_elems];
  for (int g = 0; g < pl.nseg; ++g) {
    const Segment &s = pl.seg[(size_t)g];
    auto cut = [&](int64_t b, int64_t e, int is_p2p) {
      for (int64_t x = b; x < e; x += tile_elems) {
        TileDesc t;
        t.begin = x;
        t.len = (int32_t)std::min<int64_t>(tile_elems, e - x);
        t.meta = (g << 1) | is_p2p;
        tiles.push_back(t);
      }
    };
    cut(std::min(s.ring_begin, pl.n), s.ring_end, 0);
    cut(s.p2p_begin, s.p2p_end, 1);
  }
  return tiles;
}

// Number of tiles host_tiles cuts for tiles of tile_elems elements.
int64_t tile_count(const optcc_plan_t &pl, int tile_elems) {
  int64_t t = 0;
  for (int g = 0; g < pl.nseg; ++g) {
    const Segment &s = pl.seg[(size_t)g];
    const int64_t rb = std::min(s.ring_begin, pl.n);
    if (s.ring_end > rb) t += (s.ring_end - rb + tile_elems - 1) / tile_elems;
    if (s.p2p_end > s.p2p_begin) t += (s.p2p_end - s.p2p_begin + tile_elems - 1) / tile_elems;
  }
  return t;
}

// The plan's tables for tiles of tile_elems elements on the current device,
// uploaded on first use and cached.  The upload (hipMalloc, hipMemcpy) may
// not run while `stream` is being captured into a graph: such a first call
// fails before touching the device, and the capture stays valid.
int device_tables(const optcc_plan_t &pl, int tile_elems, hipStream_t stream, DeviceTables *out) {
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return fail(OPTCC_EDEVICE, std::string("hipGetDevice: ") + hipGetErrorString(err));
  std::lock_guard<std::mutex> lk(pl.mu);
  auto it = pl.dev.find({dev, tile_elems});
  if (it != pl.dev.end()) {
    *out = it->second;
    return OPTCC_OK;
  }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone)
    return fail(OPTCC_EINVAL,
                "the stream is being captured and this plan's tables for this device and "
                "element size are not uploaded yet: run the plan once outside the capture first");
  const std::vector<TileDesc> &tiles = host_tiles(pl, tile_elems);
  DeviceTables d;
  const size_t sb = pl.segdesc.size() * sizeof(SegDesc);
  const size_t tb = std::max<size_t>(tiles.size(), 1) * sizeof(TileDesc);
  err = hipMalloc(&d.segs, sb);
  if (err == hipSuccess) err = hipMalloc(&d.tiles, tb);
  if (err == hipSuccess) err = hipMemcpy(d.segs, pl.segdesc.data(), sb, hipMemcpyHostToDevice);
  if (err == hipSuccess && !tiles.empty())
    err = hipMemcpy(d.tiles, tiles.data(), tiles.size() * sizeof(TileDesc), hipMemcpyHostToDevice);
  if (err != hipSuccess) {
    if (d.segs) (void)hipFree(d.segs);
    if (d.tiles) (void)hipFree(d.tiles);
    return fail(err == hipErrorOutOfMemory ? OPTCC_ENOMEM : OPTCC_EDEVICE,
                std::string("uploading plan tables: ") + hipGetErrorString(err));
  }
  d.ntiles = (int64_t)tiles.size();
  pl.dev[{dev, tile_elems}] = d;
  *out = d;
  return OPTCC_OK;
}

// The work-stealing counter blocks of the plan's tables for tiles of
// tile_elems elements on the current device: kStealSlots blocks, allocated
// and zeroed on the first launch that steals (never under capture: such
// launches keep the static order).  NULL if they cannot be allocated; the
// caller then keeps the static order, which gives the same result.
uint32_t *steal_counters(const optcc_plan_t &pl, int tile_elems) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  std::lock_guard<std::mutex> lk(pl.mu);
  auto it = pl.dev.find({dev, tile_elems});
  if (it == pl.dev.end()) return nullptr;
  DeviceTables &d = it->second;
  if (!d.steal) {
    const size_t wb = (size_t)kStealSlots * kStealWords * sizeof(uint32_t);
    uint32_t *c = nullptr;
    if (hipMalloc(&c, wb) != hipSuccess) return nullptr;
    // zeroed in place before this call returns, like the tables
    const std::vector<uint32_t> zero((size_t)kStealSlots * kStealWords, 0u);
    if (hipMemcpy(c, zero.data(), wb, hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipFree(c);
      return nullptr;
    }
    d.steal = c;
  }
  return d.steal;
}

// Device memory of optcc_allreduce_emulate_noalloc: the plan's tables are
// staged here on every call instead of in memory of their own.  One copy per
// GPU, held until the process ends; calls on one GPU share it.
static __device__ __align__(256) unsigned char scratch[OPTCC_NOALLOC_SCRATCH_BYTES];

// Device address of this GPU's `scratch` (the array's name is a host-side
// stand-in in host code): looked up once per device, with it current.
int scratch_address(void **out) {
  static std::mutex mu;
  static std::map<int, void *> addr;
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return fail(OPTCC_EDEVICE, std::string("hipGetDevice: ") + hipGetErrorString(err));
  std::lock_guard<std::mutex> lk(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    void *ptr = nullptr;
    err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (err != hipSuccess || !ptr)
      return fail(OPTCC_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(err));
    it = addr.emplace(dev, ptr).first;
  }
  *out = it->second;
  return OPTCC_OK;
}

// Bytes of the plan's tables for `ntiles` tiles staged in the no-allocation
// array: segment descriptors (rounded up to 256 bytes), then the tiles.
size_t scratch_bytes(const optcc_plan_t &pl, int64_t ntiles) {
  const size_t seg_bytes = pl.segdesc.size() * sizeof(SegDesc);
  return (seg_bytes + 255) / 256 * 256 + (size_t)ntiles * sizeof(TileDesc);
}

// The plan's tables staged in `scratch` by two copies on `stream` (no device
// allocation).  The host tables are the plan's and live as long as it does.
int scratch_tables(const optcc_plan_t &pl, int tile_elems, hipStream_t stream, DeviceTables *out) {
  const std::vector<TileDesc> *tiles;
  {
    std::lock_guard<std::mutex> lk(pl.mu);
    tiles = &host_tiles(pl, tile_elems);
  }
  const size_t seg_bytes = pl.segdesc.size() * sizeof(SegDesc);
  const size_t tile_off = (seg_bytes + 255) / 256 * 256;
  const size_t tile_bytes = tiles->size() * sizeof(TileDesc);
  if (scratch_bytes(pl, (int64_t)tiles->size()) > (size_t)OPTCC_NOALLOC_SCRATCH_BYTES)
    return fail(OPTCC_EUNSUPPORTED,
                "the plan's tables need " + std::to_string(tile_off + tile_bytes) +
                    " bytes, more than the " + std::to_string(OPTCC_NOALLOC_SCRATCH_BYTES) +
                    " of the no-allocation scratch array: use optcc_allreduce_emulate");
  void *base = nullptr;
  int rc = scratch_address(&base);
  if (rc != OPTCC_OK) return rc;
  char *b = static_cast<char *>(base);
  hipError_t err = hipMemcpyAsync(b, pl.segdesc.data(), seg_bytes, hipMemcpyHostToDevice, stream);
  if (err == hipSuccess && tile_bytes)
    err = hipMemcpyAsync(b + tile_off, tiles->data(), tile_bytes, hipMemcpyHostToDevice, stream);
  if (err != hipSuccess)
    return fail(OPTCC_EDEVICE, std::string("staging plan tables: ") + hipGetErrorString(err));
  out->segs = reinterpret_cast<SegDesc *>(b);
  out->tiles = reinterpret_cast<TileDesc *>(b + tile_off);
  out->ntiles = (int64_t)tiles->size();
  return OPTCC_OK;
}

// Dynamic LDS (not used by the kernel) that holds a launch to at most n
// workgroups per CU on the current device (0 if the device cannot reserve
// that much), cached per device and n.
// fixed: the kernel's own static LDS bytes.
int workgroups_per_cu_lds(int n, int fixed = (int)(sizeof(void *) * kMaxRanks)) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int>, int> cache;
  int dev = 0;
  if (n < 1 || hipGetDevice(&dev) != hipSuccess) return 0;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find({dev, n, fixed});
  if (it != cache.end()) return it->second;
  int per_cu = 0, per_block = 0;
  int v = 0;
  if (hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) ==
          hipSuccess &&
      hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) ==
          hipSuccess) {
    // fixed + want is just over 1/(n+1) of the CU's LDS, so n + 1
    // workgroups never fit, and n still do (n * 256 bytes of margin is far
    // below per_cu / (n + 1) for the n used here)
    const int want = per_cu / (n + 1) + 256 - fixed;
    if (want > 0 && fixed + want <= per_block && (int64_t)n * (fixed + want) <= per_cu) v = want;
  }
  cache[{dev, n, fixed}] = v;
  return v;
}

// Workgroups of the launch's kernel variant the whole device holds at once
// (CUs x workgroups per CU at its registers and dynamic LDS), cached per
// device and variant; 0 if the runtime cannot tell.
int resident_workgroups(const KArgs &a, optcc_dtype_t dtype, bool servers, bool two) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int, int, int, int, int>, int> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const auto key = std::make_tuple(dev, (int)dtype, (int)servers, (int)two,
                                   servers ? a.g : 0, a.occ_lds, a.kept);
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int per_cu = 0, cus = 0;
  hipError_t err = hipSuccess;
  switch (dtype) {
    case OPTCC_F32: err = launch_f32(a, servers, two, nullptr, &per_cu); break;
    case OPTCC_BF16: err = launch_bf16(a, servers, two, nullptr, &per_cu); break;
    case OPTCC_F16: err = launch_f16(a, servers, two, nullptr, &per_cu); break;
    default: err = launch_i32(a, servers, two, nullptr, &per_cu); break;
  }
  if (err != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    per_cu = cus = 0;
  const int v = per_cu > 0 && cus > 0 ? per_cu * cus : 0;
  cache[key] = v;
  return v;
}

// How a whole AllReduce with one GPU per server is launched on the chain
// kernel.  Measured with fp32, bf16 and fp16, 2 to 124 healthy ranks and
// 16 MiB to 4 GiB of rank buffers (back-to-back calls on random data, every
// result bit for bit equal), 10 to 20 shapes each; a row is the shape with the
// least mean loss against the best one at each of its sizes (1-3 %).
constexpr uintptr_t kLine = 128;  // bytes of an L2 line
struct ChainRule {
  int max_pp;  // the row holds up to this many healthy ranks (servers: ranks)
  int bytes;
  ChainPolicy pol;
  int threads, per_cu, runs;  // per_cu 0: as many workgroups as fit; see kRunsByLength
  // Up to this many MiB of buffers the row also takes rank buffers that do not
  // all begin on a 128-byte line; beyond, they run the general kernel.  A wave's
  // 256 bytes (4 per lane) off a line touch one line more, half as much again;
  // the general kernel's 1 KiB one in eight.  Time over the general kernel's, mean
  // of a class of sizes, 1,500 shapes with rows at 16-byte steps off a line or at
  // odd elements: in the cached range 0.35-1.0; above, 4 bytes per lane 0.95-1.26
  // with 5-48 healthy ranks, 0.98-1.5 with more, servers 0.94-1.36 (0.73-0.95 in
  // the classes with a limit here); 8 and 16 bytes per lane 0.84-1.0.  At odd
  // elements the general kernel's accesses are slower too, and chains with one GPU
  // per server keep the chain kernel up to kOddMib (f32 and i32 0.71-1.05 of its
  // time there, bf16 and f16 0.75-1.0, 118 ranks of f16 at 113 MiB 0.81).
  int off_line_mib;
};
constexpr int kAny = INT32_MAX;
constexpr int kOddMib = 256;
// runs 3 where the rank vectors are a multiple of 512 KiB long, else 0.  Buffers
// such a distance apart, powers of two above all, put the same position of every
// rank on the same memory channels, and 8 distant positions at once spread them
// (7 ranks of 2^24 bf16 0.94 of the time before the chains with runs 3, 1.12 with
// 0; 6 x 2 of 2^22 f16 0.96 and 1.23); at other distances neighbouring positions
// are 5-15 % faster (10 ranks of 7,494,663 f16, 4 x 4 GPUs of 3,680,384 f32).
constexpr int kRunsByLength = -1;
// Buffers that the 256 MB memory-side cache holds from the call before or from
// the kernels that wrote them: ordinary accesses keep them there, where
// streaming ones cost 14-46 % from 64 MiB up.  Each XCD takes one run of the
// vector.  Wider accesses win for the shortest chains (3 healthy ranks at 128
// MiB 5 %) and 4 bytes for the others (23 at 64 MiB 10 %).
// When every call finds other buffers in that cache (three sets in turn), the
// same accesses write back lines the cache could have dropped: 3-7 healthy
// ranks lose up to 14 % to the kernel before from 96 MiB up, more than 90 up
// to 11 %.  So those two classes take this table up to 80 MiB (three sets fit) and
// the next one above.  9-90 healthy ranks keep it to 256 MiB: on the same buffers
// they gain 15-28 % by it, on others in turn they lose up to 10 % or gain as much
// (16 ranks of bf16 at 130-256 MiB 0.77 and 1.04 of the time before).
constexpr ChainRule kChainCached32[] = {{5, 8, kResident, 256, 0, 3, kAny},
                                        {kChainMaxHealthy, 4, kResident, 256, 0, 3, kAny}};
constexpr ChainRule kChainCached16[] = {{5, 8, kResident, 256, 0, 3, kAny},
                                        {16, 16, kResident, 256, 0, 3, kAny},
                                        {kChainMaxHealthy, 4, kResident, 256, 0, 3, kAny}};
// Sizes where the cache holds a part, or holds it only sometimes: streaming
// accesses except for the partials, which are overwritten at once.  7 healthy
// ranks at 320 MiB 105 us, all streaming 122, 109 before; 3 at 96-250 MiB 9 %
// faster than before on the same buffers and on others in turn.  Rows 16 and 90
// of 32-bit types, 8 and 16 of 16-bit ones: the shape with the least mean time of
// 20 on 9-20 aligned sizes each, powers of two and others, of the time before and
// the worst of them: 0.84 (0.87), 0.86 (0.94); 0.86 (0.98), 0.87 (0.91).  The last
// 16-bit row: 0.93 (1.06); streaming the partials too, in runs, 0.89 (1.02) but 1.5
// times as long on rows at odd elements.
constexpr ChainRule kChainPartly32[] = {{8, 16, kMixed, 256, 4, 0, kAny},
                                        {16, 4, kStreaming, 256, 0, 0, 0},
                                        {32, 4, kStreaming, 256, 4, 0, kAny},
                                        {90, 4, kStreaming, 256, 2, 0, 0},
                                        {kChainMaxHealthy, 4, kMixed, 256, 0, 3, 256}};
constexpr ChainRule kChainPartly16[] = {{4, 16, kMixed, 256, 4, 0, kAny},
                                        {8, 16, kMixed, 256, 4, kRunsByLength, kAny},
                                        {16, 4, kStreaming, 256, 0, 0, 0},
                                        {32, 4, kStreaming, 256, 4, 0, 0},
                                        {90, 4, kStreaming, 256, 2, 0, 0},
                                        {kChainMaxHealthy, 4, kMixed, 256, 4, 0, 0}};
// Beyond that HBM bounds every chain: each rank's line is read once and written
// once (counters at 2 GiB to 8 GiB of buffers: writes 1.00-1.04 of the results'
// bytes with 8, 16, 64 and 128 ranks).  What a shape decides is the bytes in
// flight per CU (fewer than about 48 KiB leave latency uncovered; the longest
// chains, whose registers hold 256 KiB, lose nothing to L2 by it) and how long a
// piece of each rank's vector a workgroup touches at once (64 ranks in
// workgroups of one wave: 19 % slower than of four).  Longer chains keep the
// same bytes in flight in fewer waves.  fp32 us at 2 GiB of buffers, before
// and now: 2 healthy ranks 822 -> 754, 5 784 -> 713, 7 801 -> 726, 15 813 ->
// 738, 32 864 -> 751, 62 834 -> 783, 95 866 -> 835; at 8 GiB 124 are equal
// (3370).
constexpr ChainRule kChainMemory32[] = {{2, 16, kStreaming, 512, 2, 3, kAny},
                                        {4, 8, kStreaming, 256, 4, 3, kAny},
                                        {8, 4, kStreaming, 512, 0, 0, 0},
                                        {16, 4, kStreaming, 256, 4, 0, 0},
                                        {28, 4, kStreaming, 512, 1, 0, 0},
                                        {48, 4, kStreaming, 1024, 1, 0, 0},
                                        {64, 4, kMixed, 512, 1, 0, 0},
                                        {112, 4, kStreaming, 256, 2, 0, 0},
                                        {kChainMaxHealthy, 4, kMixed, 512, 1, 0, 0}};
constexpr ChainRule kChainMemory16[] = {{4, 16, kMixed, 256, 4, 0, kAny},
                                        {8, 4, kStreaming, 512, 0, 0, 0},
                                        {16, 4, kStreaming, 256, 4, 0, 0},
                                        {28, 4, kStreaming, 512, 2, 0, 0},
                                        {48, 4, kStreaming, 512, 1, 0, 0},
                                        {kChainMaxHealthy, 4, kStreaming, 256, 2, 0, 0}};

// The row for `ranks` (healthy ranks; servers: ranks) and vectors of `bytes`.
ChainRule rule_for(const ChainRule *r, int ranks, int64_t bytes) {
  while (ranks > r->max_pp) ++r;
  ChainRule s = *r;
  if (s.runs == kRunsByLength) s.runs = bytes % (512 << 10) == 0 ? 3 : 0;
  return s;
}
// A chain launch has one lane per `bytes` of the rank vector, in 2^runs runs of
// chain_per_run workgroups.
int64_t chain_per_run(const ChainRule &r, int64_t n, size_t es) {
  const int64_t per = (int64_t)r.threads * (r.bytes / (int64_t)es);  // elements per workgroup
  const int64_t blocks = ((n + kQuantum - 1) / kQuantum * kQuantum + per - 1) / per;
  return ((blocks - 1) >> r.runs) + 1;
}
int64_t chain_work_items(const ChainRule &r, int64_t n, size_t es) {
  return (chain_per_run(r, n, es) << r.runs) * r.threads;
}
// HIP launches fewer than 2^32 work-items in a dimension.
constexpr int64_t kMaxWorkItems = (int64_t)UINT32_MAX;

ChainShape shape_of(const ChainRule &r) {
  ChainShape s;
  s.bytes = r.bytes;
  s.pol = r.pol;
  s.threads = r.threads;
  s.lds = r.per_cu ? workgroups_per_cu_lds(r.per_cu, 0) : 0;
  s.runs = r.runs;
  return s;
}

ChainRule chain_rule(const optcc_plan_t &pl, size_t es) {
  constexpr int64_t kMiB = (int64_t)1 << 20;
  const int64_t buf_bytes = (int64_t)pl.p * pl.n * (int64_t)es;
  const int pp = pl.pp;
  const ChainRule *r;
  if (buf_bytes <= (pp <= 8 || pp > 90 ? 80 : 256) * kMiB) r = es == 4 ? kChainCached32 : kChainCached16;
  else if (buf_bytes <= (pp <= 8 ? 448 : 352) * kMiB) r = es == 4 ? kChainPartly32 : kChainPartly16;
  else r = es == 4 ? kChainMemory32 : kChainMemory16;
  ChainRule s = rule_for(r, pp, pl.n * (int64_t)es);
  // A wave runs the sections it touches one after the other.  Where they are
  // not several times as long as its span, it takes 4 bytes per lane (16
  // healthy ranks of bf16 in sections of one or two quanta: 26 us with 16
  // bytes, 11 with 4).
  const int64_t section = pl.n / ((int64_t)pl.k * pl.pp);
  if (s.bytes > 4 && section < 4 * 64 * (s.bytes / (int64_t)es)) {
    s.bytes = 4;
    if (s.pol == kMixed) s.pol = kStreaming;
    if (s.pol == kStreaming) s.off_line_mib = 0;
  }
  return s;
}

// Granlund and Montgomery's multiplier and shifts for d >= 1.
ChainDiv chain_div(uint32_t d) {
  int l = 0;
  while (l < 32 && ((uint64_t)1 << l) < d) ++l;
  ChainDiv r;
  r.m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << l) - d)) / d + 1);
  r.s1 = (uint32_t)std::min(l, 1);
  r.s2 = (uint32_t)std::max(l - 1, 0);
  return r;
}

int launch_chain_plan(void *const *bufs, const optcc_plan_t &pl, optcc_dtype_t dtype, size_t es,
                      hipStream_t st) {
  const ChainRule rule = chain_rule(pl, es);
  const ChainShape s = shape_of(rule);
  ChainArgs a;  // entries of ptr past the last rank are never used
  std::memset(static_cast<ChainHead *>(&a), 0, sizeof(ChainHead));
  const int64_t nq = (pl.n + kQuantum - 1) / kQuantum;
  a.n = pl.n;
  a.nq = (uint32_t)nq;
  a.k = (uint32_t)pl.k;
  a.pp = pl.pp;
  a.m = pl.m;
  a.wide = nq * pl.k > (int64_t)UINT32_MAX ? 1 : 0;
  a.lq = (uint32_t)(nq / pl.k);
  a.by_nq = chain_div(a.nq);
  a.by_k = chain_div(a.k);
  for (int i = 0; i < 4; ++i)
    if (pl.seg[(size_t)i].ordering == 2) a.ord2 |= 1u << i;
  // Segment 0 has floor(nq / k) quanta; the first one with a quantum more,
  // when k does not divide nq, is the first g with (g + 1) (nq mod k) >= k.
  const int64_t rem = nq % pl.k;
  for (int v = 0; v < (rem ? 2 : 1); ++v) {
    const Segment &sg = pl.seg[v ? (size_t)((pl.k + rem - 1) / rem - 1) : 0];
    ChainSeg &c = a.seg[v];
    c.qbase = (uint32_t)sg.qbase;
    c.nbig = (uint32_t)sg.nbig;
    c.dq = a.lq + (uint32_t)v - (uint32_t)(sg.qbase * pl.pp + sg.nbig);
    c.by_big = chain_div(c.qbase + 1);
    c.by_small = chain_div(std::max(c.qbase, 1u));
  }
  a.runs = s.runs;
  a.per_run = (int32_t)chain_per_run(rule, pl.n, es);
  a.waves = s.threads / 64;
  for (int i = 0; i < 2 * pl.pp; ++i)
    a.ptr[i] = reinterpret_cast<uint64_t>(bufs[pl.ring[(size_t)(i % pl.pp)]]);
  for (int i = 0; i < pl.m; ++i)
    a.ptr[2 * pl.pp + i] = reinterpret_cast<uint64_t>(bufs[pl.strag[(size_t)i]]);
  hipError_t err = hipSuccess;
  switch (dtype) {
    case OPTCC_F32: err = launch_chain_f32(a, s, st); break;
    case OPTCC_BF16: err = launch_chain_bf16(a, s, st); break;
    case OPTCC_F16: err = launch_chain_f16(a, s, st); break;
    default: err = launch_chain_i32(a, s, st); break;
  }
  if (err != hipSuccess)
    return fail(OPTCC_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(err));
  return OPTCC_OK;
}

// Whether a whole AllReduce with one GPU per server runs the chain kernel: every
// chain in registers, the stragglers in its pointer table, quanta within 31 bits
// and a grid that HIP launches (with 4 bytes per lane up to 2^32 elements of a
// 32-bit type per rank).
bool chain_fits(const optcc_plan_t &pl, size_t es) {
  return pl.pp <= kChainMaxHealthy && pl.m <= kChainStragglers &&
         pl.n <= (int64_t)INT32_MAX * kQuantum &&
         chain_work_items(chain_rule(pl, es), pl.n, es) <= kMaxWorkItems;
}

// The same for the server chain kernel, by all p ranks (4 bytes per lane
// everywhere).  Against the kernel that stored each partial as its step ran, 3 to
// 64 servers of 2, 4 and 8 GPUs, aligned buffers, three sets in turn, mean (worst)
// of 5-20 sizes each: up to 80 MiB 0.53-0.76 of its time with 32-bit types,
// 0.51-0.90 with 16-bit ones (1.0 (1.2) for 16-bit messages up to 16 MiB over more
// than 90 ranks, whatever the shape); between, 0.84-0.92 (1.03) and 0.83-0.99
// (1.07-1.15, 128 ranks at 100 MiB 1.26); beyond, 0.87-0.95 and 0.82-0.98 (1.03).
// Between, 16-bit types take one run of the vector per XCD where the rank vectors
// are a multiple of 512 KiB long: powers of two lose up to 68 % without, the other
// multiples up to 13 % with them.  At other lengths runs cost 16-bit types up to
// 27 % (15 x 2 GPUs of 7,514,816 f16 187 and 238 us), and 32-bit types over more
// than 24 ranks up to 22 % (3 % in the mean) at every length.  Ordinary accesses
// throughout would be 17-42 % faster there on the same buffers, but up to 12 %
// slower on others in turn.
constexpr ChainRule kServerCached[] = {{kServerChainMaxRanks, 4, kResident, 256, 0, 3, kAny}};
constexpr ChainRule kServerPartly32[] = {{8, 4, kMixed, 256, 0, 0, 0},
                                         {24, 4, kMixed, 256, 4, kRunsByLength, 0},
                                         {48, 4, kMixed, 512, 1, 0, 448},
                                         {kServerChainMaxRanks, 4, kMixed, 512, 1, 0, 256}};
constexpr ChainRule kServerPartly16[] = {{8, 4, kMixed, 256, 0, 0, 0},
                                         {kServerChainMaxRanks, 4, kMixed, 256, 4, kRunsByLength, 0}};
constexpr ChainRule kServerMemory32[] = {{8, 4, kStreaming, 512, 0, 0, 0},
                                         {24, 4, kStreaming, 256, 4, 0, 0},
                                         {48, 4, kStreaming, 512, 1, 0, 0},
                                         {kServerChainMaxRanks, 4, kMixed, 512, 1, 0, 0}};
constexpr ChainRule kServerMemory16[] = {{8, 4, kStreaming, 512, 0, 0, 0},
                                         {24, 4, kStreaming, 256, 4, 0, 0},
                                         {48, 4, kStreaming, 512, 1, 0, 0},
                                         {kServerChainMaxRanks, 4, kMixed, 512, 0, 3, 0}};

// The middle table reaches further with more than 48 ranks (16-bit types over 49-128
// ranks at 448 to 1000 MiB: 0.89-0.97 of the time before, the last table 0.89-1.00;
// the rows of 32-bit types are the same there).
ChainRule server_chain_rule(const optcc_plan_t &pl, size_t es) {
  const int64_t mib = ((int64_t)pl.p * pl.n * (int64_t)es) >> 20;
  const ChainRule *r = es == 4 ? kServerMemory32 : kServerMemory16;
  if (mib < 80) r = kServerCached;
  else if (mib < (pl.p > 48 ? 1000 : 448)) r = es == 4 ? kServerPartly32 : kServerPartly16;
  return rule_for(r, pl.p, pl.n * (int64_t)es);
}

// Whether a server plan's whole AllReduce runs the server chain kernel: 2, 4 or
// 8 GPUs per server, every rank in registers, quanta times segments (or parts)
// within 32 bits and a grid that HIP launches.
bool server_chain_fits(const optcc_plan_t &pl, size_t es) {
  const int64_t nq = (pl.n + kQuantum - 1) / kQuantum;
  return (pl.g == 2 || pl.g == 4 || pl.g == 8) && pl.p <= kServerChainMaxRanks &&
         nq <= (int64_t)UINT32_MAX / std::max(pl.g, pl.k) && nq >= pl.g &&
         chain_work_items(server_chain_rule(pl, es), pl.n, es) <= kMaxWorkItems;
}

int launch_server_plan(void *const *bufs, const optcc_plan_t &pl, optcc_dtype_t dtype, size_t es,
                       hipStream_t st) {
  const ChainRule rule = server_chain_rule(pl, es);
  const ChainShape s = shape_of(rule);
  ServerChainArgs a;  // entries of ptr past the last server are never used
  const int64_t nq = (pl.n + kQuantum - 1) / kQuantum;
  const int g = pl.g;
  a.n = pl.n;
  a.nq = (uint32_t)nq;
  a.k = (uint32_t)pl.k;
  a.pp = pl.pp;
  a.lp = (uint32_t)(nq / g);
  a.lq = a.lp / a.k;
  a.by_nq = chain_div(a.nq);
  a.by_g = chain_div((uint32_t)g);
  a.by_k = chain_div(a.k);
  for (uint32_t v = 0; v < 2; ++v) {
    a.by_lp[v] = chain_div(std::max(a.lp + v, 1u));
    // a part of lp or lp + 1 quanta has segments of lq and lq + 1 quanta only
    ChainSeg &c = a.seg[v];
    c.dq = 0;
    c.qbase = (a.lq + v) / (uint32_t)pl.pp;
    c.nbig = (a.lq + v) % (uint32_t)pl.pp;
    c.by_big = chain_div(c.qbase + 1);
    c.by_small = chain_div(std::max(c.qbase, 1u));
  }
  a.runs = s.runs;
  a.per_run = (int32_t)chain_per_run(rule, pl.n, es);
  a.waves = s.threads / 64;
  for (int h = 0; h <= pl.pp; ++h) {
    const int sv = h < pl.pp ? pl.ring[(size_t)h] : pl.strag[0];
    for (int e = 0; e < 2 * g; ++e)
      a.ptr[h * 2 * g + e] = reinterpret_cast<uint64_t>(bufs[sv * g + g - 1 - e % g]);
  }
  hipError_t err = hipSuccess;
  switch (dtype) {
    case OPTCC_F32: err = launch_server_chain_f32(a, g, s, st); break;
    case OPTCC_BF16: err = launch_server_chain_bf16(a, g, s, st); break;
    case OPTCC_F16: err = launch_server_chain_f16(a, g, s, st); break;
    default: err = launch_server_chain_i32(a, g, s, st); break;
  }
  if (err != hipSuccess)
    return fail(OPTCC_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(err));
  return OPTCC_OK;
}

// Whether a call is a whole AllReduce on one of the chain kernels.  align: largest
// power of two up to kLine that divides every rank buffer's address.
bool takes_chain(const optcc_plan_t &pl, size_t es, int sb, int se, int launches,
                 uintptr_t align) {
  if (launches != 1 || sb != 0 || se != pl.nslots) return false;
  const bool servers = pl.kind == OPTCC_KIND_SERVERS;
  if (!(servers ? server_chain_fits(pl, es) : chain_fits(pl, es))) return false;
  const ChainRule r = servers ? server_chain_rule(pl, es) : chain_rule(pl, es);
  const int mib = align < 16 && !servers ? std::max(r.off_line_mib, kOddMib) : r.off_line_mib;
  return align >= kLine || (int64_t)pl.p * pl.n * (int64_t)es <= (int64_t)mib << 20;
}
size_t element_size(optcc_dtype_t dtype) {
  return dtype == OPTCC_BF16 || dtype == OPTCC_F16 ? 2 : 4;
}

// choice: not NULL when the call is only asked what it would launch (bufs is not
// looked at).
int emulate(void *const *bufs, int p, int64_t N, optcc_dtype_t dtype, const optcc_plan_t *pl,
            int sb, int se, int launches, void *stream, bool noalloc = false,
            CallChoice *choice = nullptr) {
  set_error("");
  if (!pl) return fail(OPTCC_EINVAL, "plan is NULL");
  if (!bufs && !choice) return fail(OPTCC_EINVAL, "bufs is NULL");
  if (p != pl->p || N != pl->n) return fail(OPTCC_EINVAL, "p or N differ from the plan's");
  if (dtype != OPTCC_F32 && dtype != OPTCC_BF16 && dtype != OPTCC_I32 && dtype != OPTCC_F16)
    return fail(OPTCC_EINVAL, "unknown dtype");
  if (sb < 0 || se > pl->nslots || sb > se)
    return fail(OPTCC_EINVAL, "slot range must satisfy 0 <= begin <= end <= " + std::to_string(pl->nslots));
  if (launches != 0 && launches != 1)
    return fail(OPTCC_EINVAL, "launches must be 0 (one per slot) or 1 (fused)");
  if (p > kMaxRanks) return fail(OPTCC_EUNSUPPORTED, "p exceeds OPTCC_MAX_EMULATE_RANKS");
  if (N == 0 || sb == se) return OPTCC_OK;  // nothing to move; pointers are not touched
  const size_t es = element_size(dtype);
  // pointers: non-NULL, element-aligned, pairwise disjoint
  uintptr_t align = choice ? (uintptr_t)choice->align : kLine;
  std::vector<std::pair<uintptr_t, int>> ranges;
  for (int r = 0; r < p && !choice; ++r) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(bufs[r]);
    if (!a) return fail(OPTCC_EINVAL, "bufs[" + std::to_string(r) + "] is NULL");
    if (a > UINTPTR_MAX - (uintptr_t)N * es)
      return fail(OPTCC_EINVAL, "bufs[" + std::to_string(r) + "] + N elements would run past the end of the address space");
    if (a % es)
      return fail(OPTCC_EINVAL, "bufs[" + std::to_string(r) + "] is not aligned to the element size");
    while (a % align) align /= 2;
    ranges.push_back({a, r});
  }
  std::sort(ranges.begin(), ranges.end());
  for (size_t i = 1; i < ranges.size(); ++i)
    if (ranges[i - 1].first + (uintptr_t)N * es > ranges[i].first)
      return fail(OPTCC_EINVAL, "rank buffers overlap");
  // The device tables index a segment's ring quanta in 32 bits (SegDesc,
  // section_of): refuse a plan whose segments would not fit.
  for (const Segment &s : pl->seg)
    if (s.qbase * (int64_t)pl->pp + s.nbig > (int64_t)INT32_MAX)
      return fail(OPTCC_EUNSUPPORTED, "a segment's ring sections hold 2^31 or more quanta; use "
                                      "more segments (n_chunks) or a smaller N");

  // The launch of the general kernel.  Its rules were chosen on whole AllReduces
  // of every plan, which it ran before the chain kernels; they now decide slot
  // ranges, and whole AllReduces of more than 128 healthy ranks, more than 16
  // stragglers or other numbers of GPUs per server.  The figures beside each are
  // of such calls: us with the rule and without it, "per slot" one launch per
  // slot, "ranges" the slots [0, 2) and [2, 6) (servers: [0, 4) and [4, 12)),
  // one straggler unless said.
  //
  // Tile length: 2048 elements, doubled (up to 8192) while a tile would move
  // less than kTileMinBytes4/2 of algorithmic traffic (about 3p - 2 accesses per
  // element).  Per slot at 2^24: fp32 p = 3 180 and 212, p = 4 209 and 235, bf16
  // p = 3 112 and 151 (ranges 66 and 77); bf16 p = 6 at 2^22 45.6 and 52.9.
  int tile_elems = kTileElems;
  const int64_t per_elem = (3 * (int64_t)p - 2) * (int64_t)es;
  const int64_t min_bytes = es == 2 ? kTileMinBytes2 : kTileMinBytes4;
  while (tile_elems < kTileElemsMax && (int64_t)tile_elems * per_elem < min_bytes) tile_elems *= 2;
  // Small messages: halve the tile, down to one 16-byte vector per lane,
  // while there would be fewer than kTileMinCount tiles, so that more CUs
  // take part.  Per slot, fp32: p = 4 at 2^16 19.6 and 25.2, p = 8 at 2^18 23.5
  // and 27.7, p = 128 (one-vector tiles anyway) at 2^16 49.4 and 49.4.
  const int vec_tile = kern::kThreads * (int)(16 / es);
  while (tile_elems > vec_tile && N / tile_elems < kTileMinCount) tile_elems /= 2;

  // Launch shape.  Short chains (inputs per lane: P' for one GPU per
  // server, p for several) of 32-bit elements: two vectors per lane and per-XCD
  // tile runs; a single hop (two healthy ranks): one vector in the identity
  // order.  Mid-size messages on chains of 3 to 7 healthy ranks (16 MiB to 2 GiB
  // of buffers) take one vector per lane in the identity order, in 1024-element
  // tiles from 5 healthy ranks up: p = 8 at 2^20 per slot 38.9 and 47.3, ranges
  // 20.7 and 23.9, at 2^22 116 and 113 (71.0 and 73.4), p = 4 at 2^23 124 and
  // 141; p = 6 at 2^22 105 and 98, and at 2^24 p = 8 loses: per slot 449 and 377,
  // ranges 264 and 249.
  // Longer chains, 2-byte types too: one vector per lane, one workgroup per CU.
  // Ranges, fp32: 64 ranks at 2^20 140 and 157, at 2^24 2220 and 2413, 128 ranks
  // at 2^24 4718 and 5079; whole: 160 ranks at 2^20 304 and 344, 256 at 2^22 1912
  // and 2200, bf16 256 at 2^21 499 and 608; per slot 64 ranks lose (2^22 686 and
  // 630, 2^24 2948 and 2607).  Server plans of more than 32 ranks: whole, 16 x 6
  // GPUs fp32 at 2^23 1307 and 1414, 40 x 3 1634 and 1728, 20 x 8 at 2^22 1188 and
  // 1262; slot ranges lose: 16 x 4 at 2^22 per slot 1455 and 822, 32 x 4 at 2^23
  // ranges 4372 and 2522.
  const bool servers = pl->kind == OPTCC_KIND_SERVERS;
  const int chain = servers ? pl->p : pl->pp;
  const bool long_chain = chain > kTwoVectorMaxHealthy;
  const bool single_hop = !servers && pl->pp == 2;
  const int64_t buf_bytes = (int64_t)p * N * (int64_t)es;
  const bool mid_short = !servers && es == 4 && pl->pp >= 3 && pl->pp <= kOneVectorMaxHealthy &&
                         buf_bytes >= kOneVectorMinBytes && buf_bytes < kOneVectorMaxBytes;
  if (mid_short && pl->pp >= 5) tile_elems = std::min(tile_elems, vec_tile);
  // Longer one-GPU-per-server chains take one vector per lane per tile too
  // (1024 elements for 32-bit types; 2-byte types have it already), so a
  // workgroup moves on to a new tile after every chain.  fp32 ranges at 2^24: 64
  // ranks 2220 and 2335, 128 ranks 4718 and 4848; whole: 160 ranks at 2^23 2160
  // and 2196, 256 at 2^22 1912 and 2086; per slot 2-8 % slower with it.
  if (long_chain && !servers) tile_elems = std::min(tile_elems, vec_tile);
  const int64_t ntiles = tile_count(*pl, tile_elems);
  if (noalloc && scratch_bytes(*pl, ntiles) > (size_t)OPTCC_NOALLOC_SCRATCH_BYTES)
    return fail(OPTCC_EUNSUPPORTED,
                "the plan's tables need " + std::to_string(scratch_bytes(*pl, ntiles)) +
                    " bytes, more than the " + std::to_string(OPTCC_NOALLOC_SCRATCH_BYTES) +
                    " of the no-allocation scratch array: use optcc_allreduce_emulate");
  const bool two = !long_chain && !single_hop && !mid_short;
  const bool two_vec = two && es == 4;  // two vectors per lane: 32-bit types only
  hipStream_t st = static_cast<hipStream_t>(stream);
  // Whole AllReduces run the chain kernels (slot ranges, longer chains, more
  // stragglers, other server sizes and large buffers off a line the general kernel
  // below: 20 stragglers among 30 ranks of bf16 are 4-18 % faster there; the
  // no-allocation entry point, which stages tables for it, keeps the chain kernel
  // off a line).  They read no tile table;
  // the plan's tables are uploaded on the first call all the same, so that
  // every later call of the plan, a slot range too, may be captured, and the
  // no-allocation entry point refuses the same plans whichever kernel runs.
  const bool whole = launches == 1 && sb == 0 && se == pl->nslots;
  if (takes_chain(*pl, es, sb, se, launches, noalloc ? kLine : align)) {
    if (choice) {
      choice->kernel = servers ? 2 : 1;
      choice->work_items =
          chain_work_items(servers ? server_chain_rule(*pl, es) : chain_rule(*pl, es), N, es);
      return OPTCC_OK;
    }
    if (!noalloc) {
      DeviceTables dt;
      const int rc = device_tables(*pl, tile_elems, st, &dt);
      if (rc != OPTCC_OK) return rc;
    }
    return servers ? launch_server_plan(bufs, *pl, dtype, es, st)
                   : launch_chain_plan(bufs, *pl, dtype, es, st);
  }
  KArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = N;
  a.pp = pl->pp;
  a.m = pl->m;
  a.g = pl->g;
  if (choice) {  // no buffers
  } else if (servers) {  // per server (healthy in ring order, then the straggler): its g GPUs
    const int g = pl->g;
    for (int h = 0; h < pl->pp; ++h)
      for (int l = 0; l < g; ++l) a.ptr[h * g + l] = bufs[pl->ring[(size_t)h] * g + l];
    for (int l = 0; l < g; ++l) a.ptr[pl->pp * g + l] = bufs[pl->strag[0] * g + l];
  } else {
    for (int i = 0; i < pl->pp; ++i) a.ptr[i] = bufs[pl->ring[(size_t)i]];
    for (int i = 0; i < pl->m; ++i) a.ptr[pl->pp + i] = bufs[pl->strag[(size_t)i]];
  }
  int per_cu = long_chain ? 1 : 0;  // workgroups per CU; 0: as many as fit
  // 32-bit chains of 11-32 healthy ranks (one GPU per server, two vectors
  // per lane, 181 VGPRs: two workgroups per CU) with at most one straggler, and
  // server plans of at most 32 ranks with 4 or more GPUs per server, run
  // one workgroup per CU too from kTwoVecOnePerCuMinBytes of rank buffers.
  // Whole, fp32 at 2^24: 3 x 6 GPUs 467 and 476, 4 x 5 525 and 529; 16 ranks at
  // 2^25 ranges 1136 and 1140; per slot it loses: 16 ranks 1578 and 1403, 12
  // 1311 and 1123, 32 ranks int32 at 2^24 1411 and 1328, 4 x 4 GPUs 1551 and 1039.
  const bool two_vec_one_per_cu =
      servers ? pl->g >= 4 : (pl->m <= 1 && pl->pp >= kTwoVecOnePerCuMinHealthy);
  if (two_vec && two_vec_one_per_cu && buf_bytes >= kTwoVecOnePerCuMinBytes)
    per_cu = 1;
  // The mid-size short chains of 6 or 7 healthy ranks with at least
  // kThreePerCuMinBytes of rank buffers run at three workgroups per CU instead of
  // the four their registers allow.  It was worth 1.5-5 % to whole AllReduces
  // from 480 MiB to 1.75 GiB, which run the chain kernel now; slot ranges lose by
  // it (p = 8 fp32 at 2^24 per slot 449 and 401, ranges 264 and 251, int32 at 2^25
  // per slot 858 and 776).
  if (mid_short && pl->pp >= kThreePerCuMinHealthy && buf_bytes >= kThreePerCuMinBytes)
    per_cu = 3;
  // bf16 chains of kBf16ThreePerCuMinHealthy to kTwoVectorMaxHealthy
  // healthy ranks (one GPU per server) run at three workgroups per CU as well:
  // 16 ranks at 2^24 ranges 262 and 266; per slot it loses, 362 and 347, 24 ranks
  // at 2^22 134 and 130.
  if (!servers && dtype == OPTCC_BF16 && pl->pp >= kBf16ThreePerCuMinHealthy &&
      pl->pp <= kTwoVectorMaxHealthy)
    per_cu = 3;
  a.occ_lds = per_cu ? workgroups_per_cu_lds(per_cu) : 0;
  // The same mid-size short chains take each vector's Stage 4 stores into
  // the next vector's Stage 1 chain (the kernel's pipelined ring tiles) when the
  // launch is a whole AllReduce, which has more than 16 stragglers then.  With 17,
  // fp32: 3 healthy ranks at 2^22 135 and 155, 7 at 2^24 601 and 610, at 2^22 171
  // and 171, at 2^20 35.8 and 35.4; int32 5 at 2^22 141 and 141, at 2^24 575 and
  // 569.
  a.pipe = mid_short ? 1 : 0;
  // Long 32-bit chains (one GPU per server) with at least
  // kHopWindowWideMinElems elements per rank keep kHopWindowWide hop loads
  // in flight per vector instead of kHopWindow: 64 ranks at 2^24 per slot 2948
  // and 2964, ranges 2220 and 2234, 128 ranks 4718 and 4728, whole 160 ranks at
  // 2^23 2160 and 2172.
  a.wide_window = long_chain && !servers && es == 4 && N >= kHopWindowWideMinElems ? 1 : 0;
  // Ordinary instead of streaming accesses (one GPU per server) where the
  // memory-side cache holds the buffers between launches: slot ranges up to
  // kKeptMaxBytes of rank buffers, whole AllReduces of more healthy ranks than
  // the chain kernel takes up to kKeptWholeMaxBytes.  Measured, streaming ->
  // ordinary, one slot per launch, on three sets of buffers in turn: 48 MiB
  // p = 4 fp32 62.9 -> 54.5 us, p = 8 57.3 -> 52.9, 16 ranks bf16 47.9 -> 44.0,
  // 128 ranks 62.3 -> 51.9; 96 MiB 14 % faster to 2 % slower; 128 MiB 6 % faster
  // to 5 % slower (on the same buffers 8-28 % faster up to 192 MiB).  160 ranks
  // whole: 48 MiB 56.7 -> 39.5 us, 72 MiB 71 -> 42, 192 MiB 149 -> 136, 320 MiB
  // 10 % faster to 4 % slower.  Server plans: -15 to +8 %, so they stay with streaming.
  a.kept = !servers && (whole ? pl->pp > kChainMaxHealthy && buf_bytes <= kKeptWholeMaxBytes
                              : buf_bytes <= kKeptMaxBytes);
  bool runs = servers || two;
  // Per-XCD runs for long chains with more than one round of resident
  // workgroups, up to kXcdRunsMaxTiles tiles, kXcdRunsMaxTilesMid with fewer than
  // kXcdRunsWideHealthy healthy ranks; beyond, stealing.  fp32, 64 ranks at 2^20
  // (1024 tiles) per slot 173 and 248, ranges 140 and 169, at 2^22 (4096) per slot
  // 686 and 796; whole: 160 ranks at 2^20 304 and 326, bf16 256 ranks at 2^21 499
  // and 533.
  const int64_t runs_max = pl->pp < kXcdRunsWideHealthy ? kXcdRunsMaxTilesMid : kXcdRunsMaxTiles;
  if (long_chain && !servers && ntiles <= runs_max) {
    const int resident = resident_workgroups(a, dtype, servers, two_vec);
    runs = resident <= 0 || ntiles > resident;
  }
  // Server plans of at least kXcdRunsWideHealthy ranks (one workgroup per
  // CU) with more than kServerStealMinTiles tiles (kXcdRunsMaxTiles from
  // kServerStealWideRanks ranks) take work stealing (below) instead of the
  // per-XCD runs, when it is available; otherwise the runs.  Whole at 2^23-2^24:
  // 16 x 6 GPUs fp32 1307 and 1340, bf16 1264 and 1343, 40 x 3 fp32 1634 and 1663;
  // ranges, 32 x 4 fp32 at 2^23 4372 and 4392 (per slot 5635 and 5573).  Without
  // the runs, at fewer tiles: 20 x 8 GPUs at 2^22 1188 and 1322, 40 x 4 at 2^20 310
  // and 397.
  const int64_t server_steal_min =
      pl->p >= kServerStealWideRanks ? kXcdRunsMaxTiles : kServerStealMinTiles;
  const bool server_steal = servers && long_chain && pl->p >= kXcdRunsWideHealthy &&
                            ntiles > server_steal_min && !noalloc;
  if (server_steal) runs = false;
  a.xcd_runs = runs ? 1 : 0;
  // Work stealing for the same long chains at one workgroup per CU when
  // their tiles take the identity order (more than runs_max): a
  // grid of the resident workgroups takes tiles from a device counter.  The
  // eight XCDs do not run equally fast (per-wave timestamps of 128 ranks:
  // XCDs 1, 3, 5, 7 spend about 5 % longer per tile than 0, 2, 4, 6), and
  // with one eighth of the tiles each the fast ones wait at the end.  fp32 at
  // 2^24, ranges: 64 ranks 2220 and 2320, 128 ranks 4718 and 5073, per slot 5396
  // and 5576 (64 ranks 2948 and 2849); bf16 128 ranks at 2^23 per slot 1464 and
  // 1499; whole: 160 ranks at 2^23 2160 and 2252, 256 at 2^22 1912 and 1866.  Not
  // under graph capture: a captured launch keeps its counter block, and replays
  // of the graph on two streams at once would share it; the no-allocation entry
  // point keeps the static order too.
  bool steal = long_chain && (!servers || server_steal) && a.occ_lds > 0 && !runs && !noalloc;
  int steal_grid = 0;
  if (steal) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    steal = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
  }
  if (steal) {
    steal_grid = resident_workgroups(a, dtype, servers, two_vec);
    steal = steal_grid > 0 && steal_grid < ntiles;
  }
  if (server_steal && !steal) a.xcd_runs = 1;  // captured: the server plans' runs
  if (choice) {
    choice->tile_elems = tile_elems;
    choice->two = two_vec;
    choice->per_cu = per_cu;
    choice->wide_window = a.wide_window;
    choice->pipe = a.pipe && whole;
    choice->kept = a.kept;
    choice->xcd_runs = a.xcd_runs;
    choice->steal = steal;
    return OPTCC_OK;
  }
  DeviceTables dt;
  int rc = noalloc ? scratch_tables(*pl, tile_elems, st, &dt)
                   : device_tables(*pl, tile_elems, st, &dt);
  if (rc != OPTCC_OK) return rc;
  a.tiles = dt.tiles;
  a.segs = dt.segs;
  a.ntiles = dt.ntiles;
  uint32_t *counters = steal ? steal_counters(*pl, tile_elems) : nullptr;
  if (counters) {
    // one counter block per launch, round robin over kStealSlots: launches
    // in flight at once (any streams) use different blocks
    const uint32_t slot = pl->steal_next.fetch_add(1u, std::memory_order_relaxed) % kStealSlots;
    a.steal = counters + (size_t)slot * kStealWords;
    a.grid = steal_grid;
  }
  const int nl = launches == 1 ? 1 : se - sb;
  for (int l = 0; l < nl; ++l) {
    a.sb = launches == 1 ? sb : sb + l;
    a.se = launches == 1 ? se : sb + l + 1;
    hipError_t err = hipSuccess;
    switch (dtype) {
      case OPTCC_F32: err = launch_f32(a, servers, two_vec, st); break;
      case OPTCC_BF16: err = launch_bf16(a, servers, two_vec, st); break;
      case OPTCC_F16: err = launch_f16(a, servers, two_vec, st); break;
      default: err = launch_i32(a, servers, two_vec, st); break;
    }
    if (err != hipSuccess)
      return fail(OPTCC_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(err));
  }
  return OPTCC_OK;
}

}  // namespace
}  // namespace optcc

using namespace optcc;

extern "C" int optcc_allreduce_emulate(void *const *bufs, int p, int64_t N, optcc_dtype_t dtype,
                                       const optcc_plan_t *plan, void *stream) {
  return emulate(bufs, p, N, dtype, plan, 0, plan ? plan->nslots : OPTCC_NUM_SLOTS, 1, stream);
}

extern "C" int optcc_allreduce_emulate_slots(void *const *bufs, int p, int64_t N,
                                             optcc_dtype_t dtype, const optcc_plan_t *plan,
                                             int slot_begin, int slot_end, int launches,
                                             void *stream) {
  return emulate(bufs, p, N, dtype, plan, slot_begin, slot_end, launches, stream);
}

extern "C" int optcc_allreduce_emulate_noalloc(void *const *bufs, int p, int64_t N,
                                               optcc_dtype_t dtype, const optcc_plan_t *plan,
                                               void *stream) {
  return emulate(bufs, p, N, dtype, plan, 0, plan ? plan->nslots : OPTCC_NUM_SLOTS, 1, stream,
                 true);
}

extern "C" int optcc_call_choice(const optcc_plan_t *pl, int dtype, int slot_begin, int slot_end,
                                 int launches, int noalloc, int align, void *stream,
                                 optcc::CallChoice *out) {
  *out = optcc::CallChoice();
  out->align = align;
  return emulate(nullptr, pl->p, pl->n, (optcc_dtype_t)dtype, pl, slot_begin, slot_end, launches,
                 stream, noalloc != 0, out);
}

extern "C" void optcc_plan_free(optcc_plan_t *pl) {
  if (!pl) return;
  if (!pl->dev.empty()) {
    std::lock_guard<std::mutex> lk(pl->mu);
    int cur = -1;
    const bool have_dev = hipGetDevice(&cur) == hipSuccess;
    for (auto &kv : pl->dev) {
      if (have_dev) (void)hipSetDevice(kv.first.first);
      (void)hipFree(kv.second.segs);
      (void)hipFree(kv.second.tiles);
      (void)hipFree(kv.second.steal);
    }
    if (have_dev && !pl->dev.empty()) (void)hipSetDevice(cur);
    pl->dev.clear();
  }
  delete pl;
}
