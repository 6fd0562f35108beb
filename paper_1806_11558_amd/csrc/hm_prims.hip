// Device-wide primitives: exclusive scan and a stable LSD radix sort.
//
// The level-wise tree construction and traversal of Sec. 3.1 ("Block cluster
// tree traversal") compute output offsets by parallel scans; the Morton
// clustering ("Spatial data structure") needs a parallel sort.  Both are
// written here for wave64: the sort ranks keys inside a wavefront with
// ballots (no atomics on the ranking path), so it is stable and
// deterministic.
#include <map>
#include <mutex>

#include "hm_internal.h"

namespace hm {

// ------------------------------------------------------------------ memory
// All device memory of the library comes from one stream-ordered pool per
// device, created on first use.  Freed memory stays cached in the pool (its
// release threshold is unlimited), so a rebuild reuses it instead of going
// back to the driver: allocations of recently freed device memory wait for
// the driver to clear it, which cost seconds for tens of GB.  trim_pool()
// (hm_release_memory) hands the cache back.
namespace {
constexpr uint64_t kPoolKeep = ~uint64_t(0);
std::mutex g_pool_mu;
hipMemPool_t g_pool[64] = {};
}  // namespace

hipMemPool_t lib_pool() {
  int dev = 0;
  HM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) throw Error{HM_ERR_HIP, "device index out of range"};
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (!g_pool[dev]) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool = nullptr;
    HM_HIP(hipMemPoolCreate(&pool, &props));
    uint64_t keep = kPoolKeep;
    HM_HIP(hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep));
    g_pool[dev] = pool;
  }
  return g_pool[dev];
}

void trim_pool() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (g_pool[dev]) (void)hipMemPoolTrimTo(g_pool[dev], 0);
  (void)hipGetLastError();
}

// Blocks of freed handles, per device, by size.  A later build that asks for
// a block of about the same size (at most 1/8 larger) takes it back, so that
// rebuilding a problem reuses its storage instead of fresh driver memory.
namespace {
std::mutex g_cache_mu;
std::multimap<size_t, void*> g_cache[64];
}  // namespace

void* cache_take(size_t bytes, size_t* got) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  auto& c = g_cache[dev];
  auto it = c.lower_bound(bytes);
  if (it == c.end() || it->first > bytes + bytes / 8) return nullptr;
  void* p = it->second;
  *got = it->first;
  c.erase(it);
  return p;
}

void cache_put(void* p, size_t bytes) {
  int dev = 0;
  if (!p || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  g_cache[dev].emplace(bytes, p);
}

void cache_release() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  for (auto& e : g_cache[dev]) (void)hipFreeAsync(e.second, nullptr);
  g_cache[dev].clear();
  (void)hipStreamSynchronize(nullptr);
}

void* dalloc(size_t bytes, hipStream_t s) {
  if (bytes <= BuildArena::kArenaMax)
    if (BuildArena* a = BuildArena::current(s)) return a->get(bytes);
  return dalloc_pool(bytes, s);
}

// A device that is full may be so because of blocks kept for later builds: they
// go back, and the request is made once more.
void* dalloc_pool(size_t bytes, hipStream_t s) {
  void* p = nullptr;
  if (bytes == 0) bytes = 16;
  for (int again = 0; again < 2; ++again) {
    const hipError_t e = hipMallocFromPoolAsync(&p, bytes, lib_pool(), s);
    if (e == hipSuccess && p != nullptr) return p;
    (void)hipGetLastError();
    if (e != hipErrorOutOfMemory || again) break;
    cache_release();
    trim_pool();
  }
  throw Error{HM_ERR_OOM, "device allocation of " + std::to_string(bytes) + " bytes failed"};
}

void dfree(void* p, hipStream_t s) {
  if (!p) return;
  if (BuildArena* a = BuildArena::current(s))
    if (a->put(p)) return;
  (void)hipFreeAsync(p, s);
}

// ---- arena of a build
namespace {
thread_local BuildArena* t_arena = nullptr;
// pinned pages not in use, at most kKeepPages (one per build or solve running
// at once)
constexpr size_t kKeepPages = 8;
std::mutex g_page_mu;
std::vector<int64_t*> g_pages;
}  // namespace

int64_t* page_take(bool may_allocate) {
  {
    std::lock_guard<std::mutex> lk(g_page_mu);
    if (!g_pages.empty()) {
      int64_t* p = g_pages.back();
      g_pages.pop_back();
      return p;
    }
  }
  int64_t* p = nullptr;
  if (may_allocate)
    HM_HIP(hipHostMalloc((void**)&p, kPageWords * sizeof(int64_t),
                         hipHostMallocPortable | hipHostMallocMapped));
  return p;
}

void page_give(int64_t* p) {
  {
    std::lock_guard<std::mutex> lk(g_page_mu);
    if (g_pages.size() < kKeepPages) {
      g_pages.push_back(p);
      return;
    }
  }
  (void)hipHostFree(p);
}

BuildArena* BuildArena::current(hipStream_t s) {
  return t_arena && t_arena->stream == s ? t_arena : nullptr;
}

BuildArena::BuildArena(hipStream_t s) : stream(s) {
  host = page_take(true);
  outer_ = t_arena;
  t_arena = this;
}

BuildArena::~BuildArena() {
  t_arena = outer_;
  // nothing in flight may still use the chunks or the page
  (void)hipStreamSynchronize(stream);
  for (auto& c : chunks_) cache_put(c.first, c.second);
  page_give(host);
}

// Sizes rounded up to four steps per power of two, at least 256 bytes, so
// that freed blocks fit later requests of about their size.
size_t BuildArena::round_up(size_t b) {
  size_t step = 256;
  while (step * 8 < b) step <<= 1;
  return (b + step - 1) / step * step;
}

void* BuildArena::get(size_t bytes) {
  const size_t b = round_up(bytes > 0 ? bytes : 1);
  auto& f = free_[b];
  if (!f.empty()) {
    void* p = f.back();
    f.pop_back();
    return p;
  }
  if (chunks_.empty() || used_ + b > chunks_.back().second) {
    size_t got = kChunk;
    void* q = cache_take(kChunk, &got);
    if (!q) {
      q = dalloc_pool(kChunk, stream);
      got = kChunk;
    }
    chunks_.push_back({static_cast<char*>(q), got});
    used_ = 0;
  }
  void* p = chunks_.back().first + used_;
  used_ += b;
  size_[p] = b;
  return p;
}

bool BuildArena::put(void* p) {
  auto it = size_.find(p);
  if (it == size_.end()) return false;
  free_[it->second].push_back(p);
  return true;
}

// Device copies of a build: a launch costs the host 3 us, hipMemcpyAsync
// between device buffers 12 us (46 of them in a build).  Both addresses are
// 16-byte aligned at their start (allocations are).
__global__ __launch_bounds__(256) void k_copy(const uint4* __restrict__ a, uint4* __restrict__ b,
                                              int64_t n16, int tail) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16;
       i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
  if (blockIdx.x == 0 && (int)threadIdx.x < tail)
    reinterpret_cast<char*>(b + n16)[threadIdx.x] = reinterpret_cast<const char*>(a + n16)[threadIdx.x];
}
// The same for addresses that are only 4-byte aligned.
__global__ __launch_bounds__(256) void k_copy4(const uint32_t* __restrict__ a,
                                               uint32_t* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

void copy_d2d(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return;
  if ((((uintptr_t)dst | (uintptr_t)src) & 15) == 0) {
    const int64_t n16 = (int64_t)(bytes / 16);
    k_copy<<<grid_for(n16, 256, 8192), 256, 0, s>>>((const uint4*)src, (uint4*)dst, n16,
                                                    (int)(bytes % 16));
  } else {                                              // every table has 4-byte entries or larger
    const int64_t n = (int64_t)(bytes / 4);
    k_copy4<<<grid_for(n, 256, 8192), 256, 0, s>>>((const uint32_t*)src, (uint32_t*)dst, n);
  }
  HM_LAUNCH_CHECK();
}

// *dst = *src for n words (dst: pinned host memory).
__global__ void k_words(const int64_t* __restrict__ src, int n, int64_t* __restrict__ dst) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}

void d2h_words(const int64_t* d, int n, int64_t* out, hipStream_t s) {
  int64_t* h = host_words(s);
  if (h && n <= 64) {
    k_words<<<1, 64, 0, s>>>(d, n, h);
    HM_LAUNCH_CHECK();
    HM_HIP(hipStreamSynchronize(s));
    for (int k = 0; k < n; ++k) out[k] = ((volatile int64_t*)h)[k];
    return;
  }
  HM_HIP(hipMemcpyAsync(out, d, n * sizeof(int64_t), hipMemcpyDeviceToHost, s));
  HM_HIP(hipStreamSynchronize(s));
}

int64_t d2h_i64(const int64_t* d, hipStream_t s) {
  int64_t v = 0;
  d2h_words(d, 1, &v, s);
  return v;
}

int64_t scan_total(const int64_t* in, int64_t* out, int64_t n, int64_t* tmp, hipStream_t s) {
  if (int64_t* h = host_words(s)) {                     // the scan writes the total to the host
    scan_excl_i64(in, out, n, h, s);
    HM_HIP(hipStreamSynchronize(s));
    return *(volatile int64_t*)h;
  }
  scan_excl_i64(in, out, n, tmp, s);
  return d2h_i64(tmp, s);
}

// ------------------------------------------------------------------ scan
namespace {
constexpr int kScanThreads = 256;
constexpr int kScanPer = 4;
constexpr int kScanTile = kScanThreads * kScanPer;   // 1024

__device__ inline int64_t wave_incl_scan(int64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int64_t t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ inline int64_t block_excl_scan(int64_t v, int64_t* out, int64_t* lds_w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t inc = wave_incl_scan(v);
  if (lane == 63) lds_w[wave] = inc;
  __syncthreads();
  int64_t wpre = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    int64_t x = lds_w[w];
    if (w < wave) wpre += x;
    total += x;
  }
  *out = wpre + inc - v;
  __syncthreads();
  return total;
}

__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const int64_t* in, int64_t n,
                                                            int64_t* sums) {
  __shared__ int64_t lds_w[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int64_t v = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    int64_t i = base + (int64_t)threadIdx.x * kScanPer + k;
    if (i < n) v += in[i];
  }
  int64_t ex;
  int64_t total = block_excl_scan(v, &ex, lds_w);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// out[i] = offs[tile] + the exclusive prefix of in within the tile; the
// thread of element n - 1 also writes the grand total when total is given.
__global__ __launch_bounds__(kScanThreads) void k_tile_apply(const int64_t* in, int64_t* out,
                                                             int64_t n, const int64_t* offs,
                                                             int64_t* total) {
  __shared__ int64_t lds_w[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int64_t loc[kScanPer];
  int64_t v = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    int64_t i = base + (int64_t)threadIdx.x * kScanPer + k;
    loc[k] = (i < n) ? in[i] : 0;
    v += loc[k];
  }
  int64_t ex;
  block_excl_scan(v, &ex, lds_w);
  int64_t run = ex + (offs ? offs[blockIdx.x] : 0);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    int64_t i = base + (int64_t)threadIdx.x * kScanPer + k;
    if (i < n) out[i] = run;
    if (total && i == n - 1) *total = run + loc[k];
    run += loc[k];
  }
}
}  // namespace

// The whole scan in one workgroup of 1,024 threads, 4,096 values at a time
// with a running total.  Up to kScanOne values: the three launches of the
// tiled form cost 3 x 2 us on the device and as much again on the host, four
// rounds here 6 us.
namespace {
constexpr int kScanOneThreads = 1024;
constexpr int64_t kScanOne = 4 * 4 * kScanOneThreads;   // 16,384
__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const int64_t* in, int64_t* out,
                                                              int n, int64_t* total) {
  __shared__ int64_t lds_w[kScanOneThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t carry = 0;
  for (int base = 0; base < n; base += 4 * kScanOneThreads) {
    const int i0 = base + 4 * (int)threadIdx.x;
    int64_t loc[4], v = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      loc[k] = i0 + k < n ? in[i0 + k] : 0;
      v += loc[k];
    }
    const int64_t inc = wave_incl_scan(v);
    if (lane == 63) lds_w[wave] = inc;
    __syncthreads();
    int64_t pre = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kScanOneThreads / 64; ++w) {
      const int64_t x = lds_w[w];
      if (w < wave) pre += x;
      sum += x;
    }
    int64_t run = carry + pre + inc - v;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k < n) out[i0 + k] = run;
      run += loc[k];
    }
    carry += sum;
    __syncthreads();                                    // lds_w is read
  }
  if (total && threadIdx.x == 0) *total = carry;
}
}  // namespace

void scan_excl_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* d_total, hipStream_t s) {
  if (n <= 0) {
    if (d_total) {
      k_scan_one<<<1, kScanOneThreads, 0, s>>>(in, out, 0, d_total);
      HM_LAUNCH_CHECK();
    }
    return;
  }
  const int64_t tiles = ceil_div(n, kScanTile);
  if (tiles == 1) {
    k_tile_apply<<<1, kScanThreads, 0, s>>>(in, out, n, nullptr, d_total);
    HM_LAUNCH_CHECK();
  } else if (n <= kScanOne) {
    k_scan_one<<<1, kScanOneThreads, 0, s>>>(in, out, (int)n, d_total);
    HM_LAUNCH_CHECK();
  } else {
    int64_t* sums = dalloc_t<int64_t>(tiles, s);
    int64_t* offs = dalloc_t<int64_t>(tiles, s);
    k_tile_sums<<<(unsigned)tiles, kScanThreads, 0, s>>>(in, n, sums);
    HM_LAUNCH_CHECK();
    scan_excl_i64(sums, offs, tiles, nullptr, s);
    k_tile_apply<<<(unsigned)tiles, kScanThreads, 0, s>>>(in, out, n, offs, d_total);
    HM_LAUNCH_CHECK();
    dfree(sums, s);
    dfree(offs, s);
  }
}

// ------------------------------------------------------------------ radix sort
namespace {
constexpr int kRadixThreads = 256;
constexpr int kRadixWaves = kRadixThreads / 64;
constexpr int kRadixPer = 4;                             // sub-rounds per tile
constexpr int kRadixTile = kRadixThreads * kRadixPer;    // 1024 keys
constexpr int kBins = 256;

__device__ inline uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Up to kRadixDirect tiles every workgroup of the scatter adds the tile
// histograms in front of it itself; the scan of the 256 x tiles counts (one
// to three launches a pass) is then not needed.
constexpr int64_t kRadixDirect = 64;

// Histogram of one digit per tile, stored tile-major: hist[tile * 256 + d].
__global__ __launch_bounds__(kRadixThreads) void k_radix_hist_t(const uint64_t* keys, int64_t n,
                                                                int shift, int32_t* hist) {
  __shared__ int cnt[kBins];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRadixTile;
  for (int k = 0; k < kRadixPer; ++k) {
    int64_t i = base + (int64_t)k * kRadixThreads + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(int)((keys[i] >> shift) & 0xFF)], 1);
  }
  __syncthreads();
  hist[(int64_t)blockIdx.x * kBins + threadIdx.x] = cnt[threadIdx.x];
}

// Histogram of one digit per tile, stored digit-major: hist[d * tiles + tile].
__global__ __launch_bounds__(kRadixThreads) void k_radix_hist(const uint64_t* keys, int64_t n,
                                                              int shift, int64_t tiles,
                                                              int64_t* hist) {
  __shared__ int cnt[kBins];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRadixTile;
  for (int k = 0; k < kRadixPer; ++k) {
    int64_t i = base + (int64_t)k * kRadixThreads + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(int)((keys[i] >> shift) & 0xFF)], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * tiles + blockIdx.x] = cnt[threadIdx.x];
}

// Stable scatter: keys of a tile are visited in index order, ranked inside
// each wavefront by ballot matching, then across wavefronts via LDS.  The
// start of digit d in this tile comes from the scanned counts (offs), or,
// with `hist` (tile-major counts), from the counts of the tiles in front and
// of the smaller digits.
__global__ __launch_bounds__(kRadixThreads) void k_radix_scatter(
    const uint64_t* kin, const int32_t* vin, uint64_t* kout, int32_t* vout, int64_t n, int shift,
    int64_t tiles, const int64_t* offs, const int32_t* hist) {
  __shared__ int wcnt[kRadixWaves][kBins];
  __shared__ int run[kBins];
  __shared__ int64_t start[kBins];
  __shared__ int64_t wtot[kRadixWaves];
  const int wave = threadIdx.x >> 6;
  run[threadIdx.x] = 0;
  if (hist) {                                           // thread t owns digit t
    int before = 0, all = 0;
#pragma unroll 8
    for (int t = 0; t < (int)tiles; ++t) {
      const int c = hist[t * kBins + threadIdx.x];
      before += t < (int)blockIdx.x ? c : 0;
      all += c;
    }
    const int64_t inc = wave_incl_scan(all);
    if ((threadIdx.x & 63) == 63) wtot[wave] = inc;
    __syncthreads();
    int64_t pre = inc - all;
    for (int w = 0; w < wave; ++w) pre += wtot[w];
    start[threadIdx.x] = pre + before;
  } else {
    start[threadIdx.x] = offs[(int64_t)threadIdx.x * tiles + blockIdx.x];
  }
  const int64_t base = (int64_t)blockIdx.x * kRadixTile;
  for (int k = 0; k < kRadixPer; ++k) {
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) wcnt[w][threadIdx.x] = 0;
    __syncthreads();
    const int64_t i = base + (int64_t)k * kRadixThreads + threadIdx.x;
    const bool valid = i < n;
    uint64_t key = valid ? kin[i] : 0;
    int32_t val = valid ? vin[i] : 0;
    const int d = (int)((key >> shift) & 0xFF);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const int rank = (int)lanes_below(peers);
    const int npeers = __popcll(peers);
    if (valid && rank == npeers - 1) wcnt[wave][d] = npeers;   // last peer writes the count
    __syncthreads();
    {
      // thread t owns digit t: turn per-wave counts into exclusive offsets
      const int t = threadIdx.x;
      int acc = run[t];
#pragma unroll
      for (int w = 0; w < kRadixWaves; ++w) {
        int c = wcnt[w][t];
        wcnt[w][t] = acc;
        acc += c;
      }
      run[t] = acc;
    }
    __syncthreads();
    if (valid) {
      int64_t pos = start[d] + wcnt[wave][d] + rank;
      kout[pos] = key;
      vout[pos] = val;
    }
    __syncthreads();
  }
}
}  // namespace

// Up to kSortRank pairs: the position of a pair is the number of pairs in front
// of it, counted against all keys (equal keys: by index, so the order is
// stable; keys have no bits at or above `bits`, so comparing them whole is the
// same order).  Lane = pair, the wavefronts of a workgroup share the keys,
// which come as scalar loads, two instructions per comparison (keys staged in
// LDS or handed round by readlane took longer: 14 and 12 us at 2,880 pairs).
// 1,280 pairs 7 us and 2,880 12 us, in one workgroup's LDS by a bitonic network
// 39 us, by eight radix passes more than 100; at 16,000 pairs it saves nothing
// over the radix passes.
constexpr int kSortRank = 8192, kSortThreads = 1024, kSortWaves = kSortThreads / 64;
__global__ __launch_bounds__(kSortThreads) void k_sort_rank(const uint64_t* __restrict__ keys,
                                                            const int32_t* __restrict__ vals, int n,
                                                            uint64_t* __restrict__ kout,
                                                            int32_t* __restrict__ vout) {
  __shared__ int part[kSortWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = blockIdx.x * 64, i = i0 + lane;
  const uint64_t mine = keys[min(i, n - 1)];
  const int per = (n + kSortWaves - 1) / kSortWaves;
  const int j0 = min(n, wave * per), j1 = min(n, j0 + per);
  int r = 0;
  // keys in front of, among and behind the workgroup's own
#pragma unroll 8
  for (int j = j0; j < min(j1, i0); ++j) r += keys[j] <= mine;
  for (int j = max(j0, i0); j < min(j1, i0 + 64); ++j) {
    const uint64_t k = keys[j];
    r += k < mine || (k == mine && j < i);
  }
#pragma unroll 8
  for (int j = max(j0, i0 + 64); j < j1; ++j) r += keys[j] < mine;
  part[wave][lane] = r;
  __syncthreads();
  if (wave == 0 && i < n) {
    int pos = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) pos += part[w][lane];
    kout[pos] = mine;
    vout[pos] = vals[i];
  }
}

__global__ void k_copy_pairs(const uint64_t* __restrict__ ki, const int32_t* __restrict__ vi, int n,
                             uint64_t* __restrict__ ko, int32_t* __restrict__ vo) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    ko[i] = ki[i];
    vo[i] = vi[i];
  }
}

void radix_sort_u64_i32(uint64_t* keys, int32_t* vals, int64_t n, int bits, hipStream_t s) {
  if (n <= 1 || bits <= 0) return;
  if (n <= kSortRank) {
    uint64_t* k2 = dalloc_t<uint64_t>(n, s);
    int32_t* v2 = dalloc_t<int32_t>(n, s);
    k_sort_rank<<<(unsigned)ceil_div(n, 64), kSortThreads, 0, s>>>(keys, vals, (int)n, k2, v2);
    HM_LAUNCH_CHECK();
    k_copy_pairs<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(k2, v2, (int)n, keys, vals);
    HM_LAUNCH_CHECK();
    dfree(k2, s);
    dfree(v2, s);
    return;
  }
  const int passes = (bits + 7) / 8;
  const int64_t tiles = ceil_div(n, kRadixTile);
  const bool direct = tiles <= kRadixDirect;
  uint64_t* k2 = dalloc_t<uint64_t>(n, s);
  int32_t* v2 = dalloc_t<int32_t>(n, s);
  int64_t* hist = dalloc_t<int64_t>(tiles * kBins, s);
  int64_t* offs = direct ? nullptr : dalloc_t<int64_t>(tiles * kBins, s);
  uint64_t *ka = keys, *kb = k2;
  int32_t *va = vals, *vb = v2;
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    if (direct) {
      k_radix_hist_t<<<(unsigned)tiles, kRadixThreads, 0, s>>>(ka, n, shift, (int32_t*)hist);
    } else {
      k_radix_hist<<<(unsigned)tiles, kRadixThreads, 0, s>>>(ka, n, shift, tiles, hist);
      HM_LAUNCH_CHECK();
      scan_excl_i64(hist, offs, tiles * kBins, nullptr, s);
    }
    HM_LAUNCH_CHECK();
    k_radix_scatter<<<(unsigned)tiles, kRadixThreads, 0, s>>>(
        ka, va, kb, vb, n, shift, tiles, offs, direct ? (const int32_t*)hist : nullptr);
    HM_LAUNCH_CHECK();
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  if (ka != keys) {
    copy_d2d(keys, ka, n * sizeof(uint64_t), s);
    copy_d2d(vals, va, n * sizeof(int32_t), s);
  }
  dfree(k2, s);
  dfree(v2, s);
  dfree(hist, s);
  if (offs) dfree(offs, s);
}

}  // namespace hm
