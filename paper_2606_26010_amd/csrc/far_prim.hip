// far_prim.hip -- device-wide primitives: stable LSD radix sort of (uint64 key,
// uint32 value) pairs and an exclusive prefix sum, written for wave64.
//
// The insert needs a *stable* grouping of points by voxel key so that each
// voxel's candidates are visited in input order (the sequential capped-insert
// semantics); an LSD radix sort whose every pass is stable gives exactly that.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstring>
#include <mutex>
#include <utility>
#include <vector>

#include "far_internal.h"

namespace far {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// ---------------------------------------------------------------- scan
constexpr int kScanItems = 8;
constexpr int kScanTile = kThreads * kScanItems;

// Exclusive scan of one value per thread across the block; returns the
// thread's exclusive prefix and writes the block total.
__device__ inline uint32_t block_exscan(uint32_t v, uint32_t* lds, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds[wave] = x;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    uint32_t s = lds[w];
    pre += (w < wave) ? s : 0u;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

__global__ __launch_bounds__(kThreads) void k_scan_tile_sums(const uint32_t* in, int64_t n,
                                                             uint32_t* sums) {
  __shared__ uint32_t lds[kWaves];
  int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) s += (base + j < n) ? in[base + j] : 0u;
  uint32_t tot;
  (void)block_exscan(s, lds, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Scan each tile, adding carry[blockIdx.x] (scanned tile sums) when given.
// The last tile writes the grand total.
__global__ __launch_bounds__(kThreads) void k_scan_tiles(const uint32_t* in, uint32_t* out,
                                                         int64_t n, const uint32_t* carry,
                                                         uint32_t* total) {
  __shared__ uint32_t lds[kWaves];
  int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = (base + j < n) ? in[base + j] : 0u;
    s += v[j];
  }
  uint32_t tot;
  uint32_t pre = block_exscan(s, lds, &tot);
  uint32_t c = carry ? carry[blockIdx.x] : 0u;
  uint32_t run = c + pre;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    if (base + j < n) out[base + j] = run;
    run += v[j];
  }
  if (total && threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *total = c + tot;
}

// ---------------------------------------------------------------- radix sort
// Each pass is a histogram of every tile and a scatter; a tile is kThreads *
// kItems elements.  Jobs of up to kOwnTiles tiles give every scatter block the
// histograms themselves (kOwn): it adds up the tiles' rows (at most kOwnTiles
// words per lane), so that a pass is two launches instead of
// three to five, and their tiles are smaller, so that 15k points (4 blocks of
// 4096) still spread over the chip.  Larger jobs take the scanned table: the
// rows would cost each block 1 kB a tile.  A pass over 100k pairs: 24 us in
// five launches of 4096-element tiles before, 13 us now; over 5k to 13k pairs
// 15 -> 8.6 us; over 512k pairs 27 -> 21 us.
constexpr int kOwnTiles = 128;

template <int kItems, bool kOwn>
__global__ __launch_bounds__(kThreads) void k_rs_hist(const uint64_t* keys, int64_t n,
                                                      int shift, uint32_t* hist,
                                                      int64_t nblocks) {
  __shared__ uint32_t cnt[256];
  cnt[threadIdx.x] = 0;
  const int64_t base = int64_t(blockIdx.x) * (kThreads * kItems);
  uint64_t k[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + int64_t(r) * kThreads + threadIdx.x;
    k[r] = keys[i < n ? i : n - 1];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kItems; ++r)
    if (base + int64_t(r) * kThreads + threadIdx.x < n)
      atomicAdd(&cnt[uint32_t(k[r] >> shift) & 255u], 1u);
  __syncthreads();
  hist[kOwn ? int64_t(blockIdx.x) * 256 + threadIdx.x
            : int64_t(threadIdx.x) * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

// Inclusive prefix of one value per thread across the block's four waves.
__device__ inline uint32_t block_iscan(uint32_t v, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += wsum[w];
  return v;
}

// Stable scatter of one 8-bit digit.  Each block ranks its tile in LDS, then
// writes it out digit by digit, so that equal digits of a tile land in
// consecutive addresses (whole cache lines) instead of one scattered element
// per lane.  Each wave ranks its own contiguous quarter of the tile in index
// order, 64 elements a round: an element's rank among equal digits is the
// wave's running count of its digit plus its equal digits in lower lanes
// (found with eight ballots); one prefix over the waves per digit then
// places the quarters after each other.  hist holds the digit counts of every
// tile, tile-major (kOwn: the lanes of a block read a tile's row together), or
// their exclusive prefix, digit-major, of which a block's count of digit d is
// the difference of its entry and the next one (n after the last).
template <int kItems, bool kOwn>
__global__ __launch_bounds__(kThreads) void k_rs_scatter(const uint64_t* kin,
                                                         const uint32_t* vin, uint64_t* kout,
                                                         uint32_t* vout, int64_t n, int shift,
                                                         const uint32_t* hist,
                                                         int64_t nblocks) {
  constexpr int kTile = kThreads * kItems;
  constexpr int kPerWave = kTile / kWaves;
  constexpr int kRounds = kPerWave / 64;
  __shared__ uint64_t lkey[kTile];
  __shared__ uint32_t lval[kTile];
  __shared__ uint32_t gbase[256];   // global start of this block's digit d
  __shared__ uint32_t lbase[256];   // local start of digit d in the tile
  __shared__ uint32_t wcnt[kWaves][256];
  __shared__ uint32_t wsum[kWaves], wsum2[kWaves];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t blk = int64_t(blockIdx.x) * kTile;
  const int64_t wbase = blk + int64_t(wave) * kPerWave;
  // the wave's quarter into registers first, so that ranking does not wait
  uint64_t kr[kRounds];
  uint32_t vr[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = wbase + r * 64 + lane;
    kr[r] = i < n ? kin[i] : 0ull;
    vr[r] = i < n ? vin[i] : 0u;
  }
  uint32_t g0, cnt;
  if constexpr (kOwn) {
    // this lane's digit: its count in all tiles, in the tiles before, in ours;
    // sixteen loads in flight
    const int nt = int(nblocks), me = int(blockIdx.x);
    uint32_t all = 0, before = 0;
    for (int b = 0; b < nt; b += 16) {
      uint32_t c[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) c[u] = hist[min(b + u, nt - 1) * 256 + t];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const uint32_t x = b + u < nt ? c[u] : 0u;
        all += x;
        before += b + u < me ? x : 0u;
      }
    }
    cnt = hist[me * 256 + t];
    g0 = block_iscan(all, wsum2) - all + before;
  } else {
    const int64_t hi = int64_t(t) * nblocks + blockIdx.x;
    g0 = hist[hi];
    cnt = (hi + 1 < 256 * nblocks ? hist[hi + 1] : uint32_t(n)) - g0;
  }
  gbase[t] = g0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) wcnt[w][t] = 0;
  // exclusive prefix of the 256 counts
  lbase[t] = block_iscan(cnt, wsum) - cnt;
  // rank inside the wave's quarter (the wave's LDS operations stay in order,
  // so a group's leader updates the count after every lane of it has read it)
  const uint64_t lower = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t pos[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool ok = wbase + r * 64 + lane < n;
    const uint32_t d = uint32_t(kr[r] >> shift) & 255u;
    uint64_t m = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      m &= bit ? bal : ~bal;
    }
    const uint32_t rank = __popcll(m & lower);
    const uint32_t prev = wcnt[wave][d];
    pos[r] = prev + rank;
    if (ok && rank == 0) wcnt[wave][d] = prev + __popcll(m);
  }
  __syncthreads();
  // per digit, the waves' quarters one after the other from the digit's start
  uint32_t run = lbase[t];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t c = wcnt[w][t];
    wcnt[w][t] = run;
    run += c;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    if (wbase + r * 64 + lane < n) {
      const uint32_t off = wcnt[wave][uint32_t(kr[r] >> shift) & 255u] + pos[r];
      lkey[off] = kr[r];
      lval[off] = vr[r];
    }
  __syncthreads();
  // write out in local order: consecutive positions of one digit go to
  // consecutive global addresses
  const int tile = int(min(int64_t(kTile), n - blk));
  for (int p = t; p < tile; p += kThreads) {
    const uint64_t k = lkey[p];
    const uint32_t d = uint32_t(k >> shift) & 255u;
    const uint32_t off = gbase[d] + uint32_t(p) - lbase[d];
    kout[off] = k;
    vout[off] = lval[p];
  }
}

// The whole sort of up to 1024 * kItems pairs by one block, every pass through
// LDS: a few thousand pairs in two launches a pass leave most of the chip idle and cost
// the host and the device about 40 us for five passes at 5000 pairs; one block takes
// 28 us in one launch (at 13k pairs 57 against 31 us: above 8192 the passes).  Each of the sixteen waves ranks its own contiguous part of the tile
// as k_rs_scatter's four do; keys, then values, change places through one
// buffer (8 bytes a pair: 64 KB at kItems = 8, next to 17 KB of counts).
template <int kItems>
__global__ __launch_bounds__(1024) void k_rs_block(uint64_t* keys, uint32_t* vals, int32_t n,
                                                   int32_t passes) {
  constexpr int kW = 16;
  constexpr int kPart = 64 * kItems;   // elements of a wave
  __shared__ uint64_t buf[1024 * kItems];
  __shared__ uint32_t wcnt[kW][256];
  __shared__ uint32_t wsum[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int base = wave * kPart + lane;
  uint64_t kr[kItems];
  uint32_t vr[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int i = base + r * 64;
    kr[r] = i < n ? keys[i] : 0ull;
    vr[r] = i < n ? vals[i] : 0u;
  }
  const uint64_t lower = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
#pragma unroll
    for (int q = 0; q < 4; ++q) wcnt[4 * q + (t >> 8)][t & 255] = 0;
    __syncthreads();
    uint32_t pos[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const bool ok = base + r * 64 < n;
      const uint32_t d = uint32_t(kr[r] >> shift) & 255u;
      uint64_t m = __ballot(ok);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bal = __ballot(bit);
        m &= bit ? bal : ~bal;
      }
      const uint32_t rank = __popcll(m & lower);
      const uint32_t prev = wcnt[wave][d];
      pos[r] = prev + rank;
      if (ok && rank == 0) wcnt[wave][d] = prev + __popcll(m);
    }
    __syncthreads();
    // per digit: the waves' counts to offsets inside the digit, the digit's
    // start from a prefix over the 256 totals (the first four waves)
    uint32_t run = 0, incl = 0;
    if (t < 256) {
#pragma unroll
      for (int w = 0; w < kW; ++w) {
        const uint32_t c = wcnt[w][t];
        wcnt[w][t] = run;
        run += c;
      }
      incl = run;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (lane == 63) wsum[wave] = incl;
    }
    __syncthreads();
    if (t < 256) {
      uint32_t start = incl - run;
      for (int w = 0; w < wave; ++w) start += wsum[w];
#pragma unroll
      for (int w = 0; w < kW; ++w) wcnt[w][t] += start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
      if (base + r * 64 < n) {
        pos[r] += wcnt[wave][uint32_t(kr[r] >> shift) & 255u];
        buf[pos[r]] = kr[r];
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
      if (base + r * 64 < n) kr[r] = buf[base + r * 64];
    __syncthreads();
    uint32_t* vbuf = reinterpret_cast<uint32_t*>(buf);
#pragma unroll
    for (int r = 0; r < kItems; ++r)
      if (base + r * 64 < n) vbuf[pos[r]] = vr[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
      if (base + r * 64 < n) vr[r] = vbuf[base + r * 64];
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int i = base + r * 64;
    if (i < n) {
      keys[i] = kr[r];
      vals[i] = vr[r];
    }
  }
}

template <int kItems>
far_status_t rs_passes(uint64_t*& ka, uint32_t*& va, uint64_t*& kb, uint32_t*& vb, int64_t n,
                       int passes, hipStream_t st, Scratch& scr) {
  const int64_t nblocks = (n + kThreads * kItems - 1) / (kThreads * kItems);
  const bool own = nblocks <= kOwnTiles;
  const unsigned grid = unsigned(nblocks);
  uint32_t* hist = nullptr;
  FAR_TRY(scr.get(&hist, size_t(256 * nblocks)));
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    if (own) {
      k_rs_hist<kItems, true><<<grid, kThreads, 0, st>>>(ka, n, shift, hist, nblocks);
      FAR_HIP(hipGetLastError());
      k_rs_scatter<kItems, true><<<grid, kThreads, 0, st>>>(ka, va, kb, vb, n, shift, hist,
                                                            nblocks);
    } else {
      k_rs_hist<kItems, false><<<grid, kThreads, 0, st>>>(ka, n, shift, hist, nblocks);
      FAR_HIP(hipGetLastError());
      FAR_TRY(scan_exclusive(hist, hist, 256 * nblocks, nullptr, st, scr));
      k_rs_scatter<kItems, false><<<grid, kThreads, 0, st>>>(ka, va, kb, vb, n, shift, hist,
                                                             nblocks);
    }
    FAR_HIP(hipGetLastError());
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  return FAR_OK;
}

}  // namespace

far_status_t scan_exclusive(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total,
                            hipStream_t st, Scratch& scr) {
  if (n <= 0) {
    if (total) FAR_HIP(hipMemsetAsync(total, 0, sizeof(uint32_t), st));
    return FAR_OK;
  }
  int64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles == 1) {
    k_scan_tiles<<<1, kThreads, 0, st>>>(in, out, n, nullptr, total);
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  }
  uint32_t* sums = nullptr;
  FAR_TRY(scr.get(&sums, size_t(tiles)));
  k_scan_tile_sums<<<dim3(uint32_t(tiles)), kThreads, 0, st>>>(in, n, sums);
  FAR_HIP(hipGetLastError());
  FAR_TRY(scan_exclusive(sums, sums, tiles, nullptr, st, scr));
  k_scan_tiles<<<dim3(uint32_t(tiles)), kThreads, 0, st>>>(in, out, n, sums, total);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

far_status_t radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt,
                              uint32_t* vals_alt, int64_t n, int bits, hipStream_t st,
                              Scratch& scr, bool* in_alt) {
  if (in_alt) *in_alt = false;
  if (n <= 1 || bits <= 0) return FAR_OK;
  uint64_t *ka = keys, *kb = keys_alt;
  uint32_t *va = vals, *vb = vals_alt;
  const int passes = (bits + 7) / 8;
  if (n <= 8 * 1024) {       // one block, in place
    if (n <= 4 * 1024)
      k_rs_block<4><<<1, 1024, 0, st>>>(ka, va, int32_t(n), passes);
    else
      k_rs_block<8><<<1, 1024, 0, st>>>(ka, va, int32_t(n), passes);
    FAR_HIP(hipGetLastError());
  } else if (n <= 64 * 1024)        // at most 64 tiles of 1024
    FAR_TRY(rs_passes<4>(ka, va, kb, vb, n, passes, st, scr));
  else if (n <= 256 * 1024)  // at most 128 tiles of 2048
    FAR_TRY(rs_passes<8>(ka, va, kb, vb, n, passes, st, scr));
  else                       // tiles of 4096, scanned tables beyond 512k
    FAR_TRY(rs_passes<16>(ka, va, kb, vb, n, passes, st, scr));
  if (in_alt) {
    *in_alt = ka != keys;
    return FAR_OK;
  }
  if (ka != keys) {
    FAR_HIP(hipMemcpyAsync(keys, ka, size_t(n) * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    FAR_HIP(hipMemcpyAsync(vals, va, size_t(n) * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
  }
  return FAR_OK;
}

// ---------------------------------------------------------------- scratch pool
// A call's temporary buffers are allocated and freed on its stream.  The
// device's default pool hands freed memory back to the driver at every
// synchronisation (release threshold 0), so each call would map its scratch
// afresh, which costs more than many of the kernels it serves.  The library's
// own pool keeps what it has reserved (threshold unlimited) until
// far_scratch_release or a request that the device cannot hold.  Its footprint is
// what was out at once at most: for calls one after the other on one stream the
// largest scratch of any of them, else at most the kept chunks (kScratchKept) and
// those of the calls in flight, each no larger than the largest.
namespace {
struct Kept {
  void* p;
  size_t bytes;
  hipStream_t stream;
  hipEvent_t ev;   // behind its last work; null: the null stream's (see Idle)
};
struct Pools {
  std::mutex mu;
  std::vector<hipMemPool_t> pool;          // per device id, null until first use
  std::vector<std::vector<Kept>> kept;     // per device id
  std::vector<std::vector<hipEvent_t>> events;   // per device id, not in use
};
Pools& pools() {
  static Pools p;
  return p;
}
}  // namespace

// While it lives, this thread's calls are checked neither against nor by a capture
// on any thread's stream (a query or a wait in the default mode would end such a
// capture).
namespace {
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool swapped;
  RelaxedCapture() { swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess; }
  ~RelaxedCapture() {
    if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
  RelaxedCapture(const RelaxedCapture&) = delete;
  RelaxedCapture& operator=(const RelaxedCapture&) = delete;
};
}  // namespace

// Whether the work of a kept chunk has ended: the null stream's when that stream
// is idle.  (The first query after a kernel only asks the device for a mark, so
// the null stream is asked for 30 us, about what a pool request costs; at most
// once per object.)
class Idle {
  int null_ = -1;
  static bool ended(hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();   // hipErrorNotReady
    return e == hipSuccess;
  }

 public:
  bool operator()(const Kept& k) {
    RelaxedCapture relaxed;
    if (k.ev) return ended(hipEventQuery(k.ev));
    const auto t0 = std::chrono::steady_clock::now();
    while (null_ < 0) {
      if (ended(hipStreamQuery(nullptr)))
        null_ = 1;
      else if (std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(30))
        null_ = 0;
    }
    return null_ == 1;
  }
};

// The idle kept chunks of the current device dev back to its pool, on a stream made
// for it: work on the null stream waits for other streams, and a free on it crashed
// the runtime while another thread captured a stream that the null stream waits
// for.  Only the frees are waited for.  (With the pools locked.)
static void free_idle(int dev) {
  RelaxedCapture relaxed;
  Pools& P = pools();
  auto& kept = P.kept[dev];
  hipStream_t st = nullptr;
  if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess) {
    // (a call still running, or a free that fails: its chunk stays)
    Idle idle;
    auto gone = [&](const Kept& k) {
      if (!idle(k) || hipFreeAsync(k.p, st) != hipSuccess) return false;
      if (k.ev) (void)hipEventDestroy(k.ev);
      return true;
    };
    kept.erase(std::remove_if(kept.begin(), kept.end(), gone), kept.end());
    (void)hipStreamSynchronize(st);
    (void)hipStreamDestroy(st);
  }
  for (hipEvent_t e : P.events[dev]) (void)hipEventDestroy(e);
  P.events[dev].clear();
  (void)hipGetLastError();
}

static bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  return stream && (hipStreamIsCapturing(stream, &cs) != hipSuccess ||
                    cs != hipStreamCaptureStatusNone);
}

void scratch_return(hipStream_t stream, size_t bytes, void* p) {
  RelaxedCapture relaxed;
  int dev = 0;
  if (!capturing(stream) && hipGetDevice(&dev) == hipSuccess) {
    Pools& P = pools();
    std::lock_guard<std::mutex> lk(P.mu);
    if (size_t(dev) < P.kept.size() && P.kept[dev].size() == kScratchKept) {
      // the longest kept of the idle chunks makes room
      auto& kept = P.kept[dev];
      Idle idle;
      const auto old = std::find_if(kept.begin(), kept.end(), [&](const Kept& k) { return idle(k); });
      if (old != kept.end() && hipFreeAsync(old->p, stream) == hipSuccess) {
        if (old->ev) P.events[dev].push_back(old->ev);
        kept.erase(old);
      }
    }
    if (size_t(dev) < P.kept.size() && P.kept[dev].size() < kScratchKept) {
      Kept k{p, bytes, stream, nullptr};
      if (stream) {
        auto& ev = P.events[dev];
        if (!ev.empty()) {
          k.ev = ev.back();
          ev.pop_back();
        } else if (hipEventCreateWithFlags(&k.ev, hipEventDisableTiming) != hipSuccess) {
          k.ev = nullptr;
        }
        if (k.ev && hipEventRecord(k.ev, stream) != hipSuccess) {
          ev.push_back(k.ev);
          k.ev = nullptr;
        }
      }
      if (!stream || k.ev) {
        P.kept[dev].push_back(k);
        return;
      }
      (void)hipGetLastError();
    }
  }
  (void)hipFreeAsync(p, stream);
}

far_status_t scratch_take(hipStream_t stream, size_t bytes, size_t* got, void** out) {
  *out = nullptr;
  *got = bytes;
  int dev = 0;
  FAR_HIP(hipGetDevice(&dev));
  const bool cap = capturing(stream);
  Pools& P = pools();
  std::unique_lock<std::mutex> lk(P.mu);
  if (size_t(dev) >= P.pool.size()) {
    P.pool.resize(size_t(dev) + 1, nullptr);
    P.kept.resize(size_t(dev) + 1);
    P.events.resize(size_t(dev) + 1);
  }
  if (!cap) {
    // the smallest chunk of this stream that holds the request, then the
    // smallest idle one of up to four times the request (a small call on one
    // stream would take the large chunk that another stream's next call needs, and
    // that call would ask the pool for another); without either the largest
    // smaller idle one goes back
    auto& kept = P.kept[dev];
    Idle idle;
    int best = -1, drop = -1;
    auto own = [&](const Kept& k) { return k.stream == stream; };
    for (int i = 0; i < int(kept.size()); ++i)
      if (own(kept[i]) && kept[i].bytes >= bytes &&
          (best < 0 || kept[i].bytes < kept[best].bytes))
        best = i;
    if (best < 0)
      for (int i = 0; i < int(kept.size()); ++i)
        if (!own(kept[i]) && kept[i].bytes >= bytes && kept[i].bytes / 4 <= bytes &&
            (best < 0 || kept[i].bytes < kept[best].bytes) && idle(kept[i]))
          best = i;
    if (best < 0)
      for (int i = 0; i < int(kept.size()); ++i)
        if (kept[i].bytes < bytes && (drop < 0 || kept[i].bytes > kept[drop].bytes) &&
            (own(kept[i]) || idle(kept[i])))
          drop = i;
    const int at = best >= 0 ? best : drop;
    if (at >= 0) {
      const Kept k = kept[at];
      kept.erase(kept.begin() + at);
      if (k.ev) {
        // (also where the handles are equal: the stream may be a new one)
        const hipError_t e = hipStreamWaitEvent(stream, k.ev, 0);
        P.events[dev].push_back(k.ev);
        if (e != hipSuccess) {
          (void)hipEventSynchronize(k.ev);
          (void)hipGetLastError();
        }
      }
      if (best >= 0) {
        *out = k.p;
        *got = k.bytes;
        return FAR_OK;
      }
      (void)hipFreeAsync(k.p, stream);
    }
  }
  if (!P.pool[dev]) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t p = nullptr;
    FAR_HIP(hipMemPoolCreate(&p, &props));
    uint64_t keep = ~uint64_t(0);
    const hipError_t e = hipMemPoolSetAttribute(p, hipMemPoolAttrReleaseThreshold, &keep);
    if (e != hipSuccess) {
      (void)hipMemPoolDestroy(p);
      return hip_fail(e, "hipMemPoolSetAttribute(release threshold)", __FILE__, __LINE__);
    }
    P.pool[dev] = p;
  }
  hipMemPool_t pool = P.pool[dev];
  lk.unlock();
  hipError_t e = hipMallocFromPoolAsync(out, bytes, pool, stream);
  if (e != hipSuccess && !cap) {
    // the kept chunks that are idle, and what else the pool holds unused, back to
    // the driver first
    (void)hipGetLastError();
    lk.lock();
    free_idle(dev);
    lk.unlock();
    (void)hipMemPoolTrimTo(pool, 0);
    e = hipMallocFromPoolAsync(out, bytes, pool, stream);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();   // (not for the next call to find)
    *out = nullptr;
    return hip_fail(e, "hipMallocFromPoolAsync", __FILE__, __LINE__);
  }
  return FAR_OK;
}

// ---------------------------------------------------------------- host slots
namespace {
struct HostSlots {
  std::mutex mu;
  char* host = nullptr;
  char* dev = nullptr;
  uint64_t used = 0;   // bit per slot
  std::atomic<uint32_t> ticket{0};
};
HostSlots& host_slots() {
  static HostSlots h;
  return h;
}

// Words of a, then b, into the slot, then the ticket: a system-scope release
// behind a barrier, so that the host that sees the ticket sees the words.
__global__ __launch_bounds__(256) void k_publish(const uint32_t* a, int32_t na, const uint32_t* b,
                                                 int32_t nb, uint32_t* slot, uint32_t ticket) {
  for (int32_t i = threadIdx.x; i < na + nb; i += blockDim.x)
    slot[16 + i] = i < na ? a[i] : b[i - na];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(slot, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace

void HostSlot::take(hipStream_t st) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();   // (the legacy stream while another stream captures)
    return;
  }
  HostSlots& h = host_slots();
  std::lock_guard<std::mutex> lk(h.mu);
  if (!h.host) {
    void *p = nullptr, *d = nullptr;
    if (hipHostMalloc(&p, kHostSlots * kSlotBytes, hipHostMallocPortable | hipHostMallocMapped) !=
        hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    if (hipHostGetDevicePointer(&d, p, 0) != hipSuccess) {
      (void)hipGetLastError();
      (void)hipHostFree(p);
      return;
    }
    memset(p, 0, kHostSlots * kSlotBytes);
    h.host = static_cast<char*>(p);
    h.dev = static_cast<char*>(d);
  }
  if (~h.used == 0) return;
  const int i = __builtin_ctzll(~h.used);
  h.used |= uint64_t(1) << i;
  host = reinterpret_cast<uint32_t*>(h.host + size_t(i) * kSlotBytes);
  dev = reinterpret_cast<uint32_t*>(h.dev + size_t(i) * kSlotBytes);
  *host = 0u;   // no ticket, no progress (no kernel writes a free slot)
  do {
    ticket = ++h.ticket;
  } while (ticket == 0);
}

HostSlot::~HostSlot() {
  if (!host) return;
  if (busy) (void)hipStreamSynchronize(pending);   // nothing writes a slot given back
  HostSlots& h = host_slots();
  std::lock_guard<std::mutex> lk(h.mu);
  const size_t i = size_t(reinterpret_cast<char*>(host) - h.host) / kSlotBytes;
  h.used &= ~(uint64_t(1) << i);
}

far_status_t fetch(hipStream_t st, void* a_host, const void* a, size_t a_bytes, void* b_host,
                   const void* b, size_t b_bytes) {
  HostSlot slot;
  if (a_bytes + b_bytes <= kSlotData) slot.take(st);
  if (!slot.host) {
    FAR_HIP(hipMemcpyAsync(a_host, a, a_bytes, hipMemcpyDeviceToHost, st));
    if (b) FAR_HIP(hipMemcpyAsync(b_host, b, b_bytes, hipMemcpyDeviceToHost, st));
    FAR_HIP(hipStreamSynchronize(st));
    return FAR_OK;
  }
  slot.pending = st;
  slot.busy = true;
  k_publish<<<1, 256, 0, st>>>(static_cast<const uint32_t*>(a), int32_t(a_bytes / 4),
                               static_cast<const uint32_t*>(b), int32_t(b_bytes / 4), slot.dev,
                               slot.ticket);
  FAR_HIP(hipGetLastError());
  // watch for two milliseconds, then let the runtime wait (and report faults)
  const auto t0 = std::chrono::steady_clock::now();
  bool seen = false;
  for (int spin = 0; !seen; ++spin) {
    seen = __atomic_load_n(slot.host, __ATOMIC_ACQUIRE) == slot.ticket;
    if (!seen && (spin & 255) == 255 &&
        std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(2))
      break;
  }
  if (!seen) {
    FAR_HIP(hipStreamSynchronize(st));
    if (__atomic_load_n(slot.host, __ATOMIC_ACQUIRE) != slot.ticket) {
      set_error("internal: a result did not reach its host slot");
      return FAR_E_HIP;
    }
  }
  slot.busy = false;
  const char* w = reinterpret_cast<const char*>(slot.host) + 64;
  memcpy(a_host, w, a_bytes);
  if (b) memcpy(b_host, w + a_bytes, b_bytes);
  return FAR_OK;
}

// ---------------------------------------------------------------- timing
namespace {
struct Timing {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending[FAR_TIME_KINDS];
  double ms[FAR_TIME_KINDS] = {};
  int64_t count[FAR_TIME_KINDS] = {};
};
Timing& timing() {
  static Timing t;
  return t;
}
}  // namespace

bool timing_on() {
  std::lock_guard<std::mutex> lk(timing().mu);
  return timing().on;
}

void timing_push(int kind, hipEvent_t ev0, hipEvent_t ev1) {
  std::lock_guard<std::mutex> lk(timing().mu);
  timing().pending[kind].push_back({ev0, ev1});
}

}  // namespace far

extern "C" {

far_status_t far_scratch_release(void) {
  far::Pools& P = far::pools();
  std::lock_guard<std::mutex> lk(P.mu);
  far::RelaxedCapture relaxed;
  int here = 0;
  FAR_HIP(hipGetDevice(&here));
  for (size_t d = 0; d < P.kept.size(); ++d) {
    if (P.kept[d].empty() && P.events[d].empty()) continue;
    FAR_HIP(hipSetDevice(int(d)));
    far::free_idle(int(d));
    FAR_HIP(hipSetDevice(here));
  }
  for (hipMemPool_t p : P.pool)
    if (p) FAR_HIP(hipMemPoolTrimTo(p, 0));
  return FAR_OK;
}

far_status_t far_scratch_reserved(int64_t* bytes) {
  if (!bytes) {
    far::set_error("far_scratch_reserved: invalid argument");
    return FAR_E_INVALID;
  }
  *bytes = 0;
  int dev = 0;
  FAR_HIP(hipGetDevice(&dev));
  far::Pools& P = far::pools();
  std::lock_guard<std::mutex> lk(P.mu);
  if (size_t(dev) >= P.pool.size() || !P.pool[dev]) return FAR_OK;
  uint64_t v = 0;
  FAR_HIP(hipMemPoolGetAttribute(P.pool[dev], hipMemPoolAttrReservedMemCurrent, &v));
  *bytes = int64_t(v);
  return FAR_OK;
}

far_status_t far_timing_enable(int32_t on) {
  std::lock_guard<std::mutex> lk(far::timing().mu);
  far::timing().on = on != 0;
  return FAR_OK;
}

far_status_t far_timing_read_kind(int32_t kind, double* ms, int64_t* count, int32_t reset) {
  if (kind < 0 || kind >= FAR_TIME_KINDS) {
    far::set_error("far_timing_read_kind: kind %d out of range", kind);
    return FAR_E_INVALID;
  }
  std::lock_guard<std::mutex> lk(far::timing().mu);
  far::Timing& t = far::timing();
  for (auto& pr : t.pending[kind]) {
    FAR_HIP(hipEventSynchronize(pr.second));
    float e = 0.0f;
    FAR_HIP(hipEventElapsedTime(&e, pr.first, pr.second));
    t.ms[kind] += e;
    t.count[kind] += 1;
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  t.pending[kind].clear();
  if (ms) *ms = t.ms[kind];
  if (count) *count = t.count[kind];
  if (reset) {
    t.ms[kind] = 0.0;
    t.count[kind] = 0;
  }
  return FAR_OK;
}

far_status_t far_timing_read(double* linearize_ms, int64_t* launches, int32_t reset) {
  return far_timing_read_kind(FAR_TIME_LINEARIZE, linearize_ms, launches, reset);
}

}  // extern "C"
