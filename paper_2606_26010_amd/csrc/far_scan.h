// far_scan.h -- prefix sums of 0/1 flags in two launches, with the flag and the
// use of the prefix given as functors, so that the passes around a compaction
// (computing the flags, writing the kept items) need no launches of their own.
#pragma once

#include "far_internal.h"

namespace far {

// Sum of v over the block's 256 threads, in every thread.
__device__ inline uint32_t block_total(uint32_t v) {
  __shared__ uint32_t part[4];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += uint32_t(__shfl_xor(int(v), d));
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  v = (part[0] + part[1]) + (part[2] + part[3]);
  __syncthreads();
  return v;
}

// A tile is 256 threads times kRounds items each: one up to 256k items, so that
// small jobs spread over the chip (a lookup per item in eight rounds took 19 us
// for 13k items on 7 blocks, 5.3 us on 52), eight beyond.
constexpr int kFlagThreads = 256;
constexpr int64_t kFlagSmall = 256 * 1024;
// Up to this many tiles every block of the second launch adds the tile sums
// before its own itself (at most 16 loads per lane); beyond, they are scanned
// by launches of their own.
constexpr int64_t kFlagOwnCarry = 4096;

// Launch 1: the flags of each tile counted.  F: bool flag(i), which may also
// store what the second launch's flag reads back.
template <int kRounds, class F>
__global__ __launch_bounds__(kFlagThreads) void k_flag_sums(F f, int64_t n, uint32_t* sums) {
  const int64_t base = int64_t(blockIdx.x) * (kFlagThreads * kRounds) + threadIdx.x;
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kFlagThreads;
    if (i < n && f.first(i)) ++c;
  }
  c = block_total(c);
  if (threadIdx.x == 0) sums[blockIdx.x] = c;
}

// Launch 2: f.use(i, flag, number of flags before i, number of all flags) of
// every item; *total receives the number of all.  The ranks inside a tile come
// from one ballot per wave and round.
template <int kRounds, class F>
__global__ __launch_bounds__(kFlagThreads) void k_flag_scan(F f, int64_t n, const uint32_t* sums,
                                                            int64_t tiles, const uint32_t* carry,
                                                            uint32_t* total) {
  constexpr int kCells = kRounds * kFlagThreads / 64;
  __shared__ uint32_t cell[kCells];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t base = int64_t(blockIdx.x) * (kFlagThreads * kRounds) + threadIdx.x;
  uint32_t before = 0, all = 0;
  if (carry) {
    before = carry[blockIdx.x];
    all = *total;
  } else {
    for (int64_t t = threadIdx.x; t < tiles; t += kFlagThreads) {
      const uint32_t s = sums[t];
      all += s;
      before += t < int64_t(blockIdx.x) ? s : 0u;
    }
    all = block_total(all);
    before = block_total(before);
    if (blockIdx.x == 0 && threadIdx.x == 0) *total = all;
  }
  uint64_t bal[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kFlagThreads;
    bal[r] = __ballot(i < n && f.again(i));
    if (lane == 0) cell[r * 4 + wave] = uint32_t(__popcll(bal[r]));
  }
  __syncthreads();
  const uint64_t lower = (uint64_t(1) << lane) - 1;
  uint32_t at = before;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kFlagThreads;
    uint32_t pre = at;
    for (int w = 0; w < 4; ++w) {
      const uint32_t s = cell[r * 4 + w];
      pre += w < wave ? s : 0u;
      at += s;
    }
    if (i < n) f.use(i, ((bal[r] >> lane) & 1u) != 0, pre + uint32_t(__popcll(bal[r] & lower)), all);
  }
}

// Both launches over n items; *total [dev] receives the number of flags.
// F: bool first(i) (launch 1), bool again(i) (launch 2, the same value),
// void use(i, flag, prefix, all).
template <int kRounds, class F>
far_status_t scan_flags_tiled(const F& f, int64_t n, uint32_t* total, hipStream_t st,
                              Scratch& scr) {
  constexpr int64_t kTile = int64_t(kFlagThreads) * kRounds;
  const int64_t tiles = n > 0 ? (n + kTile - 1) / kTile : 1;
  uint32_t *sums, *carry = nullptr;
  FAR_TRY(scr.get(&sums, size_t(tiles)));
  k_flag_sums<kRounds, F><<<unsigned(tiles), kFlagThreads, 0, st>>>(f, n, sums);
  FAR_HIP(hipGetLastError());
  if (tiles > kFlagOwnCarry) {
    FAR_TRY(scr.get(&carry, size_t(tiles)));
    FAR_TRY(scan_exclusive(sums, carry, tiles, total, st, scr));
  }
  k_flag_scan<kRounds, F><<<unsigned(tiles), kFlagThreads, 0, st>>>(f, n, sums, tiles, carry,
                                                                    total);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

template <class F>
far_status_t scan_flags(const F& f, int64_t n, uint32_t* total, hipStream_t st, Scratch& scr) {
  return n <= kFlagSmall ? scan_flags_tiled<1>(f, n, total, st, scr)
                         : scan_flags_tiled<8>(f, n, total, st, scr);
}

}  // namespace far
