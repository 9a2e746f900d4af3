// far_gicp.hip -- sparsity-aware GICP linearisation and the Gauss-Newton
// iteration (Sec. III-A.2, Eqs. (2)-(6)), for one scan or many scans per
// launch.
//
// Work decomposition: every scan is cut into tiles of 256 consecutive points
// (128 to 512); one block linearises one tile (one point per thread) and writes
// 29 FP64 partial sums (21 upper-triangle H entries, 6 b entries, cost,
// inlier count).  A second kernel runs one block per scan: it sums the scan's
// tile partials in tile order (deterministic) and one lane solves the 6x6
// system in FP64 and updates the pose.  Finished scans skip their tiles.
// The first iteration is therefore two launches whatever the number of scans
// and a later one four (certify, search the rest, terms, solve); a small job
// takes one launch an iteration (k_wide_iter), in the same order of sums.  On
// a stream that allows capture the whole align (state init + max_iters
// iterations) is captured into a HIP graph per repeating argument set and
// replayed; a one-scan align launched directly stops once its scan is done.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "far_knn.h"

namespace far {
namespace {

// Points per linearisation tile (= threads per block, one point per lane):
// 128, 256 or 512, chosen per map (far_map_set_schedule / far_autotune).
constexpr int kTileDefault = 256;
constexpr int kTileMin = 128;
constexpr int kTileMax = 512;
constexpr int kVals = 29;     // 21 H + 6 b + cost + count
constexpr int kStride = 32;   // partial row stride (doubles)

// How far a one-scan align has come, for the host that enqueues it: the solve
// of iteration `step` (from 1) stores it in word 0 of the slot, and kAlignDone
// once the scan is done (a captured align has none).
constexpr uint32_t kAlignDone = 0xFFFFu;
struct Progress {
  uint32_t* word;
  uint32_t step;
};

struct Params {
  double r2;        // min(tau, v)^2
  double kappa2;
  double inv_v;     // 1 / v
  int32_t v_pow2;   // v is a power of two (1/v exact)
  double eps;
  int32_t max_iters;
  int32_t recenter;
  int32_t fine_nn;  // correspondence search over the fine index (cells v/2)
  int32_t sa_off;   // drop pairs with an invalid covariance (no sparsity-aware term)
};

// ---------------------------------------------------------------- tiles
// Tile table of a job in two launches: k_tile_begin takes the per-scan tile
// counts into begin[] (one lane; S is small) and flags a malformed offsets
// array; k_tile_fill then writes one tile per lane (tile_scan -1 past the
// last tile), finding its scan by bisection of begin[] in LDS.
__global__ __launch_bounds__(64) void k_tile_begin(const int64_t* offsets, int32_t S,
                                                   int64_t n_total, int64_t max_tiles,
                                                   int32_t tile, int32_t* begin, int32_t* bad) {
  if (threadIdx.x != 0) return;
  int32_t b = (offsets[0] != 0 || offsets[S] != n_total) ? 1 : 0;
  int64_t acc = 0;
  begin[0] = 0;
  for (int32_t s = 0; s < S; ++s) {
    int64_t len = offsets[s + 1] - offsets[s];
    if (len < 0) b = 1;
    acc += len > 0 ? (len + tile - 1) / tile : 0;
    begin[s + 1] = int32_t(acc);
  }
  if (acc > max_tiles) b = 1;
  if (b)
    for (int32_t s = 0; s <= S; ++s) begin[s] = 0;
  *bad = b;
}

constexpr int kTileLdsScans = 2048;

__global__ __launch_bounds__(256) void k_tile_fill(const int64_t* offsets, int32_t S,
                                                   int64_t max_tiles, int32_t tile,
                                                   const int32_t* begin, int32_t* tile_scan,
                                                   uint32_t* tile_lo, uint32_t* tile_hi) {
  __shared__ int32_t s_begin[kTileLdsScans + 1];
  const bool lds = S <= kTileLdsScans;
  if (lds)
    for (int32_t s = threadIdx.x; s <= S; s += blockDim.x) s_begin[s] = begin[s];
  __syncthreads();
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= max_tiles) return;
  const int32_t* bg = lds ? s_begin : begin;
  if (t >= bg[S]) {
    tile_scan[t] = -1;
    return;
  }
  // the scan s with begin[s] <= t < begin[s + 1]
  int32_t lo = 0, hi = S - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (bg[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const int64_t a = offsets[lo] + (t - bg[lo]) * int64_t(tile);
  const int64_t e = offsets[lo + 1];
  tile_scan[t] = lo;
  tile_lo[t] = uint32_t(a);
  tile_hi[t] = uint32_t(a + tile < e ? a + tile : e);
}

// Offsets {0, n}, pose and fixed centre of a one-scan job, passed by value
// (no host copy to stage); n < 0: a batch, whose offsets and poses the caller
// holds on the device.
struct SingleArgs {
  int64_t n;
  double T[16];
  double c[3];
};

// Per-scan state reset: not done, zero stats, linearisation centre.
__global__ __launch_bounds__(256) void k_init(int32_t S, const double* T, const int32_t* bad,
                                              int32_t recenter, const double* c_fixed,
                                              far_align_stats_t* stats, int32_t* done,
                                              double* ctr) {
  int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  int32_t b = *bad;
  done[s] = b;
  far_align_stats_t st = {};
  st.status = b ? FAR_E_INVALID : FAR_OK;
  stats[s] = st;
  const double* Ts = T + 16 * int64_t(s);
  for (int a = 0; a < 3; ++a)
    ctr[3 * s + a] = c_fixed ? c_fixed[a] : (recenter ? Ts[4 * a + 3] : 0.0);
}

// The whole job setup in one launch for up to kTileLdsScans scans: every block
// takes the per-scan tile counts into a prefix in LDS itself (S values), then
// fills its tiles, and the first blocks the per-scan state; block 0 writes the
// prefix, the flag of malformed offsets and a one-scan job's inputs.  (As
// k_tile_begin, k_tile_fill, k_init and a launch for the inputs: 18 us for one
// scan, 22 us for 64, whose prefix one lane took in turn; 4.7 us.)
__global__ __launch_bounds__(256) void k_setup(SingleArgs one, int64_t* offsets, double* T,
                                               double* cfix, int32_t S, int64_t n_total,
                                               int64_t max_tiles, int32_t tile, int32_t* begin,
                                               int32_t* bad, int32_t* tile_scan,
                                               uint32_t* tile_lo, uint32_t* tile_hi,
                                               int32_t recenter, const double* c_fixed,
                                               far_align_stats_t* stats, int32_t* done,
                                               double* ctr, uint32_t* counter) {
  __shared__ int32_t s_begin[kTileLdsScans + 1];
  __shared__ int64_t wsum[4];
  __shared__ int32_t s_bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool single = one.n >= 0;
  auto off = [&](int32_t s) { return single ? (s == 0 ? int64_t(0) : one.n) : offsets[s]; };
  if (tid == 0) {
    s_bad = off(0) != 0 || off(S) != n_total ? 1 : 0;
    s_begin[0] = 0;
  }
  __syncthreads();
  int64_t carry = 0;
  for (int32_t s0 = 0; s0 < S; s0 += 256) {
    const int32_t s = s0 + tid;
    const int64_t len = s < S ? off(s + 1) - off(s) : 0;
    if (len < 0) s_bad = 1;
    int64_t x = len > 0 ? (len + tile - 1) / tile : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t u = __shfl_up((long long)x, d);
      if (lane >= d) x += u;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int64_t total = 0;
    for (int w = 0; w < 4; ++w) {
      x += w < wave ? wsum[w] : 0;
      total += wsum[w];
    }
    if (s < S) s_begin[s + 1] = int32_t(carry + x);
    carry += total;
    __syncthreads();
  }
  if (tid == 0 && carry > max_tiles) s_bad = 1;
  __syncthreads();
  const int32_t b = s_bad;
  const int32_t n_tiles = b ? 0 : s_begin[S];
  if (blockIdx.x == 0) {
    for (int32_t s = tid; s <= S; s += 256) begin[s] = b ? 0 : s_begin[s];
    if (tid == 0) *bad = b;
    if (single) {
      if (tid < 16) T[tid] = one.T[tid];
      if (tid < 3 && cfix) cfix[tid] = one.c[tid];
      if (tid < 2) offsets[tid] = tid == 0 ? 0 : one.n;
    }
  }
  const int64_t t = int64_t(blockIdx.x) * 256 + tid;
  if (t < S) {
    // (a scan without points has no tile whose block would end its align)
    const bool empty = !b && !c_fixed && s_begin[t] == s_begin[t + 1];
    done[t] = b || empty ? 1 : 0;
    counter[t] = 0u;
    far_align_stats_t st = {};
    st.status = b ? FAR_E_INVALID : (empty ? FAR_E_FEW_CORR : FAR_OK);
    stats[t] = st;
    for (int a = 0; a < 3; ++a) {
      const double ta = single ? one.T[4 * a + 3] : T[16 * t + 4 * a + 3];
      ctr[3 * t + a] = c_fixed ? (single ? one.c[a] : c_fixed[a]) : (recenter ? ta : 0.0);
    }
  }
  if (t >= max_tiles) return;
  if (t >= n_tiles) {
    tile_scan[t] = -1;
    return;
  }
  // the scan s with begin[s] <= t < begin[s + 1]
  int32_t lo = 0, hi = S - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (s_begin[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const int64_t a = off(lo) + (t - s_begin[lo]) * int64_t(tile), e = off(lo + 1);
  tile_scan[t] = lo;
  tile_lo[t] = uint32_t(a);
  tile_hi[t] = uint32_t(a + tile < e ? a + tile : e);
}

// ---------------------------------------------------------------- reduction
// Wave-wide sum of one value per lane, carried in FP64 (an FP32 per-point
// term is widened first, which is at least as accurate as a compensated FP32
// sum and takes one add per level instead of a TwoSum).
// The four in-row levels use DPP lane swaps (quad_perm [1,0,3,2] and
// [2,3,0,1], row_half_mirror, row_mirror: each pairs a lane with a partner
// holding the other half of its group), the two cross-row levels row swaps in
// registers (as shuffles through LDS the 29 sums of a wave took 8200 cycles, 5700
// now: an FP64 iteration of 20000 points 37.5 us, 35.4 now).
// Partners add the same two values, so every lane ends with the same sum.
__device__ inline double wave_sum(double v) {
  v += dpp_partner<0xB1>(v);
  v += dpp_partner<0x4E>(v);
  v += dpp_partner<0x141>(v);
  v += dpp_partner<0x140>(v);
  double a, b;
  swap_partner<false>(v, &a, &b);
  v = a + b;
  swap_partner<true>(v, &a, &b);
  return a + b;
}

// Wave sums of many FP32 values per lane through LDS (the FP32 kernels):
// each lane stores its values as one column of a [value][lane] table whose
// rows are padded to 65 words (no bank conflicts on the writes, at most two
// lanes per bank on the reads); then four lanes per value each add sixteen
// entries in lane order in FP64 and two DPP levels join the four quarters.
// About 4 instructions per value instead of the 18 of a DPP/shuffle tree.
// The order is fixed, so the sums are deterministic; a sum of 64 FP32 values
// in FP64 is exact unless their binary exponents span more than 29.
constexpr int kRedChunk = 16;   // values per pass: lanes 4v .. 4v+3 take value v
constexpr int kRedRow = 65;     // words per table row

// ---------------------------------------------------------------- locality
// Before the iterations every point is given a locality key (scan id, then
// the Morton code of its sensor-frame voxel) and the source is packed, in key
// order, into 40 bytes per point:
//   A float4 (x, y, z, original index bits)
//   B float4 (xx or -1 when the covariance is invalid, xy, xz, yy)
//   C float2 (yz, zz)
// so that a 256-point tile is a compact patch of one scan: its lanes share
// map voxels and its map neighbourhood fits in LDS.  The order only changes
// the rounding order of the sums, never which points are summed.
__device__ inline uint32_t spread10(uint32_t x) {
  x &= 0x3ffu;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

__device__ inline uint32_t quant8(float x, double v) {
  double q = floor(double(x) / v) + 128.0;
  q = q < 0.0 ? 0.0 : (q > 255.0 ? 255.0 : q);
  return uint32_t(q);
}

__global__ __launch_bounds__(256) void k_order_keys(const float* src, int64_t n,
                                                    const int64_t* offsets, int32_t S, double v,
                                                    uint64_t* keys, uint32_t* vals) {
  int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  int32_t lo = 0, hi = S;
  while (hi - lo > 1) {
    int32_t mid = (lo + hi) >> 1;
    if (offsets[mid] <= i) lo = mid; else hi = mid;
  }
  float x = src[i], y = src[n + i], z = src[2 * n + i];
  uint32_t code = (1u << 24) - 1u;
  if (isfinite(x) && isfinite(y) && isfinite(z))
    code = spread10(quant8(x, v)) | (spread10(quant8(y, v)) << 1) |
           (spread10(quant8(z, v)) << 2);
  keys[i] = (uint64_t(lo) << 24) | code;
  vals[i] = uint32_t(i);
}

// Index of this thread's item when blocks are dealt to the eight XCDs in
// contiguous ranges (a grid of 8 * ceil(blocks / 8)); -1 past the end.  The
// sort keeps each scan's points in the scan's own index range, so the
// scattered writes of a block stay in the few MB of the scans its XCD works
// through, in that XCD's L2.
__device__ inline int64_t xcd_item(int64_t n) {
  const int64_t nb = (n + 255) / 256, chunk = (nb + 7) >> 3;
  const int64_t i = (int64_t(blockIdx.x & 7) * chunk + (blockIdx.x >> 3)) * 256 + threadIdx.x;
  return ((blockIdx.x >> 3) >= chunk || i >= n) ? -1 : i;
}

// inv = perm^-1.  A caller's order is trusted to be a permutation of its
// scans' own ranges (else the results are meaningless); entries out of range
// are skipped so that nothing is written out of bounds.
__global__ __launch_bounds__(256) void k_invert(const uint32_t* perm, int64_t n,
                                                uint32_t* inv) {
  const int64_t m = xcd_item(n);
  if (m >= 0 && perm[m] < uint64_t(n)) inv[perm[m]] = uint32_t(m);
}

// Pack in key order: read the caller's SoA arrays in their own order
// (coalesced) and write each point's 40 bytes to its sorted position.
__global__ __launch_bounds__(256) void k_pack(const float* src, const float* cov6,
                                              const uint8_t* valid, int64_t n,
                                              const uint32_t* inv, float4* A, float4* B,
                                              float2* C) {
  const int64_t i = xcd_item(n);
  if (i < 0) return;
  uint32_t m = inv[i];
  if (m >= uint64_t(n)) return;   // not a permutation (a caller's order): no write
  A[m] = make_float4(src[i], src[n + i], src[2 * n + i], __int_as_float(int32_t(i)));
  bool ok = valid[i] != 0;
  B[m] = make_float4(ok ? cov6[i] : -1.0f, cov6[n + i], cov6[2 * n + i], cov6[3 * n + i]);
  C[m] = make_float2(cov6[4 * n + i], cov6[5 * n + i]);
}

// The same packing by gather, one launch instead of two: for jobs of up to
// kGatherPack points.  Gathered, a scan in its sensor's order takes 3.5, 4.1 and 8.7 us
// at 60k, 120k and 500k points (5.8, 6.7 and 11.6 in the two launches), one in random
// order 5.6, 10.2 and 60.4 (7.0, 8.9 and 20.5: scattered reads of ten words a point
// against scattered writes of three); the line lies where the worse order meets.
constexpr int64_t kGatherPack = 128 * 1024;

__global__ __launch_bounds__(256) void k_pack_gather(const float* src, const float* cov6,
                                                     const uint8_t* valid, int64_t n,
                                                     const uint32_t* perm, float4* A, float4* B,
                                                     float2* C) {
  const int64_t m = xcd_item(n);
  if (m < 0) return;
  const uint32_t i = perm[m];
  if (i >= uint64_t(n)) return;   // not a permutation (a caller's order): no write
  A[m] = make_float4(src[i], src[n + i], src[2 * n + i], __int_as_float(int32_t(i)));
  const bool ok = valid[i] != 0;
  B[m] = make_float4(ok ? cov6[i] : -1.0f, cov6[n + i], cov6[2 * n + i], cov6[3 * n + i]);
  C[m] = make_float2(cov6[4 * n + i], cov6[5 * n + i]);
}

// ---------------------------------------------------------------- GICP term
// One GICP term (Eqs. (3)-(5), sparsity-aware), accumulated into acc:
//   d = r - p, a = p - c
//   M = Sigma_r + R Sigma_s R^T if both covariances are valid, else I
//   W = M^-1, e2 = d^T W d, w = k2/(k2 + e2), rho = k2/2 ln(1 + e2/k2)
//   J = [[a]x, -I]: H += w J^T W J (21 upper entries), b += w J^T W d,
//   cost += rho, count += 1
template <class Real>
struct Core {
  Real W00, W01, W02, W11, W12, W22;   // W = M^-1 (symmetric)
  Real g0, g1, g2;                     // u = W d
  Real w, rho;
  bool both;                           // M carries both covariances
};

// The part shared by the linearisation and the gradient: M, W = M^-1,
// u = W d, e2 = d^T u, the Cauchy weight and cost.
template <class Real>
__device__ inline Core<Real> gicp_core(Real d0, Real d1, Real d2, float4 ca, float4 cb,
                                       float4 sB, float2 sC, const double* R, double kappa2) {
  Core<Real> c;
  Real M00, M01, M02, M11, M12, M22;
  c.both = sB.x >= 0.0f && cb.z != 0.0f;
  if (c.both) {
    const Real q00 = sB.x, q01 = sB.y, q02 = sB.z, q11 = sB.w, q12 = sC.x, q22 = sC.y;
    const Real r00 = Real(R[0]), r01 = Real(R[1]), r02 = Real(R[2]);
    const Real r10 = Real(R[3]), r11 = Real(R[4]), r12 = Real(R[5]);
    const Real r20 = Real(R[6]), r21 = Real(R[7]), r22 = Real(R[8]);
    // U = R Sigma_s, then M = Sigma_r + U R^T
    const Real u00 = r00 * q00 + r01 * q01 + r02 * q02;
    const Real u01 = r00 * q01 + r01 * q11 + r02 * q12;
    const Real u02 = r00 * q02 + r01 * q12 + r02 * q22;
    const Real u10 = r10 * q00 + r11 * q01 + r12 * q02;
    const Real u11 = r10 * q01 + r11 * q11 + r12 * q12;
    const Real u12 = r10 * q02 + r11 * q12 + r12 * q22;
    const Real u20 = r20 * q00 + r21 * q01 + r22 * q02;
    const Real u21 = r20 * q01 + r21 * q11 + r22 * q12;
    const Real u22 = r20 * q02 + r21 * q12 + r22 * q22;
    M00 = Real(ca.x) + (u00 * r00 + u01 * r01 + u02 * r02);
    M01 = Real(ca.y) + (u00 * r10 + u01 * r11 + u02 * r12);
    M02 = Real(ca.z) + (u00 * r20 + u01 * r21 + u02 * r22);
    M11 = Real(ca.w) + (u10 * r10 + u11 * r11 + u12 * r12);
    M12 = Real(cb.x) + (u10 * r20 + u11 * r21 + u12 * r22);
    M22 = Real(cb.y) + (u20 * r20 + u21 * r21 + u22 * r22);
  } else {
    M00 = Real(1); M01 = Real(0); M02 = Real(0);
    M11 = Real(1); M12 = Real(0); M22 = Real(1);
  }
  // W = M^-1 by the adjugate (M is symmetric positive definite)
  const Real A00 = M11 * M22 - M12 * M12;
  const Real A01 = M02 * M12 - M01 * M22;
  const Real A02 = M01 * M12 - M02 * M11;
  const Real A11 = M00 * M22 - M02 * M02;
  const Real A12 = M01 * M02 - M00 * M12;
  const Real A22 = M00 * M11 - M01 * M01;
  const Real inv_det = Real(1) / (M00 * A00 + M01 * A01 + M02 * A02);
  c.W00 = A00 * inv_det; c.W01 = A01 * inv_det; c.W02 = A02 * inv_det;
  c.W11 = A11 * inv_det; c.W12 = A12 * inv_det; c.W22 = A22 * inv_det;
  c.g0 = c.W00 * d0 + c.W01 * d1 + c.W02 * d2;
  c.g1 = c.W01 * d0 + c.W11 * d1 + c.W12 * d2;
  c.g2 = c.W02 * d0 + c.W12 * d1 + c.W22 * d2;
  const Real e2 = d0 * c.g0 + d1 * c.g1 + d2 * c.g2;
  const Real k2 = Real(kappa2);
  c.w = k2 / (k2 + e2);
  c.rho = Real(0.5) * k2 * log1p(e2 / k2);
  return c;
}

template <class Real>
__device__ inline void gicp_term(double px, double py, double pz, float4 r, float4 ca,
                                 float4 cb, float4 sB, float2 sC, const double* R, double cx,
                                 double cy, double cz, double kappa2, Real* acc) {
  const Real d0 = Real(double(r.x) - px), d1 = Real(double(r.y) - py),
             d2 = Real(double(r.z) - pz);
  const Real a0 = Real(px - cx), a1 = Real(py - cy), a2 = Real(pz - cz);
  const Core<Real> c = gicp_core<Real>(d0, d1, d2, ca, cb, sB, sC, R, kappa2);
  const Real W00 = c.W00, W01 = c.W01, W02 = c.W02, W11 = c.W11, W12 = c.W12, W22 = c.W22;
  const Real g0 = c.g0, g1 = c.g1, g2 = c.g2, w = c.w, rho = c.rho;
  // Columns of A = [a]x: A0 = (0, a2, -a1), A1 = (-a2, 0, a0), A2 = (a1, -a0, 0);
  // B = W A column by column.  H_rr[p][q] = A_p . B_q, H_rt[p][q] = -B[q][p],
  // H_tt = W; b = (A_p . g, -g).
  const Real B00 = W01 * a2 - W02 * a1, B10 = W11 * a2 - W12 * a1, B20 = W12 * a2 - W22 * a1;
  const Real B01 = W02 * a0 - W00 * a2, B11 = W12 * a0 - W01 * a2, B21 = W22 * a0 - W02 * a2;
  const Real B02 = W00 * a1 - W01 * a0, B12 = W01 * a1 - W11 * a0, B22 = W02 * a1 - W12 * a0;
  auto dotA0 = [&](Real x1, Real x2) { return a2 * x1 - a1 * x2; };
  auto dotA1 = [&](Real x0, Real x2) { return a0 * x2 - a2 * x0; };
  auto dotA2 = [&](Real x0, Real x1) { return a1 * x0 - a0 * x1; };
  int v = 0;
  acc[v++] = w * dotA0(B10, B20);
  acc[v++] = w * dotA0(B11, B21);
  acc[v++] = w * dotA0(B12, B22);
  acc[v++] = -w * B00; acc[v++] = -w * B10; acc[v++] = -w * B20;
  acc[v++] = w * dotA1(B01, B21);
  acc[v++] = w * dotA1(B02, B22);
  acc[v++] = -w * B01; acc[v++] = -w * B11; acc[v++] = -w * B21;
  acc[v++] = w * dotA2(B02, B12);
  acc[v++] = -w * B02; acc[v++] = -w * B12; acc[v++] = -w * B22;
  acc[v++] = w * W00; acc[v++] = w * W01; acc[v++] = w * W02;
  acc[v++] = w * W11; acc[v++] = w * W12;
  acc[v++] = w * W22;
  acc[v++] = w * dotA0(g1, g2);
  acc[v++] = w * dotA1(g0, g2);
  acc[v++] = w * dotA2(g0, g1);
  acc[v++] = -w * g0; acc[v++] = -w * g1; acc[v++] = -w * g2;
  acc[v++] = rho;
  acc[v++] = Real(1);
}

// One term of the gradient of the cost (correspondence and Sigma_s fixed),
// with u = W d and w the Cauchy weight (rho'(e2) = w / 2):
//   d cost / d t = -w u,   d cost / d R = -w u q^T,  q = s + Sigma_s R^T u
//   (the Sigma_s part from M = Sigma_r + R Sigma_s R^T; q = s when M = I),
//   d cost / d s = -w R^T u.
// acc: the 3x4 gradient of [R | t] row-major, then rho and a count.
template <class Real>
__device__ inline void grad_term(double px, double py, double pz, float4 s, float4 r, float4 ca,
                                 float4 cb, float4 sB, float2 sC, const double* R,
                                 double kappa2, Real* acc, Real* gs) {
  const Real d0 = Real(double(r.x) - px), d1 = Real(double(r.y) - py),
             d2 = Real(double(r.z) - pz);
  const Core<Real> c = gicp_core<Real>(d0, d1, d2, ca, cb, sB, sC, R, kappa2);
  const Real u0 = c.g0, u1 = c.g1, u2 = c.g2;
  // v = R^T u
  const Real v0 = Real(R[0]) * u0 + Real(R[3]) * u1 + Real(R[6]) * u2;
  const Real v1 = Real(R[1]) * u0 + Real(R[4]) * u1 + Real(R[7]) * u2;
  const Real v2 = Real(R[2]) * u0 + Real(R[5]) * u1 + Real(R[8]) * u2;
  Real q0 = Real(s.x), q1 = Real(s.y), q2 = Real(s.z);
  if (c.both) {
    q0 += Real(sB.x) * v0 + Real(sB.y) * v1 + Real(sB.z) * v2;
    q1 += Real(sB.y) * v0 + Real(sB.w) * v1 + Real(sC.x) * v2;
    q2 += Real(sB.z) * v0 + Real(sC.x) * v1 + Real(sC.y) * v2;
  }
  const Real nw = -c.w;
  const Real wu[3] = {nw * u0, nw * u1, nw * u2};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    acc[4 * a + 0] = wu[a] * q0;
    acc[4 * a + 1] = wu[a] * q1;
    acc[4 * a + 2] = wu[a] * q2;
    acc[4 * a + 3] = wu[a];
  }
  acc[12] = c.rho;
  acc[13] = Real(1);
  gs[0] = nw * v0;
  gs[1] = nw * v1;
  gs[2] = nw * v2;
}

// ---------------------------------------------------------------- linearise
// One block of kB threads per tile of kB locality-ordered points (one point
// per lane).  Blocks are dealt to the eight XCDs round-robin; block b
// takes tile (b mod 8) * chunk + b / 8 so that each XCD works through one
// contiguous range of tiles and neighbouring tiles - which share map voxels -
// meet in the same L2.

// Exact nearest map point within sqrt(r2) of one lane's point, ranked by
// (d2, id): the own voxel first, then every neighbour voxel whose
// conservative lower-bound distance can still beat the current best.  The
// needed neighbours are kept as a bit mask and visited in lockstep - each
// lane takes its own next needed neighbour in the same step - so a wave does
// as many voxel visits as its busiest lane needs, not one per offset that
// any lane needs (lower bounds: FaceOffsets).
//
// Exact search over the own voxel (unless own_done: its points were already
// ranked into top) and the neighbour voxels, continuing from the candidates
// already in top.
__device__ inline void nn_lockstep(const MapView& m, double px, double py, double pz,
                                   int32_t kx, int32_t ky, int32_t kz, double r2, bool own_done,
                                   int32_t own, int32_t cnt, TopK<1>& top) {
  const double v = m.v;
  FaceOffsets fo;
  fo.f[0] = float(px - double(kx) * v);
  fo.f[1] = float(py - double(ky) * v);
  fo.f[2] = float(pz - double(kz) * v);
  fo.v = float(v);
  fo.slack = float(1e-7 * v);
  Query q = make_query(px, py, pz, r2);
  q.bound_f = screen_bound(fmin(r2, top.bound()), q.m);
  if (!own_done) {
    own = map_find(m, kx, ky, kz, &cnt);
    if (own >= 0) scan_voxel_points<1>(m.vox_pts, own * m.nmax, cnt, q, r2, top);
  }
  uint32_t need = 0;
  {
    const float bnd = f32_up(fmin(r2, top.bound()));
#pragma unroll
    for (int rank = 1; rank < 27; ++rank)
      if (fo.lb2(nbr_code(rank)) <= bnd) need |= 1u << rank;
  }
  // neighbours come from the neighbour-table row of the own voxel, or of its
  // ghost when it is empty (absent ones cost nothing); an empty voxel that
  // is not a ghost has no occupied neighbour, so nothing lies within v
  const uint32_t* row = own >= 0 ? m.vox_nbr + int64_t(own) * 26 : nullptr;
  if (own < 0 && m.ghost_ok) {
    const int32_t g = ghost_find(m, kx, ky, kz);
    if (g < 0) return;
    row = m.gnbr + int64_t(g) * 26;
  }
  while (need) {
    const int rank = __builtin_ctz(need);
    need &= need - 1;
    const int code = nbr_code(rank);
    if (double(fo.lb2(code)) > fmin(r2, top.bound())) continue;
    int32_t vox;
    if (row) {
      const uint32_t e = row[nbr_dir(code)];
      if (e == kNbrNone) continue;
      vox = int32_t(e >> kNbrCountBits);
      cnt = int32_t(e & ((1u << kNbrCountBits) - 1u));
    } else {
      vox = map_find(m, kx + code / 9 - 1, ky + (code / 3) % 3 - 1, kz + code % 3 - 1, &cnt);
      if (vox < 0) continue;
    }
    scan_voxel_points<1>(m.vox_pts, vox * m.nmax, cnt, q, r2, top);
  }
}

// The exact search of the dense queue pass: as nn_lockstep from scratch, with
// the neighbour row (the own voxel's or its ghost's) copied into this lane's
// stretch of LDS by 13 independent 8-byte loads first, so that a visit waits
// for its points only, and the points loaded eight at a time.
__device__ inline void nn_search_dense(const MapView& m, double px, double py, double pz,
                                       int32_t kx, int32_t ky, int32_t kz, double r2,
                                       uint32_t* lrow, TopK<1>& top) {
  const double v = m.v;
  FaceOffsets fo;
  fo.f[0] = float(px - double(kx) * v);
  fo.f[1] = float(py - double(ky) * v);
  fo.f[2] = float(pz - double(kz) * v);
  fo.v = float(v);
  fo.slack = float(1e-7 * v);
  Query q = make_query(px, py, pz, r2);
  q.bound_f = screen_bound(fmin(r2, top.bound()), q.m);
  int32_t cnt;
  const int32_t own = map_find(m, kx, ky, kz, &cnt);
  const uint32_t* row = own >= 0 ? m.vox_nbr + int64_t(own) * 26 : nullptr;
  if (own < 0 && m.ghost_ok) {
    const int32_t g = ghost_find(m, kx, ky, kz);
    if (g < 0) return;
    row = m.gnbr + int64_t(g) * 26;
  }
  if (row) load_row(row, lrow);
  if (own >= 0) scan_voxel_points<1, 8>(m.vox_pts, own * m.nmax, cnt, q, r2, top);
  uint32_t need = 0;
  {
    const float bnd = f32_up(fmin(r2, top.bound()));
#pragma unroll
    for (int rank = 1; rank < 27; ++rank)
      if (fo.lb2(nbr_code(rank)) <= bnd) need |= 1u << rank;
  }
  while (need) {
    const int rank = __builtin_ctz(need);
    need &= need - 1;
    const int code = nbr_code(rank);
    if (double(fo.lb2(code)) > fmin(r2, top.bound())) continue;
    int32_t vox;
    if (row) {
      const uint32_t e = lrow[nbr_dir(code)];
      if (e == kNbrNone) continue;
      vox = int32_t(e >> kNbrCountBits);
      cnt = int32_t(e & ((1u << kNbrCountBits) - 1u));
    } else {
      vox = map_find(m, kx + code / 9 - 1, ky + (code / 3) % 3 - 1, kz + code % 3 - 1, &cnt);
      if (vox < 0) continue;
    }
    scan_voxel_points<1, 8>(m.vox_pts, vox * m.nmax, cnt, q, r2, top);
  }
}

// A candidate for a query: its vox_pts slot and point (x, y, z, id bits), its
// id and its exact squared distance.
struct Cand {
  double d;
  int32_t id;
  int32_t pos;
  float4 p;
};

// Walks from candidate c (its slot; its d2 is taken from its row) towards
// the query's nearest map point over the certificates' neighbour lists: c
// moves to the best listed point while one ranks before it by (d2, id), at
// most kCertWalks times.  True when c ends as a point that ranks before all
// its listed points and lies closer than its rho (its computed d2 below
// rho^2 (1 - 2^-30): the FP64 rounding of every d2 is far below that
// margin), so no map point ranks before it.  Each step reads the one
// 128-byte row of c's certificate; ids are read only to break a tie in d2.
constexpr int kCertWalks = 2;

__device__ inline bool certify(const MapView& m, const Query& q, Cand& c) {
  static_assert(sizeof(CertRow) == 128 && kCertK == 7, "a row is eight 16-byte loads");
  const float4* rows = reinterpret_cast<const float4*>(m.cert);
  for (int w = 0; w <= kCertWalks; ++w) {
    const float4* row = rows + 8 * int64_t(c.pos);
    float4 e[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) e[t] = row[t];
    if (w == 0) c.d = dist2(double(e[0].x), double(e[0].y), double(e[0].z), q.x, q.y, q.z);
    int32_t bpos = c.pos;
    double bd = c.d;
    float bnd = screen_bound(bd, q.m);
#pragma unroll
    for (int t = 1; t < 8; ++t) {
      const int32_t pos = __float_as_int(e[t].w);
      if (pos < 0) break;
      const float dx = e[t].x - q.fx, dy = e[t].y - q.fy, dz = e[t].z - q.fz;
      const float d2f = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
      if (d2f <= bnd) {
        const double d = dist2(double(e[t].x), double(e[t].y), double(e[t].z), q.x, q.y, q.z);
        // distinct points: a tie in d2 goes to the smaller id
        if (d < bd || (d == bd && __float_as_int(m.vox_pts[pos].w) <
                                      __float_as_int(m.vox_pts[bpos].w))) {
          bd = d;
          bpos = pos;
          bnd = screen_bound(d, q.m);
        }
      }
    }
    if (bpos == c.pos) {
      const double rho = double(e[0].w);
      return c.d < rho * rho * (1.0 - 0x1p-30);
    }
    c.pos = bpos;
    c.d = bd;
  }
  return false;
}

// First stage of the correspondence search (the nearest map point within
// sqrt(r2), ranked by (d2, id), as the 27-voxel search finds it).  The first
// candidate is the seed (the vox_pts slot of the point's match, or nearest
// point, of the previous iteration) or else the best point of the own voxel
// within the radius.  True when certify() proves the final candidate c the
// nearest map point: it is then the answer (none when c.d > r2).  Otherwise
// c (pos -1: none) is the best candidate seen, to bound the exact search
// that follows.
__device__ inline bool nn_cert_try(const MapView& m, double px, double py, double pz,
                                   int32_t kx, int32_t ky, int32_t kz, double r2, int32_t seed,
                                   Cand& c) {
  Query q = make_query(px, py, pz, r2);
  c.pos = -1;
  if (seed < 0) {
    int32_t cnt;
    const int32_t own = map_find(m, kx, ky, kz, &cnt);
    TopK<1> t1;
    t1.init();
    if (own >= 0) scan_voxel_points<1>(m.vox_pts, own * m.nmax, cnt, q, r2, t1);
    if (t1.pos[0] < 0) return false;
    seed = t1.pos[0];
  }
  c.pos = seed;
  return certify(m, q, c);
}

// Voxel index with an exact multiply when 1/v is exact (power-of-two v),
// else the division; both give floor(x / v) exactly as the FP64 quotient.
__device__ inline bool voxel_index_fast(double x, double v, double inv_v, bool pow2,
                                        int64_t* k) {
  const double f = floor(pow2 ? x * inv_v : x / v);
  if (!(f >= -double(kKeyBias) && f < double(kKeyBias))) return false;
  *k = int64_t(f);
  return true;
}

// Tile of this block: blocks are dealt to the eight XCDs round-robin, block b
// taking tile (b mod 8) * chunk + b / 8, so that each XCD works through one
// contiguous range of tiles and neighbouring tiles (which share map voxels)
// meet in the same L2.  -1 past the last tile.
__device__ inline int64_t block_tile(int64_t n_tiles, int64_t b = -1) {
  if (b < 0) b = blockIdx.x;
  const int64_t chunk = (n_tiles + 7) >> 3;
  const int64_t t = (b & 7) * chunk + (b >> 3);
  return (t >= n_tiles || (b >> 3) >= chunk) ? -1 : t;
}

// The tile passes run either one block per tile (gridDim = the virtual grid
// vgrid, a multiple of 8) or as a persistent grid of fewer blocks, also a
// multiple of 8, each taking virtual blocks b, b + gridDim.x, ... in turn
// (so every virtual block keeps its XCD); the loop runs once in the first
// case.

// The pose of scan s: R row-major and t.
struct Pose {
  double R[9];
  double tx, ty, tz;
  __device__ explicit Pose(const double* Ts)
      : R{Ts[0], Ts[1], Ts[2], Ts[4], Ts[5], Ts[6], Ts[8], Ts[9], Ts[10]},
        tx(Ts[3]), ty(Ts[7]), tz(Ts[11]) {}
};

// p = R s + t in FP64 (FMA-free) of packed point a, and its map voxel key;
// false when the point is not finite or its key is out of range.
__device__ inline bool locate(const float4& a, const Pose& P, const MapView& m,
                              const Params& prm, double& px, double& py, double& pz,
                              int64_t& kx, int64_t& ky, int64_t& kz) {
  // the three tests at once (a short-circuit test loads the coordinates one
  // after the other, a memory round trip each)
  if (!(isfinite(a.x) & isfinite(a.y) & isfinite(a.z))) return false;
  const double sx = a.x, sy = a.y, sz = a.z;
  px = ((P.R[0] * sx + P.R[1] * sy) + P.R[2] * sz) + P.tx;
  py = ((P.R[3] * sx + P.R[4] * sy) + P.R[5] * sz) + P.ty;
  pz = ((P.R[6] * sx + P.R[7] * sy) + P.R[8] * sz) + P.tz;
  return voxel_index_fast(px, m.v, prm.inv_v, prm.v_pow2, &kx) &&
         voxel_index_fast(py, m.v, prm.inv_v, prm.v_pow2, &ky) &&
         voxel_index_fast(pz, m.v, prm.inv_v, prm.v_pow2, &kz);
}

// A linearisation after the first iteration of an align is three passes
// over the active tiles, so that no pass holds a lane idle for another: the
// certified search (k_cert), seeded with each point's match of the previous
// iteration, settles most points and queues the rest; the exact search
// (k_search) runs the queued points densely; the term pass (k_linearize)
// forms every point's GICP term from its match and reduces them per tile.
// The first iteration, with no seeds, runs the exact search inside the term
// pass (kSearch), as a one-off linearisation and the gradient do.
//
// The queue is cut into kBins bins; tile t appends its entries to bin
// t mod kBins (one atomic per tile), so the bins fill without a global
// prefix.  An entry holds the packed point index, the best candidate of the
// first pass (a vox_pts slot, -1: none) and the FP64 map-frame position.
// The order of entries within a bin varies from run to run; every entry's
// result goes to its own point, so the results do not.
constexpr int kBins = 64;

struct Queue {
  uint32_t* idx;
  int32_t* cand;
  double* p;          // SoA, cap apart
  uint32_t* count;    // [kBins]
  int64_t bin_cap;    // entries per bin
  int64_t cap;        // kBins * bin_cap
};

// Pass 1, one block of kB lanes per tile: match[i] receives the vox_pts slot
// of point i's match when the certificates settle it (-1: none), prev[i] the
// seed of the next iteration; the other points are queued in lane order.
template <int kB, bool kLoop>
__global__ __launch_bounds__(kB) void k_cert(
    MapView m, const float4* __restrict__ pA, const int32_t* __restrict__ tile_scan,
    const uint32_t* __restrict__ tile_lo, const uint32_t* __restrict__ tile_hi,
    int64_t n_tiles, const double* __restrict__ T, const int32_t* __restrict__ done,
    Params prm, int32_t* __restrict__ match, int32_t* __restrict__ prev, Queue Q,
    int64_t vgrid) {
  constexpr int kWaves = kB / 64;
  __shared__ int32_t q_wcnt[kWaves];
  __shared__ uint32_t q_base;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // one tile (virtual block vb)
  auto tile_pass = [&](int64_t vb) {
    const int64_t t = block_tile(n_tiles, vb);
    if (t < 0) return;
    const int32_t s = tile_scan[t];
    if (s < 0 || done[s]) return;
    const Pose P(T + 16 * int64_t(s));
    const uint32_t lo = tile_lo[t], hi = tile_hi[t];
    const uint32_t i = lo + uint32_t(tid);
    bool queued = false;
    int32_t qc = -1;
    double px = 0.0, py = 0.0, pz = 0.0;
    if (i < hi) {
      // the point and its seed are loaded together, ahead of the transform
      const float4 a = pA[i];
      const int32_t seed = prev[i];
      int64_t kx = 0, ky = 0, kz = 0;   // within [-2^20, 2^20) once locate holds
      const bool have = locate(a, P, m, prm, px, py, pz, kx, ky, kz);
      Cand c;
      c.pos = -1;
      if (have && !nn_cert_try(m, px, py, pz, int32_t(kx), int32_t(ky), int32_t(kz), prm.r2,
                               seed, c)) {
        queued = true;
        qc = c.pos;
      } else {
        match[i] = have && c.d <= prm.r2 ? c.pos : -1;
        prev[i] = have ? c.pos : -1;
      }
    }
    const uint64_t bal = __ballot(queued);
    if (lane == 0) q_wcnt[wave] = __popcll(bal);
    __syncthreads();
    int off = 0, total = 0;
  #pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int cw = q_wcnt[w];
      off += w < wave ? cw : 0;
      total += cw;
    }
    if (total == 0) return;
    const int64_t bin = t % kBins;
    if (tid == 0) q_base = atomicAdd(&Q.count[bin], uint32_t(total));
    __syncthreads();
    if (queued) {
      const int64_t q = bin * Q.bin_cap + q_base + off + __popcll(bal & ((uint64_t(1) << lane) - 1));
      Q.idx[q] = i;
      Q.cand[q] = qc;
      Q.p[q] = px;
      Q.p[Q.cap + q] = py;
      Q.p[2 * Q.cap + q] = pz;
    }
    __syncthreads();   // the LDS words are rewritten for the next tile
  };
  if constexpr (kLoop) {
    for (int64_t vb = blockIdx.x; vb < vgrid; vb += gridDim.x) tile_pass(vb);
  } else {
    tile_pass(blockIdx.x);
  }
}

// Pass 2: the exact 27-voxel search of every queued point, one per lane,
// lanes striding over the bins in order (bin of entry g from an LDS prefix
// of the bin counts), so that the searches fill whole waves.  Five waves
// per SIMD (at most 96 registers, five blocks' LDS rows per CU): the
// searches wait on chains of loads, so more waves in flight hide more.
constexpr int kSearchThreads = 256;
__global__ __launch_bounds__(kSearchThreads, 5) void k_search(MapView m, Queue Q, Params prm,
                                                              int32_t* __restrict__ match,
                                                              int32_t* __restrict__ prev) {
  __shared__ uint32_t pre[kBins + 1];
  __shared__ uint32_t rows[kSearchThreads * kRowWords];
  if (threadIdx.x < 64) {
    // inclusive scan of the kBins counts across the first wave
    uint32_t v = threadIdx.x < kBins ? Q.count[threadIdx.x] : 0u;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t u = uint32_t(__shfl_up(int(v), d));
      if (int(threadIdx.x) >= d) v += u;
    }
    if (threadIdx.x < kBins) pre[threadIdx.x + 1] = v;
    if (threadIdx.x == 0) pre[0] = 0;
  }
  __syncthreads();
  const uint32_t total = pre[kBins];
  for (uint32_t g = blockIdx.x * kSearchThreads + threadIdx.x; g < total;
       g += gridDim.x * kSearchThreads) {
    int a = 0, b = kBins - 1;   // the last bin whose start is <= g
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (pre[mid] <= g) a = mid;
      else b = mid - 1;
    }
    const int64_t q = int64_t(a) * Q.bin_cap + (g - pre[a]);
    const uint32_t i = Q.idx[q];
    const double px = Q.p[q], py = Q.p[Q.cap + q], pz = Q.p[2 * Q.cap + q];
    int64_t kx = 0, ky = 0, kz = 0;
    (void)voxel_index_fast(px, m.v, prm.inv_v, prm.v_pow2, &kx);   // held in pass 1
    (void)voxel_index_fast(py, m.v, prm.inv_v, prm.v_pow2, &ky);
    (void)voxel_index_fast(pz, m.v, prm.inv_v, prm.v_pow2, &kz);
    Cand c;
    c.pos = Q.cand[q];
    if (c.pos >= 0) {
      c.p = m.vox_pts[c.pos];
      c.id = __float_as_int(c.p.w);
      c.d = dist2(double(c.p.x), double(c.p.y), double(c.p.z), px, py, pz);
    }
    TopK<1> top;
    top.init();
    if (c.pos >= 0 && c.d <= prm.r2) top.push(c.d, c.id, c.pos);
    nn_search_dense(m, px, py, pz, int32_t(kx), int32_t(ky), int32_t(kz), prm.r2,
                    rows + threadIdx.x * kRowWords, top);
    match[i] = top.pos[0];
    prev[i] = top.pos[0] >= 0 ? top.pos[0] : c.pos;
  }
}

// Pass 3, the term pass: one block of kB threads per tile, one point per
// lane, its GICP term from its match (match[i]; with kSearch from the exact
// search run here, whose result also seeds prev[i] when given), then the
// tile's sums.
// kGrad selects the gradient of the cost instead of H, b: 14 sums (the 3x4
// gradient of [R | t], cost, count) and, when grad_src is given, each
// point's source gradient written SoA at its original index (n_src apart).
// kNoSA (the sparsity-aware case off) is a template parameter: a run-time
// test in the match block costs the default path 8 %.
template <class Real, bool kGrad, int kB, bool kFine, bool kNoSA, bool kSearch, bool kLoop>
// The FP32 search variants ask for eight waves per SIMD (64 registers), the
// gradient too: its search waits on chains of loads, and 16 scans of 32768
// points took 217 us a call at the seven its 72 registers gave, 208 at eight (20
// bytes a lane spilled).
__global__ __launch_bounds__(kB, (kSearch && !kFine && !kLoop && sizeof(Real) == 4) ? 8 : 1)
void k_linearize(
    MapView m, const float4* __restrict__ pA, const float4* __restrict__ pB,
    const float2* __restrict__ pC, const int32_t* __restrict__ tile_scan,
    const uint32_t* __restrict__ tile_lo, const uint32_t* __restrict__ tile_hi,
    int64_t n_tiles, const double* __restrict__ T, const double* __restrict__ ctr,
    const int32_t* __restrict__ done, Params prm, double* __restrict__ partial,
    int32_t* __restrict__ corr, float* __restrict__ grad_src, int64_t n_src,
    const int32_t* __restrict__ match, int32_t* __restrict__ prev, int64_t vgrid) {
  constexpr int kWaves = kB / 64;
  constexpr int kNV = kGrad ? 14 : kVals;
  __shared__ double red[kWaves][kNV];
  __shared__ float tbl[std::is_same<Real, float>::value ? kWaves : 1][kRedChunk * kRedRow];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // one tile (virtual block vb)
  auto tile_pass = [&](int64_t vb) {
    const int64_t t = block_tile(n_tiles, vb);
    if (t < 0) return;
    const int32_t s = tile_scan[t];
    if (s < 0 || done[s]) return;
    const Pose P(T + 16 * int64_t(s));
    const double cx = ctr[3 * s], cy = ctr[3 * s + 1], cz = ctr[3 * s + 2];
    const uint32_t lo = tile_lo[t], hi = tile_hi[t];

    Real acc[kNV];
  #pragma unroll
    for (int q = 0; q < kNV; ++q) acc[q] = Real(0);
    const uint32_t i = lo + uint32_t(tid);
    if (i < hi) {
      const float4 a = pA[i];
      double px = 0.0, py = 0.0, pz = 0.0;
      int32_t res = -1;
      if constexpr (kSearch) {
        int64_t kx = 0, ky = 0, kz = 0;
        if (locate(a, P, m, prm, px, py, pz, kx, ky, kz)) {
          TopK<1> top;
          top.init();
          if constexpr (kFine)
            knn_cells<1>(px, py, pz, m.fc, m.inv_fc, true, true, prm.r2, m.fine_pts,
                         [&](int64_t a0, int64_t a1, int64_t a2, int32_t* n) {
                           return fine_find(m, a0, a1, a2, n);
                         },
                         top);
          else
            nn_lockstep(m, px, py, pz, int32_t(kx), int32_t(ky), int32_t(kz), prm.r2, false, -1,
                        0, top);
          res = top.pos[0];
        }
        if (!kFine && prev) prev[i] = res;
      } else {
        res = match[i];
      }
      int32_t id_match = -1;
      Real gs[3] = {Real(0), Real(0), Real(0)};
      if (res >= 0) {
        if constexpr (!kSearch) {
          int64_t kx, ky, kz;
          (void)locate(a, P, m, prm, px, py, pz, kx, ky, kz);   // held when the match was made
        }
        const float4 r = kFine ? m.fine_pts[res] : m.vox_pts[res];
        const int32_t id = __float_as_int(r.w);
        const float4 sB = pB[i];
        const float2 sC = pC[i];
        // the match's covariance record, by vox_pts slot (beside the points the
        // search read) or, for the fine index, by id
        const float4* cr = kFine ? m.cov + 2 * int64_t(id) : m.vox_cov + 2 * int64_t(res);
        const float4 ca = cr[0];
        const float4 cb = cr[1];
        // without the sparsity-aware case a pair lacking either covariance is
        // dropped like an outlier
        if (!kNoSA || (sB.x >= 0.0f && cb.z != 0.0f)) {
          id_match = id;
          if constexpr (kGrad)
            grad_term<Real>(px, py, pz, a, r, ca, cb, sB, sC, P.R, prm.kappa2, acc, gs);
          else
            gicp_term<Real>(px, py, pz, r, ca, cb, sB, sC, P.R, cx, cy, cz, prm.kappa2, acc);
        }
      }
      if (corr) corr[__float_as_uint(a.w)] = id_match;
      if (kGrad && grad_src) {
        const uint32_t o = __float_as_uint(a.w);
        grad_src[o] = float(gs[0]);
        grad_src[n_src + o] = float(gs[1]);
        grad_src[2 * n_src + o] = float(gs[2]);
      }
    }
    // wave sums in FP64, then the block's waves
    if constexpr (std::is_same<Real, float>::value) {
      float* tb = tbl[wave];
      const int v = lane >> 2, quarter = lane & 3;
  #pragma unroll
      for (int c0 = 0; c0 < kNV; c0 += kRedChunk) {
        if (c0 > 0) __syncthreads();   // the previous pass's reads are done
  #pragma unroll
        for (int q = 0; q < kRedChunk; ++q)
          if (c0 + q < kNV) tb[q * kRedRow + lane] = acc[c0 + q];
        __syncthreads();
        double sv = 0.0;
        if (c0 + v < kNV) {
          const float* row = tb + v * kRedRow + 16 * quarter;
  #pragma unroll
          for (int e = 0; e < 16; ++e) sv += double(row[e]);
        }
        sv += dpp_partner<0xB1>(sv);
        sv += dpp_partner<0x4E>(sv);
        if (quarter == 0 && c0 + v < kNV) red[wave][c0 + v] = sv;
      }
    } else {
  #pragma unroll
      for (int q = 0; q < kNV; ++q) {
        const double sv = wave_sum(acc[q]);
        if (lane == 0) red[wave][q] = sv;
      }
    }
    __syncthreads();
    if (tid < kNV) {
      double sum = 0.0;
  #pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += red[w][tid];
      partial[t * kStride + tid] = sum;
    }
    __syncthreads();   // the LDS tables are rewritten for the next tile
  };
  if constexpr (kLoop) {
    for (int64_t vb = blockIdx.x; vb < vgrid; vb += gridDim.x) tile_pass(vb);
  } else {
    tile_pass(blockIdx.x);
  }
}

// ---------------------------------------------------------------- solve
// One 256-lane block per scan (or the scan's last block of k_wide_iter): sum the
// scan's tile partials in tile order, then lane 0 solves H delta = -b by Cholesky
// (FP64) and applies T <- T_c Exp(delta) T_c^-1 T.
__device__ void se3_apply(const double* dl, const double* c, double* T) {
  const double wx = dl[0], wy = dl[1], wz = dl[2];
  const double th2 = wx * wx + wy * wy + wz * wz;
  const double th = sqrt(th2);
  double A, B, C;
  if (th < 1e-6) {
    A = 1.0 - th2 / 6.0;
    B = 0.5 - th2 / 24.0;
    C = 1.0 / 6.0 - th2 / 120.0;
  } else {
    double sn = sin(th), cs = cos(th);
    A = sn / th;
    B = (1.0 - cs) / th2;
    C = (th - sn) / (th2 * th);
  }
  // Rodrigues: R = I + A K + B K^2, V = I + B K + C K^2, K = [w]x,
  // K^2 = w w^T - th2 I.
  const double K[9] = {0.0, -wz, wy, wz, 0.0, -wx, -wy, wx, 0.0};
  const double w3[3] = {wx, wy, wz};
  double RE[9], V[9];
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q) {
      double k2 = w3[r] * w3[q] - (r == q ? th2 : 0.0);
      double id = (r == q) ? 1.0 : 0.0;
      RE[3 * r + q] = id + A * K[3 * r + q] + B * k2;
      V[3 * r + q] = id + B * K[3 * r + q] + C * k2;
    }
  double tE[3];
  for (int r = 0; r < 3; ++r) tE[r] = V[3 * r] * dl[3] + V[3 * r + 1] * dl[4] + V[3 * r + 2] * dl[5];
  // x -> c + RE (R x + t - c) + tE
  double Rn[9], tn[3];
  for (int r = 0; r < 3; ++r) {
    for (int q = 0; q < 3; ++q)
      Rn[3 * r + q] = RE[3 * r] * T[q] + RE[3 * r + 1] * T[4 + q] + RE[3 * r + 2] * T[8 + q];
    tn[r] = c[r] + tE[r] + RE[3 * r] * (T[3] - c[0]) + RE[3 * r + 1] * (T[7] - c[1]) +
            RE[3 * r + 2] * (T[11] - c[2]);
  }
  for (int r = 0; r < 3; ++r) {
    for (int q = 0; q < 3; ++q) T[4 * r + q] = Rn[3 * r + q];
    T[4 * r + 3] = tn[r];
  }
}

// A tile's partial sum of value v: as one row per tile, or (kHalf) as one row
// per wave of 64 points, two a tile, added as the block of a tile adds its
// waves.
template <bool kHalf>
__device__ inline double tile_sum(const double* partial, int64_t t, int v) {
  if constexpr (kHalf)
    return (0.0 + partial[2 * t * kStride + v]) + partial[(2 * t + 1) * kStride + v];
  else
    return partial[t * kStride + v];
}

// The sum of value v over tiles t, t + 8, ... below t1 in that order.  The
// loads go out sixteen at a time, the last ones too, at clamped tiles (a loop
// over the remainder waited for each load in turn: up to fifteen memory round
// trips, 3.4 us of k_reduce_solve's 14.1 on the 64-scan batch).
template <bool kHalf>
__device__ inline double strided_sum(const double* partial, int32_t t, int32_t t1, int v) {
  double acc = 0.0;
  for (; t < t1; t += 8 * 16) {
    double x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = tile_sum<kHalf>(partial, min(t + 8 * u, t1 - 1), v);
#pragma unroll
    for (int u = 0; u < 16; ++u) acc = t + 8 * u < t1 ? acc + x[u] : acc;
  }
  return acc;
}

// Gauss-Newton update of scan s from its 29 sums, by one lane, with its pose
// Tc, its centre cc and its iterations so far as read beforehand.  Its serial
// chain is what an iteration of a small job waits for: everything stays in
// registers, and the statistics are stored beside it by another wave
// (k_reduce_solve of 64 scans 10.7 -> 10.1 us; a factorisation without square
// roots and sine and cosine as series took 8.4, but their other roundings move
// the FP32 terms of the later iterations and scans).
__device__ void solve_scan(int32_t s, const double* lin, const double* Tc, const double* cc,
                           int32_t iters, double* T, double* ctr, int32_t* done,
                           far_align_stats_t* stats, const Params& prm, int32_t solve) {
  far_align_stats_t& st = stats[s];
  if (!solve) {
    done[s] = 1;
    return;
  }
  if (lin[28] < 6.0) {
    st.status = FAR_E_FEW_CORR;
    done[s] = 1;
    return;
  }
  // Cholesky H = L L^T in place of the lower triangle; a pivot not above 1e-12
  // max|H_ii| means not PD.
  double L[6][6], y[6];
  int u = 0;
#pragma unroll
  for (int p = 0; p < 6; ++p)
#pragma unroll
    for (int q = p; q < 6; ++q) L[q][p] = lin[u++];
  double dmax = 0.0;
#pragma unroll
  for (int p = 0; p < 6; ++p) dmax = fmax(dmax, fabs(L[p][p]));
  bool pd = true;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double sd = L[j][j];
#pragma unroll
    for (int l = 0; l < j; ++l) sd -= L[j][l] * L[j][l];
    pd = pd && sd > 1e-12 * dmax && isfinite(sd);
    const double dj = sqrt(sd);
    L[j][j] = dj;
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      double x = L[i][j];
#pragma unroll
      for (int l = 0; l < j; ++l) x -= L[i][l] * L[j][l];
      L[i][j] = x / dj;
    }
    // (the forward substitution beside the next columns)
    double x = -lin[21 + j];
#pragma unroll
    for (int l = 0; l < j; ++l) x -= L[j][l] * y[l];
    y[j] = x / dj;
  }
  if (!pd) {
    st.status = FAR_E_NOT_PD;
    done[s] = 1;
    return;
  }
  double dl[6];
#pragma unroll
  for (int i = 5; i >= 0; --i) {
    double x = y[i];
#pragma unroll
    for (int l = i + 1; l < 6; ++l) x -= L[l][i] * dl[l];
    dl[i] = x / L[i][i];
  }
  double Tn[12];
#pragma unroll
  for (int p = 0; p < 12; ++p) Tn[p] = Tc[p];
  se3_apply(dl, cc, Tn);
  double* Ts = T + 16 * int64_t(s);
#pragma unroll
  for (int p = 0; p < 12; ++p) Ts[p] = Tn[p];
  st.iters = ++iters;
  double nrm = 0.0;
#pragma unroll
  for (int p = 0; p < 6; ++p) nrm += dl[p] * dl[p];
  if (sqrt(nrm) <= prm.eps) {
    st.converged = 1;
    done[s] = 1;
  } else if (iters >= prm.max_iters) {
    done[s] = 1;
  }
  if (prm.recenter) {
    double* cs = ctr + 3 * s;
    cs[0] = Tn[3];
    cs[1] = Tn[7];
    cs[2] = Tn[11];
  }
}

// Sums of scan s's tile partials (tiles t0 to t1) and its Gauss-Newton update, by
// the first 256 threads of a block (all threads call it): eight groups of 32
// lanes, group g sums tiles t0+g, t0+g+8, ... in that order, then the eight
// group sums are added in group order.  What the update needs besides is read
// beside the sums by the lanes that hold none.
template <bool kHalf>
__device__ void reduce_solve_scan(int32_t s, int32_t t0, int32_t t1, const double* partial,
                                  double* T, double* ctr, int32_t* done,
                                  far_align_stats_t* stats, const Params& prm, int32_t solve,
                                  const Progress& pg) {
  __shared__ double part[8][kVals];
  __shared__ double lin[kVals];
  __shared__ double pose[15];   // the scan's pose (three rows) and centre
  __shared__ int32_t iters;
  const int g = threadIdx.x >> 5, v = threadIdx.x & 31;
  if (g < 8 && v < kVals) {
    const double acc = strided_sum<kHalf>(partial, t0 + g, t1, v);
    part[g][v] = acc;
  } else if (g < 8) {
    const int q = g * 3 + v - kVals;
    if (q < 15)
      pose[q] = q < 12 ? T[16 * int64_t(s) + q] : ctr[3 * s + q - 12];
    else if (q == 15)
      iters = stats[s].iters;
  }
  __syncthreads();
  if (threadIdx.x < kVals) {
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += part[q][threadIdx.x];
    lin[threadIdx.x] = acc;
  }
  __syncthreads();
  // the statistics by the second wave, beside the solve
  if (threadIdx.x >= 64 && threadIdx.x < 64 + 44) {
    const int e = int(threadIdx.x) - 64;
    far_lin_t& out = stats[s].last;
    if (e < 36) {
      const int a = e / 6, b = e % 6, p = min(a, b), q = max(a, b);
      out.H[e] = lin[p * 6 - p * (p - 1) / 2 + (q - p)];   // row p of the upper triangle
    } else if (e < 42) {
      out.b[e - 36] = lin[21 + e - 36];
    } else if (e == 42) {
      out.cost = lin[27];
    } else {
      out.n_inliers = int64_t(lin[28]);
    }
  }
  if (threadIdx.x != 0) return;
  solve_scan(s, lin, pose, pose + 12, iters, T, ctr, done, stats, prm, solve);
  if (pg.word)
    __hip_atomic_store(pg.word, done[s] ? kAlignDone : pg.step, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void k_reduce_solve(int32_t S, const int32_t* begin,
                                                      const double* partial, double* T,
                                                      double* ctr, int32_t* done,
                                                      far_align_stats_t* stats, Params prm,
                                                      int32_t solve, uint32_t* bins, Progress pg) {
  // the next iteration's queue starts empty (this iteration's search has
  // read its bins)
  if (bins && blockIdx.x == 0 && threadIdx.x < kBins) bins[threadIdx.x] = 0u;
  const int32_t s = blockIdx.x;
  if (s >= S || done[s]) return;
  reduce_solve_scan<false>(s, begin[s], begin[s + 1], partial, T, ctr, done, stats, prm, solve, pg);
}

// ---------------------------------------------------------------- wide jobs
// One Gauss-Newton iteration of a small job in one launch.  With one lane per
// point, a scan of a few thousand points is a few dozen waves, each as long as
// its slowest chain of loads (first iteration 40 us, queued search 14 us for
// 5000 points), and an iteration is four launches.  Here a block of kWide
// lanes takes one wave's 64 points: the first wave certifies them, the points
// left over (in the first iteration all) are searched by 32 lanes each, every
// lane probing and ranking one of the 27 voxels, the first wave forms the
// terms and sums them, and the last block of a scan to finish sums the tiles
// and solves (a count per scan; each block's sums are released before it
// counts, and the last one acquires them).  The correspondences are those of
// the exact search, and the sums are taken in the order of the tile passes (per
// wave, then the two waves of a tile of 128, then the tiles), so the results
// are theirs bit for bit.  5000 points, first iteration 45 us in two launches
// and each later one about 45 us in four; 32 and 18.5 us in one.
constexpr int kWide = 512;        // lanes per block: 16 searches at once
constexpr int kWidePts = 64;

// The nearest map point of one query by 32 lanes (lane in [0, 32)), continuing
// from the candidate in top, the same in every lane; the result in every lane.
__device__ inline void nn_wide(const MapView& m, const Params& prm, double px, double py,
                               double pz, int lane, TopK<1>& top) {
  if (lane < 27) {
    int64_t kx = 0, ky = 0, kz = 0;   // in range: held when the point was located
    (void)voxel_index_fast(px, m.v, prm.inv_v, prm.v_pow2, &kx);
    (void)voxel_index_fast(py, m.v, prm.inv_v, prm.v_pow2, &ky);
    (void)voxel_index_fast(pz, m.v, prm.inv_v, prm.v_pow2, &kz);
    FaceOffsets fo;
    fo.f[0] = float(px - double(kx) * m.v);
    fo.f[1] = float(py - double(ky) * m.v);
    fo.f[2] = float(pz - double(kz) * m.v);
    fo.v = float(m.v);
    fo.slack = float(1e-7 * m.v);
    const double bound = fmin(prm.r2, top.bound());
    if (double(fo.lb2(lane)) <= bound) {
      int32_t cnt;
      const int32_t vox = map_find(m, kx + lane / 9 - 1, ky + (lane / 3) % 3 - 1,
                                   kz + lane % 3 - 1, &cnt);
      if (vox >= 0) {
        Query q = make_query(px, py, pz, prm.r2);
        q.bound_f = screen_bound(bound, q.m);
        scan_voxel_points<1, 10>(m.vox_pts, vox * m.nmax, cnt, q, prm.r2, top);
      }
    }
  }
  const int w = group_best(top.d[0], top.id[0]);
  top.d[0] = __shfl(top.d[0], w, kGroup);
  top.id[0] = __shfl(top.id[0], w, kGroup);
  top.pos[0] = __shfl(top.pos[0], w, kGroup);
}

// Sums over one wave of kNV values per lane into row[0 .. kNV): as the tile
// passes take them (FP32 through a table of the wave's own in LDS, FP64 by
// lane swaps).
template <class Real, int kNV>
__device__ inline void wave_sums(const Real* acc, float* tb, int lane, double* row) {
  if constexpr (std::is_same<Real, float>::value) {
    const int v = lane >> 2, quarter = lane & 3;
#pragma unroll
    for (int c0 = 0; c0 < kNV; c0 += kRedChunk) {
      // one wave: its LDS operations complete in order
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int q = 0; q < kRedChunk; ++q)
        if (c0 + q < kNV) tb[q * kRedRow + lane] = acc[c0 + q];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      double sv = 0.0;
      if (c0 + v < kNV) {
        const float* r = tb + v * kRedRow + 16 * quarter;
#pragma unroll
        for (int e = 0; e < 16; ++e) sv += double(r[e]);
      }
      sv += dpp_partner<0xB1>(sv);
      sv += dpp_partner<0x4E>(sv);
      if (quarter == 0 && c0 + v < kNV) row[c0 + v] = sv;
    }
  } else {
#pragma unroll
    for (int q = 0; q < kNV; ++q) {
      const double sv = wave_sum(acc[q]);
      if (lane == 0) row[q] = sv;
    }
  }
}

template <class Real, bool kGrad, bool kNoSA>
__global__ __launch_bounds__(kWide) void k_wide_iter(
    MapView m, const float4* __restrict__ pA, const float4* __restrict__ pB,
    const float2* __restrict__ pC, const int32_t* __restrict__ tile_scan,
    const uint32_t* __restrict__ tile_lo, const uint32_t* __restrict__ tile_hi, int64_t n_half,
    const int32_t* __restrict__ begin, double* T, double* ctr, int32_t* done, Params prm,
    double* partial, uint32_t* counter, far_align_stats_t* stats, int32_t solve, int32_t first,
    int32_t* corr, float* grad_src, int64_t n_src, int32_t* prev, Progress pg,
    int64_t n_one) {
  constexpr int kNV = kGrad ? 14 : kVals;
  __shared__ double q_p[kWidePts][3];
  __shared__ double q_d[kWidePts];
  __shared__ int32_t q_id[kWidePts], q_pos[kWidePts], q_lane[kWidePts], s_match[kWidePts];
  __shared__ int32_t q_n;
  __shared__ uint32_t s_last;
  __shared__ float tbl[std::is_same<Real, float>::value ? kRedChunk * kRedRow : 1];
  const int64_t hb = block_tile(n_half);
  if (hb < 0) return;
  const int64_t t = hb >> 1;
  // one scan: its tiles are known without their table, a load less before the
  // pose and the points
  const int32_t s = n_one > 0 ? (t * kTileMin < n_one ? 0 : -1) : tile_scan[t];
  if (s < 0 || done[s]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t lo = uint32_t(hb) * kWidePts, hi = uint32_t(n_one);
  int32_t t0 = 0, t1 = int32_t((n_one + kTileMin - 1) / kTileMin);
  if (n_one <= 0) {
    t0 = begin[s];
    t1 = begin[s + 1];
    lo = tile_lo[t] + uint32_t(kWidePts) * uint32_t(hb & 1);
    hi = tile_hi[t];
  }
  const uint32_t i = lo + uint32_t(lane);
  const bool own = tid < 64 && i < hi;
  const Pose P(T + 16 * int64_t(s));
  float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  double px = 0.0, py = 0.0, pz = 0.0;
  if (tid < 64) {
    bool queued = false;
    Cand c;
    c.pos = -1;
    c.d = 0.0;
    int32_t res = -1;
    if (own) {
      a = pA[i];
      const int32_t seed = first ? -1 : prev[i];
      int64_t kx = 0, ky = 0, kz = 0;
      const bool have = locate(a, P, m, prm, px, py, pz, kx, ky, kz);
      queued = have && (first || !nn_cert_try(m, px, py, pz, int32_t(kx), int32_t(ky),
                                              int32_t(kz), prm.r2, seed, c));
      if (!queued) {
        res = have && c.d <= prm.r2 ? c.pos : -1;
        if (prev) prev[i] = have ? c.pos : -1;
      }
    }
    s_match[lane] = res;
    const uint64_t bal = __ballot(queued);
    if (lane == 0) q_n = __popcll(bal);
    if (queued) {
      const int q = __popcll(bal & ((uint64_t(1) << lane) - 1));
      q_p[q][0] = px;
      q_p[q][1] = py;
      q_p[q][2] = pz;
      q_d[q] = c.d;
      q_id[q] = c.pos >= 0 ? __float_as_int(m.vox_pts[c.pos].w) : 0;
      q_pos[q] = c.pos;
      q_lane[q] = lane;
    }
  }
  __syncthreads();
  for (int q = tid / kGroup; q < q_n; q += kWide / kGroup) {
    TopK<1> top;
    top.init();
    const int32_t cp = q_pos[q];
    if (cp >= 0 && q_d[q] <= prm.r2) top.push(q_d[q], q_id[q], cp);
    nn_wide(m, prm, q_p[q][0], q_p[q][1], q_p[q][2], tid & (kGroup - 1), top);
    if ((tid & (kGroup - 1)) == 0) {
      s_match[q_lane[q]] = top.pos[0];
      if (prev) prev[lo + uint32_t(q_lane[q])] = top.pos[0] >= 0 ? top.pos[0] : cp;
    }
  }
  __syncthreads();
  if (tid < 64) {
    const double cx = ctr[3 * s], cy = ctr[3 * s + 1], cz = ctr[3 * s + 2];
    Real acc[kNV];
#pragma unroll
    for (int q = 0; q < kNV; ++q) acc[q] = Real(0);
    const int32_t res = s_match[lane];
    int32_t id_match = -1;
    Real gs[3] = {Real(0), Real(0), Real(0)};
    if (res >= 0) {
      const float4 r = m.vox_pts[res];
      const float4 sB = pB[i];
      const float2 sC = pC[i];
      const float4 ca = m.vox_cov[2 * int64_t(res)], cb = m.vox_cov[2 * int64_t(res) + 1];
      if (!kNoSA || (sB.x >= 0.0f && cb.z != 0.0f)) {
        id_match = __float_as_int(r.w);
        if constexpr (kGrad)
          grad_term<Real>(px, py, pz, a, r, ca, cb, sB, sC, P.R, prm.kappa2, acc, gs);
        else
          gicp_term<Real>(px, py, pz, r, ca, cb, sB, sC, P.R, cx, cy, cz, prm.kappa2, acc);
      }
    }
    if (own && corr) corr[__float_as_uint(a.w)] = id_match;
    if (kGrad && own && grad_src) {
      const uint32_t o = __float_as_uint(a.w);
      grad_src[o] = float(gs[0]);
      grad_src[n_src + o] = float(gs[1]);
      grad_src[2 * n_src + o] = float(gs[2]);
    }
    wave_sums<Real, kNV>(acc, tbl, lane, partial + hb * kStride);
  }
  if constexpr (!kGrad) {
    __syncthreads();
    if (tid == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      s_last = atomicAdd(&counter[s], 1u) + 1u == 2u * uint32_t(t1 - t0) ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid == 0) counter[s] = 0u;
    reduce_solve_scan<true>(s, t0, t1, partial, T, ctr, done, stats, prm, solve, pg);
  }
}

// Twist gradient about c from the gradient g of [R | t] (row-major 3 x 4)
// at pose T: with dR = [w]x R and dt = [w]x (t - c) + v, the rotation part
// is the axial vector of A - A^T for A = R G_R^T + (t - c) G_t^T and the
// translation part is G_t.  Shared by the host (one scan) and the batched
// reduction so that both give the same bits.
__host__ __device__ inline void twist_from_grad(const double* g, const double* T,
                                                const double* c, double* tw) {
  double A[9];
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q) {
      double x = 0.0;
      for (int l = 0; l < 3; ++l) x += T[4 * r + l] * g[4 * q + l];
      A[3 * r + q] = x + (T[4 * r + 3] - c[r]) * g[4 * q + 3];
    }
  tw[0] = A[5] - A[7];
  tw[1] = A[6] - A[2];
  tw[2] = A[1] - A[3];
  for (int q = 0; q < 3; ++q) tw[3 + q] = g[4 * q + 3];
}

// One block per scan: the sum of the 14 gradient partials of the scan's
// tiles in tile order (eight interleaved groups, then the groups in order,
// as k_reduce_solve) into out[14 s ..]; with gT given also the per-scan
// outputs of the batched gradient (grad_T, the twist about c[3 s ..] or the
// origin, cost, inliers).
template <bool kHalf>
__global__ __launch_bounds__(256) void k_reduce_grad(const int32_t* begin,
                                                     const double* partial, double* out,
                                                     const double* T, const double* c,
                                                     double* gT, double* gtw, double* cost,
                                                     int64_t* n_inl) {
  __shared__ double part[8][14];
  __shared__ double sum[14];
  const int s = blockIdx.x;
  const int g = threadIdx.x >> 5, v = threadIdx.x & 31;
  if (v < 14) {
    const double acc = strided_sum<kHalf>(partial, begin[s] + g, begin[s + 1], v);
    part[g][v] = acc;
  }
  __syncthreads();
  if (threadIdx.x < 14) {
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += part[q][threadIdx.x];
    out[14 * int64_t(s) + threadIdx.x] = acc;
    sum[threadIdx.x] = acc;
  }
  if (!gT) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double zero[3] = {0.0, 0.0, 0.0};
    for (int q = 0; q < 12; ++q) gT[12 * int64_t(s) + q] = sum[q];
    twist_from_grad(sum, T + 16 * int64_t(s), c ? c + 3 * int64_t(s) : zero,
                    gtw + 6 * int64_t(s));
    if (cost) cost[s] = sum[12];
    if (n_inl) n_inl[s] = int64_t(sum[13]);
  }
}

}  // namespace

// Device workspace of the align driver, owned by the map and reused (with its
// captured graph) while the call arguments stay the same.
// Jobs of up to kWideMax points (at the smallest tile, over the voxels) run
// k_wide_iter.  Above, one lane per point fills the chip by itself and the wide
// search does more work than the pruned one (about 540 candidates a query).  One scan
// of 16000, 32000, 48000 and 64000 points, wide against the tile passes: an align of one
// iteration 87, 98, 122 and 134 us against 112, 113, 121 and 124, of six 251, 294,
// 373 and 419 against 446, 456, 453 and 454.
// A batch has half-filled blocks, and each scan's last block holds its 512 lanes
// through a solve, so tiles and scans together are limited too.  Eight iterations of
// 32, 64, 128, 160, 200, 256 and 400 scans of 700, 250, 150, 100, 50, 50 and 10 points, wide
// against the tile passes: 268, 285, 359, 436, 414, 453 and 447 us against 371, 373, 365,
// 384, 354, 367 and 326; 2000 of 10 points 1760 against 433.
constexpr int64_t kWideLoad = 440;   // of tiles (an upper bound) and scans
static_assert(kWideLoad <= kTileLdsScans, "the setup of a wide job clears its counters");
constexpr int64_t kWideMax = 48 * 1024;

struct AlignWS {
  int32_t S = 0;
  int64_t max_tiles = 0;
  int64_t n_cap = 0;
  int32_t* tile_scan = nullptr;
  uint32_t* tile_lo = nullptr;
  uint32_t* tile_hi = nullptr;
  int32_t* begin = nullptr;
  int32_t* bad = nullptr;
  int32_t* done = nullptr;
  double* ctr = nullptr;
  double* partial = nullptr;
  int64_t* offsets = nullptr;   // single-scan path
  double* T = nullptr;          // single-scan path
  double* cfix = nullptr;       // fixed centre (linearize)
  far_align_stats_t* stats = nullptr;   // single-scan path
  double* gsum = nullptr;       // gradient sums
  uint32_t* counter = nullptr;  // per scan: blocks of an iteration that are done (wide jobs)
  // locality-ordered packed source and its sort buffers
  float4* pA = nullptr;
  float4* pB = nullptr;
  float2* pC = nullptr;
  int32_t* prev = nullptr;      // per packed point: seed of the next search (vox_pts slot)
  // the three linearisation passes: per packed point its match, and the
  // search queue (kBins bins of q_bin_cap entries, SoA FP64 positions)
  int32_t* match = nullptr;
  uint32_t* q_idx = nullptr;
  int32_t* q_cand = nullptr;
  double* q_p = nullptr;
  uint32_t* q_count = nullptr;
  int64_t q_bin_cap = 0;
  uint64_t* okeys = nullptr;
  uint64_t* okeys_alt = nullptr;
  uint32_t* ovals = nullptr;
  uint32_t* ovals_alt = nullptr;
  void* arena = nullptr;
  size_t arena_cap = 0;
  // Two captured aligns (e.g. for two covariance buffers used in turn), each
  // with the argument set it was captured for; the older one is replaced.
  struct Captured {
    hipGraphExec_t exec = nullptr;
    const void* key[12] = {};
    int64_t n = -1;
    Params prm{};
    int32_t prec = -1;
    int32_t S = -1;
    int32_t tile = -1;
    int32_t grid = -1;   // g_lin_blocks_per_cu at capture
    uint64_t used = 0;
  };
  Captured cap[2];
  uint64_t clock = 0;
  // the argument sets of the last two direct launches
  const void* pending[12] = {};
  const void* pending2[12] = {};
};

void free_ws(AlignWS* w) {
  if (!w) return;
  for (auto& c : w->cap)
    if (c.exec) (void)hipGraphExecDestroy(c.exec);
  void* ptrs[] = {w->tile_scan, w->tile_lo, w->tile_hi, w->begin, w->bad, w->done, w->ctr,
                  w->partial, w->offsets, w->T, w->cfix, w->stats, w->gsum, w->counter, w->pA, w->pB, w->pC,
                  w->prev, w->match, w->q_idx, w->q_cand, w->q_p, w->q_count,
                  w->okeys, w->okeys_alt, w->ovals, w->ovals_alt, w->arena};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  delete w;
}

namespace {

int ceil_log2_i(int64_t x) {
  int l = 0;
  while ((int64_t(1) << l) < x) ++l;
  return l;
}

far_status_t ensure_ws(far_map_s* m, int32_t S, int64_t max_tiles, int64_t n, AlignWS** out) {
  AlignWS* w = m->ws;
  if (w && w->S >= S && w->max_tiles >= max_tiles && w->n_cap >= n) {
    *out = w;
    return FAR_OK;
  }
  if (w) {
    FAR_HIP(hipDeviceSynchronize());
    free_ws(w);
    m->ws = nullptr;
  }
  w = new AlignWS();
  m->ws = w;
  w->S = S < 64 ? 64 : S;
  w->max_tiles = max_tiles < 1024 ? 1024 : max_tiles;
  w->n_cap = n < 4096 ? 4096 : n;
  const size_t nc = size_t(w->n_cap);
  FAR_HIP(hipMalloc(&w->tile_scan, size_t(w->max_tiles) * sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->tile_lo, size_t(w->max_tiles) * sizeof(uint32_t)));
  FAR_HIP(hipMalloc(&w->tile_hi, size_t(w->max_tiles) * sizeof(uint32_t)));
  // (two rows a tile for the tiles of a wide job, at most kWideMax points)
  const int64_t rows = std::max(w->max_tiles,
                                std::min(2 * w->max_tiles, 2 * (kWideMax / kTileMin + w->S)));
  FAR_HIP(hipMalloc(&w->partial, size_t(rows) * kStride * sizeof(double)));
  FAR_HIP(hipMalloc(&w->counter, size_t(w->S) * sizeof(uint32_t)));
  FAR_HIP(hipMalloc(&w->begin, size_t(w->S + 1) * sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->bad, sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->done, size_t(w->S) * sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->ctr, size_t(w->S) * 3 * sizeof(double)));
  FAR_HIP(hipMalloc(&w->offsets, 2 * sizeof(int64_t)));
  FAR_HIP(hipMalloc(&w->T, 16 * sizeof(double)));
  FAR_HIP(hipMalloc(&w->cfix, 3 * sizeof(double)));
  FAR_HIP(hipMalloc(&w->stats, sizeof(far_align_stats_t)));
  FAR_HIP(hipMalloc(&w->gsum, kStride * sizeof(double)));
  FAR_HIP(hipMalloc(&w->pA, nc * sizeof(float4)));
  FAR_HIP(hipMalloc(&w->pB, nc * sizeof(float4)));
  FAR_HIP(hipMalloc(&w->pC, nc * sizeof(float2)));
  FAR_HIP(hipMalloc(&w->prev, nc * sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->match, nc * sizeof(int32_t)));
  // a bin holds the queues of its tiles (every kBins-th): at most
  // ceil(max_tiles / kBins) tiles of at most kTileMax points
  w->q_bin_cap = ((w->max_tiles + kBins - 1) / kBins) * kTileMax;
  const size_t qc = size_t(kBins) * size_t(w->q_bin_cap);
  FAR_HIP(hipMalloc(&w->q_idx, qc * sizeof(uint32_t)));
  FAR_HIP(hipMalloc(&w->q_cand, qc * sizeof(int32_t)));
  FAR_HIP(hipMalloc(&w->q_p, 3 * qc * sizeof(double)));
  FAR_HIP(hipMalloc(&w->q_count, kBins * sizeof(uint32_t)));
  FAR_HIP(hipMalloc(&w->okeys, nc * sizeof(uint64_t)));
  FAR_HIP(hipMalloc(&w->okeys_alt, nc * sizeof(uint64_t)));
  FAR_HIP(hipMalloc(&w->ovals, nc * sizeof(uint32_t)));
  FAR_HIP(hipMalloc(&w->ovals_alt, nc * sizeof(uint32_t)));
  w->arena_cap = radix_sort_scratch_bytes(w->n_cap);
  FAR_HIP(hipMalloc(&w->arena, w->arena_cap));
  *out = w;
  return FAR_OK;
}

struct Job {
  const float* src;
  const int64_t* offsets;
  int32_t S;
  int64_t n_total;
  const float* cov6;
  const uint8_t* valid;
  double* T;
  far_align_stats_t* stats;
  const double* c_fixed;   // non-null: one linearisation about this centre, no solve
  int32_t* corr;
  Params prm;
  int32_t precision;
  double* gsum = nullptr;      // non-null: one gradient pass, 14 sums per scan here
  float* grad_src = nullptr;   // gradient pass: per-point source gradient or null
  // batched gradient outputs (per scan; null for the one-scan path)
  const double* g_c = nullptr;
  double* g_T = nullptr;
  double* g_tw = nullptr;
  double* g_cost = nullptr;
  int64_t* g_n = nullptr;
  int32_t tile = kTileDefault; // points per tile (the map's schedule)
  HostSlot* slot = nullptr;    // a one-scan align the host waits for: its progress, or null
  const uint32_t* order = nullptr;   // caller's locality order of the source, or null
  // the source already packed by the caller (A, B, C as the pack writes
  // them, in a locality order), or null
  const float4* in_A = nullptr;
  const float4* in_B = nullptr;
  const float2* in_C = nullptr;
};

// Blocks per CU of the persistent launch of the tile passes (k_cert and the
// term pass); 0: one block per tile.
int32_t g_lin_blocks_per_cu = 0;

// One linearisation (or gradient) at the map's tile size: the term pass
// with its own exact search when there are no seeds (first), else the
// certified search, the exact search of the queue and the term pass.
template <class Real, bool kGrad>
far_status_t launch_lin(int32_t tile, int64_t grid, hipStream_t st, const MapView& mv,
                        const AlignWS* w, int64_t max_tiles, const Job& j, bool first) {
  // the fine-cell search only where the index exists for the current map
  const bool fine = j.prm.fine_nn && mv.fine_ok;
  int32_t* prev = kGrad ? nullptr : w->prev;
  const bool search = first || fine || !prev;
  const int64_t vgrid = grid;
  if (g_lin_blocks_per_cu > 0) {
    const int64_t pg = ((int64_t(g_lin_blocks_per_cu) * device_cu_count() + 7) / 8) * 8;
    if (pg < grid) grid = pg;
  }
  const float4* pA = j.in_A ? j.in_A : w->pA;
  const float4* pB = j.in_A ? j.in_B : w->pB;
  const float2* pC = j.in_A ? j.in_C : w->pC;
  if (!search) {
    // the bins were cleared by the solve of the previous iteration
    Queue Q{w->q_idx, w->q_cand, w->q_p, w->q_count, w->q_bin_cap, kBins * w->q_bin_cap};
    const bool loop = grid < vgrid;
    switch (tile * 2 + (loop ? 1 : 0)) {
#define FAR_CERT_CASE(B, L)                                                               \
  case B * 2 + L:                                                                         \
    k_cert<B, L><<<unsigned(grid), B, 0, st>>>(mv, pA, w->tile_scan, w->tile_lo,         \
                                               w->tile_hi, max_tiles, j.T, w->done, j.prm, \
                                               w->match, prev, Q, vgrid);                 \
    break;
      FAR_CERT_CASE(128, 0)
      FAR_CERT_CASE(128, 1)
      FAR_CERT_CASE(256, 0)
      FAR_CERT_CASE(256, 1)
      FAR_CERT_CASE(512, 0)
      FAR_CERT_CASE(512, 1)
#undef FAR_CERT_CASE
      default:
        set_error("internal: unsupported tile size %d", tile);
        return FAR_E_INVALID;
    }
    FAR_HIP(hipGetLastError());
    k_search<<<unsigned(8 * device_cu_count()), kSearchThreads, 0, st>>>(mv, Q, j.prm,
                                                                         w->match, prev);
    FAR_HIP(hipGetLastError());
  }
  const bool loop = grid < vgrid;
  switch (tile * 16 + (fine ? 8 : 0) + (j.prm.sa_off ? 4 : 0) + (search ? 2 : 0) +
          (loop ? 1 : 0)) {
#define FAR_LIN_CASE(B, F, N, X, L)                                                       \
  case B * 16 + F * 8 + N * 4 + X * 2 + L:                                                \
    k_linearize<Real, kGrad, B, F, N, X, L><<<unsigned(grid), B, 0, st>>>(               \
        mv, pA, pB, pC, w->tile_scan, w->tile_lo, w->tile_hi, max_tiles, j.T,            \
        w->ctr, w->done, j.prm, w->partial, j.corr, kGrad ? j.grad_src : nullptr,        \
        j.n_total, w->match, prev, vgrid);                                                \
    break;
#define FAR_LIN_CASES(B)           \
    FAR_LIN_CASE(B, 0, 0, 0, 0)    \
    FAR_LIN_CASE(B, 0, 0, 0, 1)    \
    FAR_LIN_CASE(B, 0, 0, 1, 0)    \
    FAR_LIN_CASE(B, 0, 0, 1, 1)    \
    FAR_LIN_CASE(B, 0, 1, 0, 0)    \
    FAR_LIN_CASE(B, 0, 1, 0, 1)    \
    FAR_LIN_CASE(B, 0, 1, 1, 0)    \
    FAR_LIN_CASE(B, 0, 1, 1, 1)    \
    FAR_LIN_CASE(B, 1, 0, 1, 0)    \
    FAR_LIN_CASE(B, 1, 0, 1, 1)    \
    FAR_LIN_CASE(B, 1, 1, 1, 0)    \
    FAR_LIN_CASE(B, 1, 1, 1, 1)
    FAR_LIN_CASES(128)
    FAR_LIN_CASES(256)
    FAR_LIN_CASES(512)
#undef FAR_LIN_CASES
#undef FAR_LIN_CASE
    default:
      set_error("internal: unsupported tile size %d", tile);
      return FAR_E_INVALID;
  }
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

// One iteration (or linearisation, or gradient) of a wide job.
template <class Real, bool kGrad>
far_status_t launch_wide(hipStream_t st, const MapView& mv, const AlignWS* w, int64_t max_tiles,
                         const Job& j, bool first, Progress pg = {}) {
  const float4* pA = j.in_A ? j.in_A : w->pA;
  const float4* pB = j.in_A ? j.in_B : w->pB;
  const float2* pC = j.in_A ? j.in_C : w->pC;
  const int64_t n_half = 2 * max_tiles;
  const unsigned grid = unsigned(((n_half + 7) / 8) * 8);
  auto go = [&](auto no_sa) {
    k_wide_iter<Real, kGrad, decltype(no_sa)::value><<<grid, kWide, 0, st>>>(
        mv, pA, pB, pC, w->tile_scan, w->tile_lo, w->tile_hi, n_half, w->begin, j.T, w->ctr,
        w->done, j.prm, w->partial, w->counter, j.stats, j.c_fixed ? 0 : 1, first ? 1 : 0,
        j.corr, kGrad ? j.grad_src : nullptr, j.n_total, kGrad ? nullptr : w->prev, pg,
        j.S == 1 ? j.n_total : 0);
  };
  if (j.prm.sa_off)
    go(std::true_type());
  else
    go(std::false_type());
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

// The job's setup: tiles, per-scan state and (one given) a one-scan job's
// inputs.
far_status_t enqueue_setup(const AlignWS* w, const Job& j, int64_t max_tiles,
                           const SingleArgs* one, hipStream_t st) {
  SingleArgs none;
  memset(&none, 0, sizeof(none));
  none.n = -1;
  if (j.S <= kTileLdsScans) {
    const int64_t items = std::max<int64_t>(max_tiles, j.S);
    k_setup<<<unsigned((items + 255) / 256), 256, 0, st>>>(
        one ? *one : none, const_cast<int64_t*>(j.offsets), j.T, w->cfix, j.S, j.n_total,
        max_tiles, j.tile, w->begin, w->bad, w->tile_scan, w->tile_lo, w->tile_hi,
        j.prm.recenter, j.c_fixed, j.stats, w->done, w->ctr, w->counter);
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  }
  k_tile_begin<<<1, 64, 0, st>>>(j.offsets, j.S, j.n_total, max_tiles, j.tile, w->begin,
                                 w->bad);
  FAR_HIP(hipGetLastError());
  k_tile_fill<<<unsigned((max_tiles + 255) / 256), 256, 0, st>>>(
      j.offsets, j.S, max_tiles, j.tile, w->begin, w->tile_scan, w->tile_lo, w->tile_hi);
  FAR_HIP(hipGetLastError());
  k_init<<<(j.S + 255) / 256, 256, 0, st>>>(j.S, j.T, w->bad, j.prm.recenter, j.c_fixed,
                                            j.stats, w->done, w->ctr);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

// Before iteration `it` (from 0) of an align whose progress the host sees:
// false when the scan is done, so that the iterations left are not launched
// (each would be up to four launches of kernels that find nothing to do, about
// 4 us of host time each).  The host stays at most kAhead iterations ahead,
// enough to keep the device busy.  Behind other work on the stream it watches a
// millisecond for each iteration and then enqueues that one all the same, so
// that the align can still stop early once the work before it has ended (the
// call waits for its result in any case).
constexpr uint32_t kAhead = 2;

bool wait_progress(HostSlot* slot, int it) {
  const auto t0 = std::chrono::steady_clock::now();
  for (int spin = 0;; ++spin) {
    const uint32_t p = __atomic_load_n(slot->host, __ATOMIC_ACQUIRE);
    if (p == kAlignDone) return false;
    if (uint32_t(it) <= p + kAhead) return true;
    if ((spin & 255) == 255 &&
        std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(1))
      return true;
  }
}

// Enqueue the whole job (setup, locality packing, iterations) on st; a
// one-scan job's setup (its pose by value) has run before.  Nothing here
// allocates or clears memory, so it can be recorded into a graph.
far_status_t enqueue(far_map_s* m, AlignWS* w, const Job& j, int64_t max_tiles, bool setup,
                     hipStream_t st) {
  MapView mv = m->view();
  if (setup) FAR_TRY(enqueue_setup(w, j, max_tiles, nullptr, st));
  if (j.n_total > 0 && !j.in_A) {   // (a source packed by the caller is used as it is)
    const unsigned nb = unsigned((j.n_total + 255) / 256);
    const uint32_t* perm = j.order;   // the caller's order (e.g. the covariance grid's)
    uint32_t* inv = w->ovals_alt;
    if (!perm) {
      k_order_keys<<<nb, 256, 0, st>>>(j.src, j.n_total, j.offsets, j.S, m->p.voxel_size,
                                       w->okeys, w->ovals);
      FAR_HIP(hipGetLastError());
      Scratch scr(st, w->arena, w->arena_cap);
      bool in_alt = false;
      FAR_TRY(radix_sort_pairs(w->okeys, w->ovals, w->okeys_alt, w->ovals_alt, j.n_total,
                               24 + ceil_log2_i(j.S), st, scr, &in_alt));
      perm = in_alt ? w->ovals_alt : w->ovals;
      inv = in_alt ? w->ovals : w->ovals_alt;
    }
    const unsigned nb8 = ((nb + 7) / 8) * 8;
    if (j.n_total <= kGatherPack) {
      k_pack_gather<<<nb8, 256, 0, st>>>(j.src, j.cov6, j.valid, j.n_total, perm, w->pA, w->pB,
                                         w->pC);
    } else {
      k_invert<<<nb8, 256, 0, st>>>(perm, j.n_total, inv);
      FAR_HIP(hipGetLastError());
      k_pack<<<nb8, 256, 0, st>>>(j.src, j.cov6, j.valid, j.n_total, inv, w->pA, w->pB, w->pC);
    }
    FAR_HIP(hipGetLastError());
  }
  const bool wide = j.n_total <= kWideMax && max_tiles + j.S <= kWideLoad &&
                    j.tile == kTileMin && !(j.prm.fine_nn && mv.fine_ok) &&
                    g_lin_blocks_per_cu == 0;
  const int64_t grid = ((max_tiles + 7) / 8) * 8;   // one block per tile
  const bool fp64 = j.precision == FAR_PREC_FP64;
  if (j.gsum) {
    if (wide) {
      FAR_TRY((fp64 ? launch_wide<double, true>(st, mv, w, max_tiles, j, true)
                    : launch_wide<float, true>(st, mv, w, max_tiles, j, true)));
      k_reduce_grad<true><<<unsigned(j.S), 256, 0, st>>>(w->begin, w->partial, j.gsum, j.T,
                                                         j.g_c, j.g_T, j.g_tw, j.g_cost, j.g_n);
    } else {
      FAR_TRY((fp64 ? launch_lin<double, true>(j.tile, grid, st, mv, w, max_tiles, j, true)
                    : launch_lin<float, true>(j.tile, grid, st, mv, w, max_tiles, j, true)));
      k_reduce_grad<false><<<unsigned(j.S), 256, 0, st>>>(w->begin, w->partial, j.gsum, j.T,
                                                          j.g_c, j.g_T, j.g_tw, j.g_cost, j.g_n);
    }
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  }
  const int iters = j.c_fixed ? 1 : j.prm.max_iters;
  for (int it = 0; it < iters; ++it) {
    if (j.slot && !wait_progress(j.slot, it)) break;
    const Progress pg{j.slot ? j.slot->dev : nullptr, uint32_t(it + 1)};
    TimedScope ts(FAR_TIME_LINEARIZE, st);
    if (wide) {
      FAR_TRY((fp64 ? launch_wide<double, false>(st, mv, w, max_tiles, j, it == 0, pg)
                    : launch_wide<float, false>(st, mv, w, max_tiles, j, it == 0, pg)));
      continue;
    }
    FAR_TRY((fp64 ? launch_lin<double, false>(j.tile, grid, st, mv, w, max_tiles, j, it == 0)
                  : launch_lin<float, false>(j.tile, grid, st, mv, w, max_tiles, j, it == 0)));
    ts.stop();
    k_reduce_solve<<<unsigned(j.S), 256, 0, st>>>(j.S, w->begin, w->partial, j.T, w->ctr,
                                                  w->done, j.stats, j.prm, j.c_fixed ? 0 : 1,
                                                  it + 1 < iters ? w->q_count : nullptr, pg);
    FAR_HIP(hipGetLastError());
  }
  return FAR_OK;
}

bool same_params(const Params& a, const Params& b) {
  return a.r2 == b.r2 && a.kappa2 == b.kappa2 && a.inv_v == b.inv_v && a.v_pow2 == b.v_pow2 &&
         a.eps == b.eps && a.max_iters == b.max_iters && a.recenter == b.recenter &&
         a.fine_nn == b.fine_nn && a.sa_off == b.sa_off;
}

// Run a job, through a cached graph when the stream allows capture.
// one: a one-scan job's inputs (its offsets and pose go to the workspace).
far_status_t run_job(far_map_s* m, const Job& j0, hipStream_t st, bool use_graph,
                     const SingleArgs* one = nullptr) {
  Job j = j0;
  j.tile = m->sched_tile;
  // a job too small to give every CU two blocks at the map's tile (one scan
  // of ~100k points) runs at the smallest tile: twice the blocks to hide
  // the search latency
  if (j.tile > kTileMin && (j.n_total + j.tile - 1) / j.tile < 2 * int64_t(device_cu_count()))
    j.tile = kTileMin;
  j.prm.fine_nn = m->sched_fine;
  const int64_t max_tiles = (j.n_total + j.tile - 1) / j.tile + j.S;
  AlignWS* w = nullptr;
  FAR_TRY(ensure_ws(m, j.S, max_tiles, j.n_total, &w));
  // the fine index of the current map (stream-ordered), when it is used
  if (j.prm.fine_nn) FAR_TRY(fine_build(m, st));
  (void)device_cu_count();   // query the device outside any capture
  if (one) FAR_TRY(enqueue_setup(w, j, max_tiles, one, st));
  // a one-scan align that is launched directly reports its progress
  HostSlot* const slot = j.slot;
  j.slot = nullptr;
  auto direct = [&]() {
    if (slot) slot->take(st);
    if (slot && slot->host) {
      slot->pending = st;
      slot->busy = true;
      j.slot = slot;
    }
    return enqueue(m, w, j, max_tiles, !one, st);
  };
  if (!use_graph || st == nullptr || timing_on()) return direct();
  // the captured map view holds the fine-index flag: a graph captured with a
  // different flag must not be replayed
  const void* key[12] = {j.src, j.offsets, j.cov6, j.valid, j.T, j.stats, j.c_fixed, j.corr,
                         j.order, j.in_A,
                         m->vox_pts,
                         reinterpret_cast<const void*>(intptr_t(m->fine_ok) |
                                                       (intptr_t(m->ghost_ok) << 1))};
  AlignWS::Captured* hit = nullptr;
  for (auto& c : w->cap)
    if (c.exec && c.n == j.n_total && c.S == j.S && c.prec == j.precision &&
        c.tile == j.tile && c.grid == g_lin_blocks_per_cu &&
        memcmp(c.key, key, sizeof(key)) == 0 && same_params(c.prm, j.prm))
      hit = &c;
  if (!hit) {
    // Capture only once an argument set repeats (two calls apart at most): a
    // call on other buffers launches directly and pays no capture.  (Buffers are
    // what is compared: the same ones with another number of points or other
    // parameters are captured anew at each call.)
    if (memcmp(w->pending, key, sizeof(key)) != 0 && memcmp(w->pending2, key, sizeof(key)) != 0) {
      memcpy(w->pending2, w->pending, sizeof(key));
      memcpy(w->pending, key, sizeof(key));
      return direct();
    }
    hit = w->cap[0].used <= w->cap[1].used ? &w->cap[0] : &w->cap[1];
    if (hit->exec) {
      FAR_HIP(hipGraphExecDestroy(hit->exec));
      hit->exec = nullptr;
    }
    hipGraph_t g = nullptr;
    FAR_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    far_status_t rs = enqueue(m, w, j, max_tiles, !one, st);
    hipError_t e = hipStreamEndCapture(st, &g);
    if (rs != FAR_OK) {
      if (g) (void)hipGraphDestroy(g);
      return rs;
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture", __FILE__, __LINE__);
    e = hipGraphInstantiate(&hit->exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      hit->exec = nullptr;
      return hip_fail(e, "hipGraphInstantiate", __FILE__, __LINE__);
    }
    memcpy(hit->key, key, sizeof(key));
    hit->n = j.n_total;
    hit->S = j.S;
    hit->prec = j.precision;
    hit->prm = j.prm;
    hit->tile = j.tile;
    hit->grid = g_lin_blocks_per_cu;
  }
  hit->used = ++w->clock;
  FAR_HIP(hipGraphLaunch(hit->exec, st));
  return FAR_OK;
}

// A precision argument: far_precision_t, optionally with FAR_OPT_NO_SA.
bool precision_ok(int32_t p) {
  const int32_t base = p & ~int32_t(FAR_OPT_NO_SA);
  return base == FAR_PREC_FP32 || base == FAR_PREC_FP64;
}
int32_t precision_of(int32_t p) { return p & ~int32_t(FAR_OPT_NO_SA); }

bool params_ok(const far_align_params_t* p) {
  return p && p->tau > 0.0 && std::isfinite(p->tau) && p->kappa > 0.0 &&
         std::isfinite(p->kappa) && p->max_iters >= 1 && p->max_iters <= 64 &&
         p->eps >= 0.0 && precision_ok(p->precision);
}

Params make_params(const far_map_s* m, double tau, double kappa, double eps, int32_t max_iters,
                   int32_t recenter, int32_t precision) {
  Params prm;
  memset(&prm, 0, sizeof(prm));
  prm.sa_off = (precision & FAR_OPT_NO_SA) ? 1 : 0;
  double r = tau < m->p.voxel_size ? tau : m->p.voxel_size;
  prm.r2 = r * r;
  prm.kappa2 = kappa * kappa;
  int e2 = 0;
  prm.v_pow2 = std::frexp(m->p.voxel_size, &e2) == 0.5 ? 1 : 0;
  prm.inv_v = 1.0 / m->p.voxel_size;
  prm.eps = eps;
  prm.max_iters = max_iters;
  prm.recenter = recenter ? 1 : 0;
  prm.fine_nn = 0;
  return prm;
}

void lin_from_stats(const far_align_stats_t& st, far_lin_t* out) { *out = st.last; }

// The linearisation a one-scan job left in its stats (zero without one),
// copied to the caller's device buffer by the lanes of one wave.
__global__ void k_copy_lin(const far_align_stats_t* st, far_lin_t* out) {
  constexpr int kWords = int(sizeof(far_lin_t) / sizeof(double));
  static_assert(sizeof(far_lin_t) % sizeof(double) == 0, "far_lin_t is whole doubles");
  const double* src = st ? reinterpret_cast<const double*>(&st->last) : nullptr;
  double* dst = reinterpret_cast<double*>(out);
  for (int q = threadIdx.x; q < kWords; q += blockDim.x) dst[q] = src ? src[q] : 0.0;
}

}  // namespace
}  // namespace far

using namespace far;

extern "C" {

const double kOrigin[3] = {0.0, 0.0, 0.0};

static SingleArgs single_args(int64_t n, const double T[16], const double c[3]) {
  SingleArgs a;
  a.n = n;
  memcpy(a.T, T, sizeof(a.T));
  memcpy(a.c, c, sizeof(a.c));
  return a;
}

far_status_t far_gicp_linearize(far_map_t m, const float* src, const float* cov6,
                                const uint8_t* valid, int64_t n, const double T[16],
                                double tau, double kappa, const double c[3],
                                int32_t precision, int32_t* corr, far_lin_t* out,
                                far_stream_t stream) {
  if (!m || !T || !out || n < 0 || n >= (int64_t(1) << 31) || !(tau > 0.0) ||
      !(kappa > 0.0) || (n > 0 && (!src || !cov6 || !valid)) ||
      !precision_ok(precision)) {
    set_error("far_gicp_linearize: invalid argument");
    return FAR_E_INVALID;
  }
  memset(out, 0, sizeof(*out));
  if (n == 0) return FAR_OK;
  hipStream_t st = S(stream);
  AlignWS* w = nullptr;
  FAR_TRY(ensure_ws(m, 1, (n + kTileMin - 1) / kTileMin + 1, n, &w));
  const SingleArgs one = single_args(n, T, c ? c : kOrigin);
  Job j{src, w->offsets, 1, n, cov6, valid, w->T, w->stats, w->cfix, corr,
        make_params(m, tau, kappa, 0.0, 1, 0, precision), precision_of(precision)};
  FAR_TRY(run_job(m, j, st, false, &one));
  far_align_stats_t hs;
  FAR_TRY(fetch(st, &hs, w->stats, sizeof(hs)));
  lin_from_stats(hs, out);
  return FAR_OK;
}

far_status_t far_gicp_linearize_async(far_map_t m, const float* src, const float* cov6,
                                      const uint8_t* valid, int64_t n, const double T[16],
                                      double tau, double kappa, const double c[3],
                                      int32_t precision, int32_t* corr, far_lin_t* out,
                                      far_stream_t stream) {
  if (!m || !T || !out || n < 0 || n >= (int64_t(1) << 31) || !(tau > 0.0) ||
      !(kappa > 0.0) || (n > 0 && (!src || !cov6 || !valid)) ||
      !precision_ok(precision)) {
    set_error("far_gicp_linearize_async: invalid argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  if (n == 0) {
    k_copy_lin<<<1, 64, 0, st>>>(nullptr, out);
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  }
  AlignWS* w = nullptr;
  FAR_TRY(ensure_ws(m, 1, (n + kTileMin - 1) / kTileMin + 1, n, &w));
  const SingleArgs one = single_args(n, T, c ? c : kOrigin);
  Job j{src, w->offsets, 1, n, cov6, valid, w->T, w->stats, w->cfix, corr,
        make_params(m, tau, kappa, 0.0, 1, 0, precision), precision_of(precision)};
  FAR_TRY(run_job(m, j, st, false, &one));
  k_copy_lin<<<1, 64, 0, st>>>(w->stats, out);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

far_status_t far_set_linearize_grid(int32_t blocks_per_cu) {
  if (blocks_per_cu < 0 || blocks_per_cu > 64) {
    set_error("far_set_linearize_grid: blocks_per_cu must be in [0, 64]");
    return FAR_E_INVALID;
  }
  g_lin_blocks_per_cu = blocks_per_cu;
  return FAR_OK;
}

far_status_t far_get_linearize_grid(int32_t* blocks_per_cu) {
  if (!blocks_per_cu) {
    set_error("far_get_linearize_grid: null argument");
    return FAR_E_INVALID;
  }
  *blocks_per_cu = g_lin_blocks_per_cu;
  return FAR_OK;
}

far_status_t far_map_reserve(far_map_t m, int64_t max_points, int32_t max_scans,
                             far_stream_t stream) {
  (void)stream;
  if (!m || max_points < 0 || max_points >= (int64_t(1) << 31) || max_scans < 1) {
    set_error("far_map_reserve: invalid argument");
    return FAR_E_INVALID;
  }
  AlignWS* w = nullptr;
  return ensure_ws(m, max_scans, (max_points + kTileMin - 1) / kTileMin + max_scans,
                   max_points, &w);
}

far_status_t far_gicp_gradient(far_map_t m, const float* src, const float* cov6,
                               const uint8_t* valid, int64_t n, const double T[16], double tau,
                               double kappa, const double c[3], int32_t precision,
                               double grad_T[12], double grad_twist[6], float* grad_src,
                               double* cost, int64_t* n_inliers, far_stream_t stream) {
  if (!m || !T || !grad_T || !grad_twist || n < 0 || n >= (int64_t(1) << 31) ||
      !(tau > 0.0) || !(kappa > 0.0) || (n > 0 && (!src || !cov6 || !valid)) ||
      !precision_ok(precision)) {
    set_error("far_gicp_gradient: invalid argument");
    return FAR_E_INVALID;
  }
  for (int q = 0; q < 12; ++q) grad_T[q] = 0.0;
  for (int q = 0; q < 6; ++q) grad_twist[q] = 0.0;
  if (cost) *cost = 0.0;
  if (n_inliers) *n_inliers = 0;
  if (n == 0) return FAR_OK;
  hipStream_t st = S(stream);
  AlignWS* w = nullptr;
  FAR_TRY(ensure_ws(m, 1, (n + kTileMin - 1) / kTileMin + 1, n, &w));
  const double cc[3] = {c ? c[0] : 0.0, c ? c[1] : 0.0, c ? c[2] : 0.0};
  {
    TimedScope ts(FAR_TIME_GRADIENT, st);
    const SingleArgs one = single_args(n, T, cc);
    Job j{src, w->offsets, 1, n, cov6, valid, w->T, w->stats, w->cfix, nullptr,
          make_params(m, tau, kappa, 0.0, 1, 0, precision), precision_of(precision)};
    j.gsum = w->gsum;
    j.grad_src = grad_src;
    FAR_TRY(run_job(m, j, st, false, &one));
  }
  double g[14];
  FAR_TRY(fetch(st, g, w->gsum, sizeof(g)));
  for (int q = 0; q < 12; ++q) grad_T[q] = g[q];
  twist_from_grad(g, T, cc, grad_twist);
  if (cost) *cost = g[12];
  if (n_inliers) *n_inliers = int64_t(g[13]);
  return FAR_OK;
}

far_status_t far_gicp_gradient_batch(far_map_t m, const float* src, const int64_t* offsets,
                                     int32_t S_, int64_t n_total, const float* cov6,
                                     const uint8_t* valid, const double* T, const double* c,
                                     double tau, double kappa, int32_t precision,
                                     double* grad_T, double* grad_twist, float* grad_src,
                                     double* cost, int64_t* n_inliers, far_stream_t stream) {
  if (!m || !offsets || !T || !grad_T || !grad_twist || S_ < 1 || n_total < 0 ||
      n_total >= (int64_t(1) << 31) || !(tau > 0.0) || !(kappa > 0.0) ||
      (n_total > 0 && (!src || !cov6 || !valid)) ||
      !precision_ok(precision)) {
    set_error("far_gicp_gradient_batch: invalid argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  Scratch scr(st);
  far_align_stats_t* sts;
  double* gsum;
  FAR_TRY(scr.get(&sts, size_t(S_)));
  FAR_TRY(scr.get(&gsum, size_t(S_) * 14));
  TimedScope ts(FAR_TIME_GRADIENT, st);
  Job j{src, offsets, S_, n_total, cov6, valid, const_cast<double*>(T), sts, nullptr, nullptr,
        make_params(m, tau, kappa, 0.0, 1, 0, precision), precision_of(precision)};
  j.gsum = gsum;
  j.grad_src = grad_src;
  j.g_c = c;
  j.g_T = grad_T;
  j.g_tw = grad_twist;
  j.g_cost = cost;
  j.g_n = n_inliers;
  return run_job(m, j, st, false);
}

far_status_t far_gicp_align(far_map_t m, const float* src, const float* cov6,
                            const uint8_t* valid, int64_t n, const double T0[16],
                            const far_align_params_t* params, double T_out[16],
                            far_align_stats_t* stats, far_stream_t stream) {
  if (!m || !T0 || !T_out || !params_ok(params) || n < 0 || n >= (int64_t(1) << 31) ||
      (n > 0 && (!src || !cov6 || !valid))) {
    set_error("far_gicp_align: invalid argument");
    return FAR_E_INVALID;
  }
  far_align_stats_t hs;
  memset(&hs, 0, sizeof(hs));
  if (n == 0) {
    memcpy(T_out, T0, 16 * sizeof(double));
    hs.status = FAR_E_FEW_CORR;
    if (stats) *stats = hs;
    return FAR_E_FEW_CORR;
  }
  hipStream_t st = S(stream);
  AlignWS* w = nullptr;
  FAR_TRY(ensure_ws(m, 1, (n + kTileMin - 1) / kTileMin + 1, n, &w));
  const SingleArgs one = single_args(n, T0, kOrigin);
  Job j{src, w->offsets, 1, n, cov6, valid, w->T, w->stats, nullptr, nullptr,
        make_params(m, params->tau, params->kappa, params->eps, params->max_iters,
                    params->recenter, params->precision),
        precision_of(params->precision)};
  HostSlot slot;   // outlives the kernels that report to it: they end before the fetch
  j.slot = &slot;
  FAR_TRY(run_job(m, j, st, true, &one));
  FAR_TRY(fetch(st, T_out, w->T, 16 * sizeof(double), &hs, w->stats, sizeof(hs)));
  slot.busy = false;
  if (stats) *stats = hs;
  return far_status_t(hs.status);
}

far_status_t far_map_get_schedule(far_map_t m, far_schedule_t* out) {
  if (!m || !out) {
    set_error("far_map_get_schedule: null argument");
    return FAR_E_INVALID;
  }
  out->tile = m->sched_tile;
  out->fine_cells = m->sched_fine;
  return FAR_OK;
}

far_status_t far_map_set_schedule(far_map_t m, const far_schedule_t* sc) {
  if (!m || !sc || (sc->tile != 128 && sc->tile != 256 && sc->tile != 512) ||
      (sc->fine_cells != 0 && sc->fine_cells != 1)) {
    set_error("far_map_set_schedule: need tile 128, 256 or 512 and fine_cells 0 or 1");
    return FAR_E_INVALID;
  }
  m->sched_tile = sc->tile;
  m->sched_fine = sc->fine_cells;
  return FAR_OK;
}

static int32_t tiles_of(int c) { return c / 2 == 0 ? 128 : (c / 2 == 1 ? 256 : 512); }

far_status_t far_autotune(far_map_t m, const float* src, const int64_t* offsets, int32_t S_,
                          int64_t n_total, const float* cov6, const uint8_t* valid,
                          const double* T, const far_align_params_t* params, int32_t reps,
                          far_schedule_t* best, double* ms, far_stream_t stream) {
  if (!m || !offsets || !T || !best || !params_ok(params) || S_ < 1 || n_total < 0 ||
      n_total >= (int64_t(1) << 31) || reps < 1 || reps > 100 ||
      (n_total > 0 && (!src || !cov6 || !valid))) {
    set_error("far_autotune: invalid argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  const far_schedule_t saved{m->sched_tile, m->sched_fine};
  int e2 = 0;
  const bool pow2 = std::frexp(m->p.voxel_size, &e2) == 0.5;
  double* Tw = nullptr;
  far_align_stats_t* sw = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  far_status_t rs = FAR_OK;
  double times[6];
  far_schedule_t win = saved;
  double win_ms = -1.0;
  auto fail = [&](far_status_t s) {
    rs = s;
    return s;
  };
  do {
    hipError_t e;
    if ((e = hipMalloc(&Tw, size_t(S_) * 16 * sizeof(double))) != hipSuccess ||
        (e = hipMalloc(&sw, size_t(S_) * sizeof(far_align_stats_t))) != hipSuccess ||
        (e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess) {
      fail(hip_fail(e, "far_autotune setup", __FILE__, __LINE__));
      break;
    }
    const int32_t tiles[3] = {128, 256, 512};
    for (int c = 0; c < 6 && rs == FAR_OK; ++c) {
      times[c] = -1.0;
      const far_schedule_t cand{tiles[c / 2], c % 2};
      if (cand.fine_cells && !pow2) continue;
      m->sched_tile = cand.tile;
      m->sched_fine = cand.fine_cells;
      double bestc = 1e300;
      for (int r = 0; r <= reps && rs == FAR_OK; ++r) {
        if ((e = hipMemcpyAsync(Tw, T, size_t(S_) * 16 * sizeof(double),
                                hipMemcpyDeviceToDevice, st)) != hipSuccess ||
            (e = hipEventRecord(e0, st)) != hipSuccess) {
          fail(hip_fail(e, "far_autotune", __FILE__, __LINE__));
          break;
        }
        far_status_t a = far_gicp_align_batch(m, src, offsets, S_, n_total, cov6, valid, Tw,
                                              params, sw, stream);
        if (a != FAR_OK) {
          fail(a);
          break;
        }
        float t = 0.0f;
        if ((e = hipEventRecord(e1, st)) != hipSuccess ||
            (e = hipEventSynchronize(e1)) != hipSuccess ||
            (e = hipEventElapsedTime(&t, e0, e1)) != hipSuccess) {
          fail(hip_fail(e, "far_autotune timing", __FILE__, __LINE__));
          break;
        }
        if (r > 0 && t < bestc) bestc = t;   // run 0 is untimed (first launch, capture)
      }
      if (rs != FAR_OK) break;
      times[c] = bestc;
      if (win_ms < 0.0 || bestc < win_ms) {
        win_ms = bestc;
        win = cand;
      }
    }
  } while (false);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (Tw || sw) (void)hipStreamSynchronize(st);
  if (Tw) (void)hipFree(Tw);
  if (sw) (void)hipFree(sw);
  if (rs != FAR_OK) {
    m->sched_tile = saved.tile;
    m->sched_fine = saved.fine_cells;
    return rs;
  }
  // the schedule in place stays unless a candidate beats it by more than 2 %
  // (equivalent schedules would otherwise flip with timing noise)
  for (int c = 0; c < 6; ++c)
    if (tiles_of(c) == saved.tile && (c % 2) == saved.fine_cells && times[c] > 0.0 &&
        times[c] <= 1.02 * win_ms)
      win = saved;
  m->sched_tile = win.tile;
  m->sched_fine = win.fine_cells;
  *best = win;
  if (ms)
    for (int c = 0; c < 6; ++c) ms[c] = times[c];
  return FAR_OK;
}

static far_status_t align_batch_impl(far_map_t m, const float* src, const int64_t* offsets,
                                     int32_t S_, int64_t n_total, const float* cov6,
                                     const uint8_t* valid, const uint32_t* order, double* T,
                                     const far_align_params_t* params,
                                     far_align_stats_t* stats, far_stream_t stream,
                                     const char* who) {
  if (!m || !offsets || !T || !stats || !params_ok(params) || S_ < 1 || n_total < 0 ||
      n_total >= (int64_t(1) << 31) || (n_total > 0 && (!src || !cov6 || !valid))) {
    set_error("%s: invalid argument", who);
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  Job j{src, offsets, S_, n_total, cov6, valid, T, stats, nullptr, nullptr,
        make_params(m, params->tau, params->kappa, params->eps, params->max_iters,
                    params->recenter, params->precision),
        precision_of(params->precision)};
  j.order = order;
  return run_job(m, j, st, true);
}

far_status_t far_gicp_align_batch(far_map_t m, const float* src, const int64_t* offsets,
                                  int32_t S_, int64_t n_total, const float* cov6,
                                  const uint8_t* valid, double* T,
                                  const far_align_params_t* params, far_align_stats_t* stats,
                                  far_stream_t stream) {
  return align_batch_impl(m, src, offsets, S_, n_total, cov6, valid, nullptr, T, params, stats,
                          stream, "far_gicp_align_batch");
}

far_status_t far_gicp_align_batch_packed(far_map_t m, const void* packed,
                                         const int64_t* offsets, int32_t S_, int64_t n_total,
                                         double* T, const far_align_params_t* params,
                                         far_align_stats_t* stats, far_stream_t stream) {
  if (!m || !offsets || !T || !stats || !params_ok(params) || S_ < 1 || n_total < 0 ||
      n_total >= (int64_t(1) << 31) || (n_total > 0 && !packed) ||
      (reinterpret_cast<uintptr_t>(packed) & 15) != 0) {
    set_error("far_gicp_align_batch_packed: invalid argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  Job j{nullptr, offsets, S_, n_total, nullptr, nullptr, T, stats, nullptr, nullptr,
        make_params(m, params->tau, params->kappa, params->eps, params->max_iters,
                    params->recenter, params->precision),
        precision_of(params->precision)};
  const char* b = static_cast<const char*>(packed);
  j.in_A = reinterpret_cast<const float4*>(b);
  j.in_B = reinterpret_cast<const float4*>(b + 16 * n_total);
  j.in_C = reinterpret_cast<const float2*>(b + 32 * n_total);
  return run_job(m, j, st, true);
}

far_status_t far_gicp_align_batch_ordered(far_map_t m, const float* src,
                                          const int64_t* offsets, int32_t S_, int64_t n_total,
                                          const float* cov6, const uint8_t* valid,
                                          const uint32_t* order, double* T,
                                          const far_align_params_t* params,
                                          far_align_stats_t* stats, far_stream_t stream) {
  if (n_total > 0 && !order) {
    set_error("far_gicp_align_batch_ordered: invalid argument");
    return FAR_E_INVALID;
  }
  return align_batch_impl(m, src, offsets, S_, n_total, cov6, valid, order, T, params, stats,
                          stream, "far_gicp_align_batch_ordered");
}

}  // extern "C"
