// far_map.hip -- the voxel hash map (Sec. III-A.2 cuVoxelMap paragraph,
// Sec. III-A.3 Adaptive, Local Submap): create, capped insert with the
// covariances of the added points, k-nearest-neighbour query, export, stats,
// and the covariances of a scan against its own (uncapped) voxel grid.
//
// Layout in HBM (all fixed at create):
//   slots     Slot[S]            open addressing, linear probing step 1,
//                                S = 2^ceil(log2(2 * voxel_capacity))
//   vox_count int32[Vc]          points held per voxel
//   vox_key   uint64[Vc]         packed key per voxel
//   vox_pts   float4[Vc * Nmax]  voxel-major point store: x, y, z, id bits
//   cov       float4[Pc * 2]     per id: (xx, xy, xz, yy), (yz, zz, valid, 0)
//   pt_xyz    float[3][Pc]       per id coordinates (SoA)
//   pt_loc    int32[Pc]          per id slot in vox_pts
#include <cmath>
#include <cstdarg>
#include <cstring>
#include <mutex>
#include <type_traits>

#include <algorithm>

#include "far_knn.h"
#include "far_scan.h"

namespace far {

// ---------------------------------------------------------------- errors
static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

far_status_t hip_fail(hipError_t e, const char* what, const char* file, int line) {
  set_error("HIP error %d (%s) in %s at %s:%d", int(e), hipGetErrorString(e), what, file, line);
  return FAR_E_HIP;
}

int device_cu_count() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cus[dev]) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return 256;
    cus[dev] = prop.multiProcessorCount;
  }
  return cus[dev];
}

namespace {

constexpr int kT = 256;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

inline unsigned blocks_for(int64_t n, int per = kT) {
  int64_t b = (n + per - 1) / per;
  return unsigned(b < 1 ? 1 : b);
}

// A place in a list for every thread of the block that wants one: the list's
// count is raised once per block.  Every thread of the block calls it.
__device__ inline uint32_t block_reserve(bool want, uint32_t* count) {
  __shared__ uint32_t wcnt[kT / 64];
  __shared__ uint32_t base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t bal = __ballot(want);
  if (lane == 0) wcnt[wave] = uint32_t(__popcll(bal));
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (int w = 0; w < kT / 64; ++w) total += wcnt[w];
    base = total ? atomicAdd(count, total) : 0u;
  }
  __syncthreads();
  uint32_t at = base + uint32_t(__popcll(bal & ((uint64_t(1) << lane) - 1)));
  for (int w = 0; w < wave; ++w) at += wcnt[w];
  __syncthreads();   // the words are free for a next call
  return at;
}

// ---------------------------------------------------------------- keys
// Voxel key of every point (Sec. III-A.2: the key is the voxel's 3-D index).
// Non-finite points get the empty key (they sort last and are skipped);
// out-of-range points are counted and make the call fail.
__global__ __launch_bounds__(kT) void k_keys(const float* xyz, int64_t n, double v,
                                             uint64_t* keys, uint32_t* vals,
                                             uint32_t* counters) {
  int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i >= n) return;
  float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
  uint64_t key = kEmptyKey;
  if (isfinite(x) && isfinite(y) && isfinite(z)) {
    int64_t kx, ky, kz;
    if (voxel_index(double(x), v, &kx) && voxel_index(double(y), v, &ky) &&
        voxel_index(double(z), v, &kz))
      key = pack_key(kx, ky, kz);
    else
      atomicAdd(&counters[1], 1u);
  } else {
    atomicAdd(&counters[0], 1u);
  }
  keys[i] = key;
  vals[i] = uint32_t(i);
}

// ---------------------------------------------------------------- downsample
// The first point (in input order) of every voxel, through a hash of the
// scan's voxels instead of a sort by voxel: every point finds or claims its
// voxel's slot and lowers the smallest index held there, and the points that
// hold their slot's index are kept.  A raw scan of 90k points: 215 us of
// kernels for eight radix passes on 63-bit keys (52 launches), 26 us now (5
// launches).
// The table has at least two slots per point, cleared to 0xFF (no key, index
// 2^32 - 1).
// Of the lanes of a wave with the same voxel the first, which has the smallest
// index, claims for all, as far as that is worth a round of compares: the first
// lane left leads those with its voxel, until it leads no other.  (One claim a point
// serialised in scans of few voxels: 1M points in one voxel 2067 us, in ten 1024 and
// in thirty 485, now 127, 180 and 259.  Until it leads fewer than four: 127, 291 and
// 362; the sort took 334 to 362.)
__global__ __launch_bounds__(kT) void k_ds_claim(const float* xyz, int64_t n, double v,
                                                 Slot* slots, uint32_t mask, int log2_slots,
                                                 uint32_t* slot_of, uint32_t* oor) {
  const int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  const int lane = threadIdx.x & 63;
  bool has = false;
  int64_t kx = 0, ky = 0, kz = 0;
  if (i < n) {
    const float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
    if (isfinite(x) && isfinite(y) && isfinite(z)) {
      has = voxel_index(double(x), v, &kx) && voxel_index(double(y), v, &ky) &&
            voxel_index(double(z), v, &kz);
      if (!has) atomicAdd(oor, 1u);
    }
  }
  const uint64_t key = has ? pack_key(kx, ky, kz) : kEmptyKey;
  int lead = lane;
  uint64_t rest = __ballot(has);
  while (rest) {
    const int src = __builtin_ctzll(rest);
    const uint64_t k = uint64_t(__shfl((unsigned long long)key, src));
    const uint64_t same = __ballot(key == k);
    if (key == k) lead = src;
    rest &= ~same;
    if (!(same & (same - 1))) break;
  }
  uint32_t at = kNoSlot;
  if (has && lead == lane) {
    uint32_t h = voxel_hash(kx, ky, kz, log2_slots);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
      // the key first as a plain load (neighbouring points share voxels, so
      // most find theirs claimed; a stale empty word only costs the swap)
      unsigned long long old = *reinterpret_cast<const volatile unsigned long long*>(&slots[h].key);
      if (old == kEmptyKey)
        old = atomicCAS(reinterpret_cast<unsigned long long*>(&slots[h].key),
                        (unsigned long long)kEmptyKey, (unsigned long long)key);
      if (old == kEmptyKey || old == key) break;
      h = (h + 1) & mask;
    }
    at = h;
    // lower points mostly come first: look before lowering
    uint32_t* first = reinterpret_cast<uint32_t*>(&slots[h].vox);
    if (uint32_t(i) < *reinterpret_cast<const volatile uint32_t*>(first))
      atomicMin(first, uint32_t(i));
  }
  at = uint32_t(__shfl(int(at), lead));
  if (i < n) slot_of[i] = at;
}

// Compaction of the kept points in input order, SoA with row stride equal to
// their number; nothing is written when a point's key is out of range.
struct DownsampleFlags {
  const float* xyz;
  int64_t n;
  const Slot* slots;
  const uint32_t* slot_of;
  const uint32_t* oor;
  float* out;
  int32_t* keep;
  __device__ bool again(int64_t i) const {
    const uint32_t h = slot_of[i];
    return h != kNoSlot && uint32_t(slots[h].vox) == uint32_t(i);
  }
  __device__ bool first(int64_t i) const { return again(i); }
  __device__ void use(int64_t i, bool flag, uint32_t o, uint32_t all) const {
    if (!flag || *oor) return;
    out[o] = xyz[i];
    out[int64_t(all) + o] = xyz[n + i];
    out[2 * int64_t(all) + o] = xyz[2 * n + i];
    if (keep) keep[o] = int32_t(i);
  }
};

// ---------------------------------------------------------------- transform
struct Rigid {
  double r[12];  // rows of [R | t]
};

// out = R s + t per point, FP64 in the order ((R_r0 x + R_r1 y) + R_r2 z) + t_r
// (no contraction: the file is built with -ffp-contract=off), rounded to float.
// Every thread reads its point before writing it, so out may alias xyz.
__global__ __launch_bounds__(kT) void k_transform(const float* xyz, int64_t n, Rigid T,
                                                  float* out) {
  int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i >= n) return;
  double x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
  float o[3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
    o[r] = float(((T.r[4 * r] * x + T.r[4 * r + 1] * y) + T.r[4 * r + 2] * z) + T.r[4 * r + 3]);
  out[i] = o[0];
  out[n + i] = o[1];
  out[2 * n + i] = o[2];
}

// The cells of sorted points: keys of at least `empty` belong to the points
// without a voxel (non-finite), which sort last.
struct SortedKeys {
  const uint64_t* k;
  uint64_t empty;
  __device__ uint64_t cell(int64_t j) const { return k[j]; }
};

// Runs of equal cells of the sorted points: seg_start, seg_end per run.
struct RunFlags {
  SortedKeys keys;
  int64_t n;
  uint32_t* seg_start;
  uint32_t* seg_end;
  __device__ bool again(int64_t j) const {
    const uint64_t c = keys.cell(j);
    return c < keys.empty && (j == 0 || keys.cell(j - 1) != c);
  }
  __device__ bool first(int64_t j) const { return again(j); }
  __device__ void use(int64_t j, bool head, uint32_t pre, uint32_t) const {
    const uint64_t c = keys.cell(j);
    if (c >= keys.empty) return;
    const uint32_t s = pre + (head ? 1u : 0u) - 1u;
    if (head) seg_start[s] = uint32_t(j);
    if (j == n - 1 || keys.cell(j + 1) != c) seg_end[s] = uint32_t(j + 1);
  }
};

// What an insert's kernels hand on without a host wait in between.
struct InsertCounts {
  uint32_t n_seg;      // voxel runs of the batch
  uint32_t n_new;      // of them new voxels
  uint32_t n_acc;      // accepted points (the last of them may not fit)
  uint32_t n_cert;     // points whose certificates are rebuilt
  uint32_t ghosts;     // copy of the map's ghost count
  uint32_t leaves;     // (eviction) 1 when a point leaves
  uint32_t pad[2];
};

// The runs of an insert, or none when its new voxels do not fit: the batch is
// then refused as a whole and every later kernel does nothing.
__device__ inline int64_t insert_runs(const InsertCounts* c, int64_t vox_room) {
  return int64_t(c->n_new) <= vox_room ? int64_t(c->n_seg) : 0;
}

// Voxel of every run: looked up in the table, and the new ones numbered in
// sorted key order after the existing ones and claimed in the table.
struct NewVoxelFlags {
  MapView m;
  const float* xyz;
  int64_t n;
  double v;
  const uint32_t* vals;
  const uint32_t* seg_start;
  InsertCounts* counts;
  int64_t n_vox_old, vox_room;
  int32_t* seg_vox;
  uint32_t* is_new;
  Slot* slots;
  uint64_t* vox_key;
  int32_t* vox_slot;
  __device__ void key(int64_t s, int64_t* kx, int64_t* ky, int64_t* kz) const {
    const uint32_t i = vals[seg_start[s]];
    (void)voxel_index(double(xyz[i]), v, kx);         // held when the key was made
    (void)voxel_index(double(xyz[n + i]), v, ky);
    (void)voxel_index(double(xyz[2 * n + i]), v, kz);
  }
  __device__ bool first(int64_t s) const {
    if (s >= int64_t(counts->n_seg)) return false;
    int64_t kx = 0, ky = 0, kz = 0;
    key(s, &kx, &ky, &kz);
    int32_t c;
    const int32_t vox = map_find(m, kx, ky, kz, &c);
    seg_vox[s] = vox;
    return vox < 0;
  }
  __device__ bool again(int64_t s) const {
    return s < int64_t(counts->n_seg) && seg_vox[s] < 0;
  }
  __device__ void use(int64_t s, bool flag, uint32_t pre, uint32_t all) const {
    if (s >= int64_t(counts->n_seg)) return;
    is_new[s] = flag ? 1u : 0u;
    if (!flag || int64_t(all) > vox_room) return;
    int64_t kx = 0, ky = 0, kz = 0;
    key(s, &kx, &ky, &kz);
    const uint64_t k = pack_key(kx, ky, kz);
    const int32_t vox = int32_t(n_vox_old + pre);
    uint32_t h = voxel_hash(kx, ky, kz, m.log2_slots);
    for (uint32_t probe = 0; probe <= m.slot_mask; ++probe) {
      const unsigned long long old = atomicCAS(
          reinterpret_cast<unsigned long long*>(&slots[h].key), (unsigned long long)kEmptyKey,
          (unsigned long long)k);
      if (old == kEmptyKey) {
        slots[h].vox = vox;
        slots[h].aux = 0;
        vox_slot[vox] = int32_t(h);
        break;
      }
      h = (h + 1) & m.slot_mask;
    }
    seg_vox[s] = vox;
    vox_key[vox] = k;
  }
};

// Sequential capped insert of one voxel's candidates in input order (runs are
// stable-sorted so candidates appear in input order).  A candidate is accepted
// while the voxel holds fewer than its cap and, with spacing on, it is at least
// dmin from every point already there.  Accepted points are appended to the
// voxel's store right away, so later candidates of the same run are checked
// against them.
//
// kGreedyLanes lanes per run: the order is serial, but the candidates are
// loaded a chunk at a time, one per lane, and each is tested against all of
// the voxel's points at once, which the lanes hold in registers (point q in
// lane q mod kGreedyLanes; at most 64 points a voxel).  One lane per run,
// with two dependent loads per candidate and one per test: 25 us for 15k
// candidates and 57 us for 500k; 7.5 and 37 us now.
constexpr int kGreedyLanes = 16;
constexpr int kGreedyHold = 64 / kGreedyLanes;

__global__ __launch_bounds__(kT) void k_greedy(const float* xyz, int64_t n,
                                               const int32_t* caps, int32_t nmax,
                                               double dmin2, const uint32_t* vals,
                                               const uint32_t* seg_start,
                                               const uint32_t* seg_end,
                                               const InsertCounts* counts, int64_t vox_room,
                                               const int32_t* seg_vox,
                                               const int32_t* vox_count, float4* vox_pts,
                                               uint32_t* acc_flag, int32_t* acc_pos,
                                               int32_t* seg_newcount) {
  constexpr int G = kGreedyLanes;
  const int l = threadIdx.x & (G - 1);
  const int shift = threadIdx.x & 63 & ~(G - 1);   // the group's first lane in its wave
  const int64_t n_seg = insert_runs(counts, vox_room);
  const int64_t step = int64_t(gridDim.x) * (kT / G);
  for (int64_t s = (int64_t(blockIdx.x) * kT + threadIdx.x) / G; s < n_seg; s += step) {
    const int32_t vox = seg_vox[s];
    int32_t cnt = vox_count[vox];
    float4* store = vox_pts + int64_t(vox) * nmax;
    const uint32_t j0 = seg_start[s], j1 = seg_end[s];
    float hx[kGreedyHold], hy[kGreedyHold], hz[kGreedyHold];
#pragma unroll
    for (int u = 0; u < kGreedyHold; ++u) {
      const int q = u * G + l;
      const float4 p = q < cnt ? store[q] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      hx[u] = p.x;
      hy[u] = p.y;
      hz[u] = p.z;
    }
    for (uint32_t j = j0; j < j1 && cnt < nmax; j += G) {
      // this lane's candidate of the chunk
      const bool have = j + l < j1;
      const uint32_t i = vals[have ? j + l : j];
      const float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
      const int32_t cap = caps ? min(caps[i], nmax) : nmax;
      int32_t pos = -1;
      const int m = int(min(uint32_t(G), j1 - j));
      for (int c = 0; c < m; ++c) {
        const int32_t ccap = __shfl(cap, c, G);
        if (cnt >= ccap) continue;   // the same in every lane of the group
        const float cx = __shfl(x, c, G), cy = __shfl(y, c, G), cz = __shfl(z, c, G);
        bool near = false;
        if (dmin2 > 0.0) {
#pragma unroll
          for (int u = 0; u < kGreedyHold; ++u)
            if (u * G + l < cnt)
              near |= dist2(double(cx), double(cy), double(cz), double(hx[u]), double(hy[u]),
                            double(hz[u])) < dmin2;
        }
        // the group's lanes of the ballot (lanes of other groups that are at
        // another point of their loops read as 0)
        if ((__ballot(near) >> shift) & ((uint64_t(1) << G) - 1)) continue;
#pragma unroll
        for (int u = 0; u < kGreedyHold; ++u)
          if (u * G + l == cnt) {
            hx[u] = cx;
            hy[u] = cy;
            hz[u] = cz;
          }
        if (l == c) pos = cnt;
        ++cnt;
      }
      if (pos >= 0) {
        store[pos] = make_float4(x, y, z, __int_as_float(-1));
        acc_flag[i] = 1u;
        acc_pos[i] = int32_t(int64_t(vox) * nmax + pos);
      }
    }
    if (l == 0) seg_newcount[s] = cnt;
  }
}

// Accepted points get their ids (input order) and are recorded by id; those
// past the point capacity are dropped.  id_local is kept for the counts of a
// truncated batch.
struct CommitFlags {
  const float* xyz;
  int64_t n;
  const uint32_t* acc_flag;
  const int32_t* acc_pos;
  uint32_t* id_local;
  int64_t id0, point_cap;
  float4* vox_pts;
  float* pt_xyz;
  int32_t* pt_loc;
  __device__ bool first(int64_t i) const { return acc_flag[i] != 0; }
  __device__ bool again(int64_t i) const { return acc_flag[i] != 0; }
  __device__ void use(int64_t i, bool flag, uint32_t pre, uint32_t) const {
    if (!flag) return;
    id_local[i] = pre;
    const int64_t id = id0 + pre;
    if (id >= point_cap) return;
    const int32_t pos = acc_pos[i];
    vox_pts[pos].w = __int_as_float(int32_t(id));
    pt_xyz[id] = xyz[i];
    pt_xyz[point_cap + id] = xyz[n + i];
    pt_xyz[2 * point_cap + id] = xyz[2 * n + i];
    pt_loc[id] = pos;
  }
};

// New per-voxel counts.  When the point capacity truncated the batch, only
// the accepted prefix whose ids fit is kept.
__global__ __launch_bounds__(kT) void k_counts(const InsertCounts* counts, int64_t vox_room,
                                               int64_t room, const int32_t* seg_vox,
                                               const int32_t* seg_newcount,
                                               const uint32_t* vals, const uint32_t* seg_start,
                                               const uint32_t* seg_end,
                                               const uint32_t* acc_flag,
                                               const uint32_t* id_local,
                                               int32_t* vox_count, const int32_t* vox_slot,
                                               Slot* slots, uint32_t* seg_changed) {
  const int64_t n_seg = insert_runs(counts, vox_room);
  const bool truncated = int64_t(counts->n_acc) > room;
  for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < n_seg;
       s += int64_t(gridDim.x) * kT) {
    const int32_t vox = seg_vox[s];
    int32_t c = seg_newcount[s];
    const int32_t old = vox_count[vox];
    if (truncated) {
      c = old;
      for (uint32_t j = seg_start[s]; j < seg_end[s]; ++j) {
        const uint32_t i = vals[j];
        if (acc_flag[i] && int64_t(id_local[i]) < room) ++c;
      }
    }
    vox_count[vox] = c;
    slots[vox_slot[vox]].aux = c;
    seg_changed[s] = c != old ? 1u : 0u;
  }
}

// ---------------------------------------------------------------- certificates
// The vox_pts slots of the marked voxels' points (of all voxels when mark is
// null), appended to list in voxel order within a block of voxels: the
// certificates below then run one point per lane.  (One lane per slot left
// 84 % of the lanes of a wave idle on a surface map of 3.3 points per voxel of
// 20 slots.)
__global__ __launch_bounds__(kT) void k_cert_list(int64_t n_vox, int32_t nmax,
                                                  const int32_t* vox_count, const uint32_t* mark,
                                                  uint32_t gen, uint32_t* list, uint32_t* count) {
  __shared__ uint32_t wsum[kT / 64];
  __shared__ uint32_t base;
  const int64_t V = int64_t(blockIdx.x) * kT + threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t c = V < n_vox && (!mark || mark[V] == gen) ? uint32_t(vox_count[V]) : 0u;
  uint32_t x = c;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = uint32_t(__shfl_up(int(x), d));
    if (lane >= d) x += u;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t at = x - c, total = 0;
#pragma unroll
  for (int w = 0; w < kT / 64; ++w) {
    at += w < wave ? wsum[w] : 0u;
    total += wsum[w];
  }
  if (total == 0) return;
  if (threadIdx.x == 0) base = atomicAdd(count, total);
  __syncthreads();
  at += base;
  for (uint32_t q = 0; q < c; ++q) list[at + q] = uint32_t(V * nmax + q);
}

// The certificate of the point p at pos from its K nearest (see k_cert_build),
// and its covariance when cov is given and its id is at least id0.
template <int K>
__device__ inline void cert_write(const MapView& m, uint32_t pos, const float4& p,
                                  const TopK<K>& top, CertRow* cert, float4* cov,
                                  float4* vox_cov, int64_t id0, int32_t k, int32_t reg) {
  // the row straight to memory (an array of its entries, indexed by a count,
  // would live in scratch)
  float4* out = reinterpret_cast<float4*>(cert + pos);
  int c = 0;
  double next = -1.0;
#pragma unroll
  for (int u = 0; u < kCertK + 2; ++u) {
    if (top.pos[u] < 0 || top.pos[u] == int32_t(pos)) continue;
    if (c < kCertK) {
      const float4 q = m.vox_pts[top.pos[u]];
      out[++c] = make_float4(q.x, q.y, q.z, __int_as_float(top.pos[u]));
    } else if (next < 0.0) {
      next = top.d[u];
    }
  }
  while (c < kCertK) out[++c] = make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
  const double half = 0.5 * (next >= 0.0 ? sqrt(next) : m.v) * (1.0 - 0x1p-20);
  out[0] = make_float4(p.x, p.y, p.z, __double2float_rd(half));
  const int32_t id = __float_as_int(p.w);
  if (!cov || id < id0) return;
  double c6[6] = {0, 0, 0, 0, 0, 0};
  const bool ok = top.found() >= k;
  if (ok) regularised_cov<K>(top, k, [&](int32_t at) { return m.vox_pts[at]; }, c6, reg);
  const float4 a = make_float4(float(c6[0]), float(c6[1]), float(c6[2]), float(c6[3]));
  const float4 b = make_float4(float(c6[4]), float(c6[5]), ok ? 1.0f : 0.0f, 0.0f);
  cov[2 * int64_t(id)] = a;
  cov[2 * int64_t(id) + 1] = b;
  vox_cov[2 * int64_t(pos)] = a;
  vox_cov[2 * int64_t(pos) + 1] = b;
}

// Certificate of every listed point, one lane each: the kCertK + 1 nearest
// other points within v by (d2, id) from the exact 27-voxel search (the point
// itself, and so kCertK + 2 entries, included), the first kCertK listed with
// their coordinates, rho half the distance of the next one (v/2 when there is
// none), shrunk by 2^-20 and rounded down to float so that it never exceeds
// the exact half distance.  With cov given, the points with ids from id0 on
// (those an insert adds, all of them listed) get their covariance from the
// k <= K nearest of the same search, into the record by id and by slot: the
// search they would otherwise repeat.
//
// Bound by the latency of the gathers and by FP64 ranking.  The neighbours
// come from the voxel's row of the neighbour table (in LDS, read in one go)
// instead of a hash probe each.  On average over two inserts of 500k points
// into an emptied map: 782 us for one lane per slot with probes and 188 us for the separate
// covariance search, now 152 us in all (300 with the row as an indexed local array and 222
// registers; 194 with the certificate's row and the covariance written in the
// loop, which spilled more).
constexpr int kCertWaves = 4;   // waves per SIMD asked for (128 registers)

template <int K>
__global__ __launch_bounds__(kT, kCertWaves) void k_cert_build(MapView m, const uint32_t* list,
                                                   const uint32_t* count, CertRow* cert,
                                                   float4* cov, float4* vox_cov, int64_t id0,
                                                   int32_t k, int32_t reg) {
  static_assert(K >= kCertK + 2, "a certificate needs kCertK + 2 entries");
  __shared__ uint32_t rows[kT * kRowWords];
  uint32_t* row = rows + threadIdx.x * kRowWords;
  const uint32_t n = *count;
  for (uint32_t t = blockIdx.x * kT + threadIdx.x; t < n; t += gridDim.x * kT) {
    const uint32_t pos = list[t];
    const int32_t V = int32_t(pos / uint32_t(m.nmax));
    const float4 p = m.vox_pts[pos];
    load_row(m.vox_nbr + int64_t(V) * 26, row);
    TopK<K> top;
    top.init();
    int64_t kx = 0, ky = 0, kz = 0;   // in range: held when the point was inserted
    (void)voxel_index(double(p.x), m.v, &kx);
    (void)voxel_index(double(p.y), m.v, &ky);
    (void)voxel_index(double(p.z), m.v, &kz);
    map_knn_row<K>(m, double(p.x), double(p.y), double(p.z), int32_t(kx), int32_t(ky),
                   int32_t(kz), V * m.nmax, m.vox_count[V], row, m.v * m.v, top);
    cert_write<K>(m, pos, p, top, cert, cov, vox_cov, id0, k, reg);
  }
}

// The same for the short list of a small insert or map, four lanes per point:
// one lane each would leave the chip at a wave per SIMD, as long as its chain of
// voxels and of FP64 insertions.  First the lanes share the points of the own
// voxel and merge their lists; then each takes every fourth of the voxels that
// the merged K-th best can still reach (the first lane on from the merged list,
// the others from its K-th entry without a place), and the lists are merged
// again.  The list is the K best by (d2, id) of the same candidates, so the
// certificates are the same.
// Where the line lies: it pays by the points of a voxel.  In a street driven
// along (30k to 60k listed, up to 20 points a voxel) an insert took 77 us by one
// lane and 51 by four, the same points after an eviction 58 and 33; in a
// sparse map (2 points a voxel) 20000 added points 16.5 and 16.7, 30000 21 and
// 28, 64000 34 and 53.
constexpr int64_t kCertQuadMax = 48 * 1024;
template <int K>
__global__ __launch_bounds__(kT, 3) void k_cert_build_quad(MapView m, const uint32_t* list,
                                                           const uint32_t* count, CertRow* cert,
                                                           float4* cov, float4* vox_cov,
                                                           int64_t id0, int32_t k, int32_t reg) {
  static_assert(K >= kCertK + 2, "a certificate needs kCertK + 2 entries");
  constexpr int kPts = kT / 4;
  __shared__ uint32_t rows[kPts * kRowWords];
  __shared__ int32_t s_pos[kPts][K];
  __shared__ double s_d[kPts][K];
  const int lane = threadIdx.x & 3, q4 = threadIdx.x >> 2;
  uint32_t* row = rows + q4 * kRowWords;
  const uint32_t n = *count;
  for (uint32_t t0 = blockIdx.x * kPts; t0 < n; t0 += gridDim.x * kPts) {
    const uint32_t t = t0 + uint32_t(q4);
    if (t < n) {   // (a quad as a whole)
      const uint32_t pos = list[t];
      const int32_t V = int32_t(pos / uint32_t(m.nmax));
      const float4 p = m.vox_pts[pos];
      const uint2* nb = reinterpret_cast<const uint2*>(m.vox_nbr + int64_t(V) * 26);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (lane + 4 * u < 13) {
          const uint2 e = nb[lane + 4 * u];
          row[2 * (lane + 4 * u)] = e.x;
          row[2 * (lane + 4 * u) + 1] = e.y;
        }
      const double px = p.x, py = p.y, pz = p.z, r2 = m.v * m.v;
      int64_t kx = 0, ky = 0, kz = 0;   // in range: held when the point was inserted
      (void)voxel_index(px, m.v, &kx);
      (void)voxel_index(py, m.v, &ky);
      (void)voxel_index(pz, m.v, &kz);
      TopK<K> own, top;
      own.init();
      const int32_t base = V * m.nmax, cnt = m.vox_count[V];
      for (int32_t j = lane; j < cnt; j += 16) {
        float4 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j + 4 * u < cnt) c[u] = m.vox_pts[base + j + 4 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j + 4 * u < cnt) {
            const double d = dist2(double(c[u].x), double(c[u].y), double(c[u].z), px, py, pz);
            if (d <= r2) own.push(d, __float_as_int(c[u].w), base + j + 4 * u);
          }
      }
      merge_lists<4>(own, top);
      // (the row was written by this wave's lanes, in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      Query q = make_query(px, py, pz, r2);
      FaceOffsets fo;
      fo.f[0] = float(px - double(kx) * m.v);
      fo.f[1] = float(py - double(ky) * m.v);
      fo.f[2] = float(pz - double(kz) * m.v);
      fo.v = float(m.v);
      fo.slack = float(1e-7 * m.v);
      const double bound = fmin(r2, top.bound());
      uint32_t need = 0;
      {
        const float bnd = f32_up(bound);
#pragma unroll
        for (int rank = 1; rank < 27; ++rank) {
          const int code = nbr_code(rank);
          if (row[nbr_dir(code)] != kNbrNone && fo.lb2(code) <= bnd) need |= 1u << rank;
        }
      }
#pragma unroll
      for (int s = 0; s < K; ++s) {
        own.d[s] = lane == 0 ? top.d[s] : top.d[K - 1];
        own.id[s] = lane == 0 ? top.id[s] : top.id[K - 1];
        own.pos[s] = lane == 0 ? top.pos[s] : -1;
      }
      q.bound_f = screen_bound(bound, q.m);
      for (int u = 0; u < lane; ++u) need &= need - 1;
      while (need) {
        const int code = nbr_code(__builtin_ctz(need));
        need &= need - 1;
        need &= need - 1;
        need &= need - 1;
        need &= need - 1;
        if (double(fo.lb2(code)) > fmin(r2, own.bound())) continue;
        const uint32_t e = row[nbr_dir(code)];
        scan_voxel_points<K>(m.vox_pts, int32_t(e >> kNbrCountBits) * m.nmax,
                             int32_t(e & ((1u << kNbrCountBits) - 1u)), q, r2, own);
      }
      merge_lists<4>(own, top);
      if (lane == 0) {
#pragma unroll
        for (int s = 0; s < K; ++s) {
          s_pos[q4][s] = top.pos[s];
          s_d[q4][s] = top.d[s];
        }
      }
    }
    __syncthreads();
    // the rows and covariances by one lane per point, all in the first wave
    if (threadIdx.x < kPts && t0 + threadIdx.x < n) {
      TopK<K> top;
#pragma unroll
      for (int s = 0; s < K; ++s) {
        top.pos[s] = s_pos[threadIdx.x][s];
        top.d[s] = s_d[threadIdx.x][s];
        top.id[s] = 0;
      }
      const uint32_t pos = list[t0 + threadIdx.x];
      cert_write<K>(m, pos, m.vox_pts[pos], top, cert, cov, vox_cov, id0, k, reg);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- links
// Ghost voxels are the empty voxels next to an occupied one.  Each has a
// neighbour-table row, so that a search from a point in an empty voxel reads
// its occupied neighbours from one row instead of probing the hash for each
// of the 26; a point whose voxel is neither occupied nor a ghost has no map
// point in its 27 voxels.  Ghosts are claimed around every new voxel, their
// rows filled from the hash, and the rows of the ghosts around every voxel
// whose count changed are updated with its new entry.  A ghost whose key
// later becomes occupied keeps its slot; the occupied voxel shadows it.
//
// The kernels take the 26 neighbours of a voxel with one thread per (voxel,
// direction): each neighbour is a chain of dependent loads (a hash probe, a
// row, a store), so one thread taking the 26 in turn was bound by that latency
// with most of the chip idle (an insert of 15k points touches about 4k voxels:
// 60 waves).
__device__ inline int dir_code(int dir) { return dir < 13 ? dir : dir + 1; }

// After the counts of an insert's voxel runs (or all voxels of a rebuilt map):
//  - neighbour rows: the entry (index and count) of every touched voxel goes
//    into the row of every existing neighbour, and a new voxel's own row is
//    filled from the hash.  The neighbours of a voxel that was there before
//    are in its row already; those that are new put their entry there and
//    take its entry from the hash themselves, so only new voxels probe.
//  - marks: a voxel that gained points marks itself and its neighbours with
//    this insert's generation, because the certificates of the points within
//    v of an added point, all of which lie in its 27 voxels, are rebuilt (a
//    new neighbour that its row does not show yet marks itself).
//  - ghosts: the empty neighbours of a new voxel are claimed (index from
//    gcount; beyond ghost_cap a ghost gets no row and the host switches the
//    ghosts off), and the ghosts there before get the entry of a voxel whose
//    count changed; new ghosts' rows are filled later.  The table has two slots
//    per ghost of the capacity, where chains are a few dozen slots at most; a claim
//    that finds no place in kGhostProbes means more ghosts than that and raises
//    gcount beyond ghost_cap.  (Unbounded, the 26 ghosts each of 20000 voxels 4 m
//    apart, in a map of just that capacity, filled the table, and every further
//    claim walked all of it: 3.9 s.)
// An entry is written only by the threads of the voxel it names and of the
// voxel whose row it is, with the same (final) value, so the writes need no
// ordering.  As one launch per voxel these four passes took 120 us for an
// insert of 15k points and 607 us for one of 500k (0.1M voxels); 12 and 172 us
// in this one.
constexpr uint32_t kGhostProbes = 1024;   // (the smallest table)

__global__ __launch_bounds__(kT) void k_links(MapView m, const InsertCounts* counts,
                                              int64_t vox_room, const int32_t* seg_vox,
                                              const uint32_t* is_new, const uint32_t* seg_changed,
                                              const uint64_t* vox_key, uint32_t* vox_nbr,
                                              uint32_t* mark, uint32_t gen, Slot* gslots,
                                              uint64_t* gkey, uint32_t* gcount,
                                              int64_t ghost_cap) {
  const int64_t total = insert_runs(counts, vox_room) * 26;
  for (int64_t t0 = int64_t(blockIdx.x) * kT; t0 < total; t0 += int64_t(gridDim.x) * kT) {
    const int64_t t = t0 + threadIdx.x;
    bool won = false, full = false;
    uint32_t h = 0;
    uint64_t nk = 0;
    if (t < total) {
      const int64_t s = t / 26;
      const int dir = int(t - s * 26), code = dir_code(dir);
      const int32_t V = seg_vox[s];
      const bool fresh = !is_new || is_new[s] != 0;
      const bool changed = seg_changed && seg_changed[s] != 0;
      const uint64_t key = vox_key[V];
      const int64_t nx = key_x(key) + code / 9 - 1, ny = key_y(key) + (code / 3) % 3 - 1,
                    nz = key_z(key) + code % 3 - 1;
      const uint32_t eV = (uint32_t(V) << kNbrCountBits) | uint32_t(m.vox_count[V]);
      int32_t N = -1;
      if (fresh) {
        int32_t cN;
        N = map_find(m, nx, ny, nz, &cN);
        vox_nbr[int64_t(V) * 26 + dir] =
            N >= 0 ? (uint32_t(N) << kNbrCountBits) | uint32_t(cN) : kNbrNone;
      } else {
        const uint32_t e = vox_nbr[int64_t(V) * 26 + dir];
        if (e != kNbrNone) N = int32_t(e >> kNbrCountBits);
      }
      if (changed && dir == 0) mark[V] = gen;
      if (N >= 0) {
        vox_nbr[int64_t(N) * 26 + nbr_dir(26 - code)] = eV;
        if (changed) mark[N] = gen;
      } else if (m.ghost_ok && (fresh || changed) && key_ok(nx) && key_ok(ny) && key_ok(nz)) {
        nk = pack_key(nx, ny, nz);
        h = voxel_hash(nx, ny, nz, m.glog2);
        full = true;
        for (uint32_t probe = 0; probe < kGhostProbes; ++probe) {
          // (most are claimed already: look before a swap)
          unsigned long long old =
              *reinterpret_cast<const volatile unsigned long long*>(&gslots[h].key);
          if (old == kEmptyKey && fresh)
            old = atomicCAS(reinterpret_cast<unsigned long long*>(&gslots[h].key),
                            (unsigned long long)kEmptyKey, (unsigned long long)nk);
          if (old == kEmptyKey) {
            won = fresh;
            full = false;
            break;
          }
          if (old == nk) {
            full = false;
            // a ghost there before; one claimed in this launch (its index not
            // yet written, or beyond those known before it) is filled later
            const int32_t g = *reinterpret_cast<const volatile int32_t*>(&gslots[h].vox);
            if (g >= 0)
              const_cast<uint32_t*>(m.gnbr)[int64_t(g) * 26 + nbr_dir(26 - code)] = eV;
            break;
          }
          if ((probe & 31u) == 31u &&
              int64_t(*reinterpret_cast<const volatile uint32_t*>(gcount)) > ghost_cap)
            break;   // known by now
          h = (h + 1) & m.gmask;
        }
      }
    }
    // one atomic per block on the shared count (they serialise, 6 to 7 ns each)
    const uint32_t g = block_reserve(won, gcount);
    if (full) atomicMax(gcount, uint32_t(ghost_cap) + 1u);
    if (won) {
      gslots[h].vox = int64_t(g) < ghost_cap ? int32_t(g) : -1;
      if (int64_t(g) < ghost_cap) gkey[g] = nk;
    }
  }
}

// Neighbour rows of the ghosts with index in [g0, min(*gcount, cap)): a grid
// of any size takes the (ghost, direction) entries in turn.  *count_out
// receives the ghost count for the host.
__global__ __launch_bounds__(kT) void k_ghost_fill(MapView m, const uint64_t* gkey,
                                                   const uint32_t* gcount, int64_t g0,
                                                   int64_t ghost_cap, uint32_t* gnbr,
                                                   uint32_t* count_out) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *count_out = *gcount;
  const int64_t end = (int64_t(*gcount) < ghost_cap ? int64_t(*gcount) : ghost_cap) * 26;
  for (int64_t t = g0 * 26 + int64_t(blockIdx.x) * kT + threadIdx.x; t < end;
       t += int64_t(gridDim.x) * kT) {
    const int64_t g = t / 26;
    const int code = dir_code(int(t - g * 26));
    const uint64_t key = gkey[g];
    int32_t c;
    const int32_t N = map_find(m, key_x(key) + code / 9 - 1, key_y(key) + (code / 3) % 3 - 1,
                               key_z(key) + code % 3 - 1, &c);
    gnbr[t] = N >= 0 ? (uint32_t(N) << kNbrCountBits) | uint32_t(c) : kNbrNone;
  }
}

// ---------------------------------------------------------------- ASMD
// Near-range points of the scan (sensor range <= r_near) and the distinct
// map-frame voxels they fall in, counted through a temporary hash set of
// keys (counters: [0] near points, [1] distinct voxels, [2] out of range).
__global__ __launch_bounds__(kT) void k_asmd_count(const float* xs, const float* xm, int64_t n,
                                                   double v, double rn2, uint64_t* set,
                                                   uint32_t set_mask, int set_log2,
                                                   uint32_t* counters) {
  const int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  bool near = false, first = false;
  if (i < n) {
    const double sx = xs[i], sy = xs[n + i], sz = xs[2 * n + i];
    const double mx = xm[i], my = xm[n + i], mz = xm[2 * n + i];
    near = isfinite(sx) && isfinite(sy) && isfinite(sz) && isfinite(mx) && isfinite(my) &&
           isfinite(mz) && (sx * sx + sy * sy) + sz * sz <= rn2;
    if (near) {
      int64_t kx, ky, kz;
      if (!voxel_index(mx, v, &kx) || !voxel_index(my, v, &ky) || !voxel_index(mz, v, &kz)) {
        atomicAdd(&counters[2], 1u);
        near = false;
      } else {
        const uint64_t key = pack_key(kx, ky, kz);
        uint32_t h = voxel_hash(kx, ky, kz, set_log2);
        for (uint32_t probe = 0; probe <= set_mask; ++probe) {
          const unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(&set[h]),
                                                   (unsigned long long)kEmptyKey,
                                                   (unsigned long long)key);
          first = old == kEmptyKey;
          if (first || old == key) break;
          h = (h + 1) & set_mask;
        }
      }
    }
  }
  (void)block_reserve(near, &counters[0]);   // one add per block and count
  (void)block_reserve(first, &counters[1]);
}

// cap_i = clamp(floor(mean (1 - r_i / r_max) + 0.5), k, nmax), FP64 in this
// order (no contraction); non-finite points get k.  mean = near points /
// distinct near voxels from k_asmd_count's counters (nmax when none).
__global__ __launch_bounds__(kT) void k_asmd_caps(const float* xs, int64_t n,
                                                  const uint32_t* counters, double r_max,
                                                  int32_t k, int32_t nmax, int32_t* caps) {
  const int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i >= n) return;
  const double mean =
      counters[1] > 0 ? double(counters[0]) / double(counters[1]) : double(nmax);
  const double sx = xs[i], sy = xs[n + i], sz = xs[2 * n + i];
  int32_t cap = k;
  if (isfinite(sx) && isfinite(sy) && isfinite(sz)) {
    const double r = sqrt((sx * sx + sy * sy) + sz * sz);
    const double c = floor(mean * (1.0 - r / r_max) + 0.5);
    cap = c < double(k) ? k : (c > double(nmax) ? nmax : int32_t(c));
  }
  caps[i] = cap;
}

// ---------------------------------------------------------------- eviction
// Every surviving point keeps its place among its voxel's points and every
// surviving voxel its place among the voxels, so the rebuild needs no sort:
// two prefix sums (voxels, points) give the new indices.  (The radix sort of
// the survivors by voxel, eight passes on 63-bit keys, was half the time of a
// rebuild.)

// Keep flag of every voxel: it holds points and its centre lies within the
// radius of c; a voxel with points beyond it raises *leaves.  The kept voxels, in
// voxel order, go into compact keys and counts.
struct EvictVoxels {
  const uint64_t* vox_key;
  const int32_t* vox_count;
  double v, cx, cy, cz, r2;
  uint32_t* vkeep;
  uint32_t* nvox;
  uint64_t* key_out;
  int32_t* count_out;
  uint32_t* leaves;
  __device__ bool first(int64_t V) const {
    const uint64_t key = vox_key[V];
    const double dx = (double(key_x(key)) + 0.5) * v - cx;
    const double dy = (double(key_y(key)) + 0.5) * v - cy;
    const double dz = (double(key_z(key)) + 0.5) * v - cz;
    const bool held = vox_count[V] > 0, in = (dx * dx + dy * dy) + dz * dz <= r2;
    vkeep[V] = held && in ? 1u : 0u;
    if (held && !in && *leaves == 0u) *leaves = 1u;   // (the same word by all)
    return held && in;
  }
  __device__ bool again(int64_t V) const { return *leaves && vkeep[V] != 0; }
  __device__ void use(int64_t V, bool flag, uint32_t pre, uint32_t) const {
    if (!flag) return;
    nvox[V] = pre;
    key_out[pre] = vox_key[V];
    count_out[pre] = vox_count[V];
  }
};

// Keep flag of every map point: its voxel's.  The survivors, in id order, go
// into compact SoA coordinates (row stride their number), covariances and new
// slots.  When no point leaves, every flag is set and nothing is read or written
// per point (a call that evicts nothing, as most of an odometry's: on 3M points in
// 1.9M voxels 159 us with the survivors copied all the same).
struct EvictPoints {
  const float* pt_xyz;
  const float4* cov;
  const int32_t* pt_loc;
  int64_t point_cap;
  int32_t nmax;
  const uint32_t* vkeep;
  const uint32_t* nvox;
  float* xyz_out;
  float4* cov_out;
  int32_t* loc_out;
  const uint32_t* leaves;
  __device__ bool again(int64_t i) const {
    return !*leaves || vkeep[uint32_t(pt_loc[i]) / uint32_t(nmax)] != 0;
  }
  __device__ bool first(int64_t i) const { return again(i); }
  __device__ void use(int64_t i, bool flag, uint32_t j, uint32_t all) const {
    if (!flag || !*leaves) return;
    xyz_out[j] = pt_xyz[i];
    xyz_out[int64_t(all) + j] = pt_xyz[point_cap + i];
    xyz_out[2 * int64_t(all) + j] = pt_xyz[2 * point_cap + i];
    cov_out[2 * int64_t(j)] = cov[2 * i];
    cov_out[2 * int64_t(j) + 1] = cov[2 * i + 1];
    const uint32_t loc = uint32_t(pt_loc[i]), V = loc / uint32_t(nmax);
    loc_out[j] = int32_t(nvox[V] * uint32_t(nmax) + (loc - V * uint32_t(nmax)));
  }
};

// Empty hash slots of the voxels and the ghosts, zero counts.  (As four memsets,
// evicting all of a small map took 77 us, with the flag passes before them more than
// by the sort; 44 us now.)
__global__ __launch_bounds__(kT) void k_clear_voxels(Slot* slots, int64_t n_slots, Slot* gslots,
                                                     int64_t n_gslots, int32_t* vox_count,
                                                     int64_t n_vox, uint32_t* gcount) {
  const uint4 e = make_uint4(~0u, ~0u, ~0u, ~0u);
  const int64_t t = int64_t(blockIdx.x) * kT + threadIdx.x, step = int64_t(gridDim.x) * kT;
#pragma unroll 4
  for (int64_t i = t; i < n_slots; i += step) reinterpret_cast<uint4*>(slots)[i] = e;
#pragma unroll 4
  for (int64_t i = t; i < n_gslots; i += step) reinterpret_cast<uint4*>(gslots)[i] = e;
  for (int64_t i = t; i < n_vox; i += step) vox_count[i] = 0;
  if (t == 0) *gcount = 0u;
}

// The rebuilt map: every survivor at its new slot and id, every kept voxel
// (they come first in the same grid) with its key, count and hash slot; all
// voxels are listed as runs for the neighbour rows.
__global__ __launch_bounds__(kT) void k_evict_store(const float* xyz, const float4* cov_in,
                                                    const int32_t* loc, int64_t n,
                                                    int64_t point_cap, const uint64_t* key_in,
                                                    const int32_t* count_in, int64_t n_vox,
                                                    float* pt_xyz, float4* cov, int32_t* pt_loc,
                                                    float4* vox_pts, float4* vox_cov, Slot* slots,
                                                    uint32_t slot_mask, int log2_slots,
                                                    uint64_t* vox_key, int32_t* vox_count,
                                                    int32_t* vox_slot, int32_t* seg_vox) {
  const int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i < n_vox) {
    const uint64_t key = key_in[i];
    vox_key[i] = key;
    vox_count[i] = count_in[i];
    seg_vox[i] = int32_t(i);
    uint32_t h = voxel_hash(key_x(key), key_y(key), key_z(key), log2_slots);
    for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
      if (atomicCAS(reinterpret_cast<unsigned long long*>(&slots[h].key),
                    (unsigned long long)kEmptyKey, (unsigned long long)key) == kEmptyKey) {
        slots[h].vox = int32_t(i);
        slots[h].aux = count_in[i];
        vox_slot[i] = int32_t(h);
        break;
      }
      h = (h + 1) & slot_mask;
    }
  }
  if (i >= n) return;
  const float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
  pt_xyz[i] = x;
  pt_xyz[point_cap + i] = y;
  pt_xyz[2 * point_cap + i] = z;
  const int32_t pos = loc[i];
  pt_loc[i] = pos;
  vox_pts[pos] = make_float4(x, y, z, __int_as_float(int32_t(i)));
  const float4 a = cov_in[2 * i], b = cov_in[2 * i + 1];
  cov[2 * i] = a;
  cov[2 * i + 1] = b;
  vox_cov[2 * int64_t(pos)] = a;
  vox_cov[2 * int64_t(pos) + 1] = b;
}

// Covariances of the *n_acc added map points from id0 on (below point_cap): k
// nearest within v on the map, into the records by id and by vox_pts slot.
template <int K>
__global__ __launch_bounds__(kT) void k_map_cov(MapView m, float4* cov, float4* vox_cov,
                                                const int32_t* pt_loc, int64_t id0,
                                                const uint32_t* n_acc, int32_t k, int32_t reg) {
  const int64_t id1 = min(id0 + int64_t(*n_acc), m.point_cap);
  for (int64_t id = id0 + int64_t(blockIdx.x) * kT + threadIdx.x; id < id1;
       id += int64_t(gridDim.x) * kT) {
    const double qx = m.pt_xyz[id], qy = m.pt_xyz[m.point_cap + id],
                 qz = m.pt_xyz[2 * m.point_cap + id];
    TopK<K> top;
    map_knn_query<K>(m, qx, qy, qz, m.v * m.v, top);
    double c6[6] = {0, 0, 0, 0, 0, 0};
    const bool ok = top.found() >= k;
    if (ok) regularised_cov<K>(top, k, [&](int32_t pos) { return m.vox_pts[pos]; }, c6, reg);
    const float4 a = make_float4(float(c6[0]), float(c6[1]), float(c6[2]), float(c6[3]));
    const float4 b = make_float4(float(c6[4]), float(c6[5]), ok ? 1.0f : 0.0f, 0.0f);
    const int64_t pos = pt_loc[id];
    cov[2 * id] = a;
    cov[2 * id + 1] = b;
    vox_cov[2 * pos] = a;
    vox_cov[2 * pos + 1] = b;
  }
}

// Bound by the latency of each lane's chain of voxels.  The neighbours come
// from the query's voxel's row of the neighbour table, or its ghost's (an empty
// voxel that is neither has nothing within v), read in one go; a hash probe
// per neighbour took 124 us for 100k queries at k = 5, 62 us now.  One wave a block,
// so that a few thousand queries spread over the chip: 4000 at k = 5 and 32 63 and 223 us
// in blocks of four waves (87 and 326 by probes), 55 and 182 so; at k = 32, with its
// spilled registers, 4166 queries on a thin map had become slower (127 -> 135, now 114).
// From 30k queries on it makes no difference.
constexpr int kKnnThreads = 64;
template <int K>
__global__ __launch_bounds__(kKnnThreads) void k_map_knn(MapView m, const float* q, int64_t n,
                                                         int32_t k, double r2, int32_t* idx,
                                                         float* d2, int32_t* count) {
  __shared__ uint32_t rows[kKnnThreads * kRowWords];
  uint32_t* lrow = rows + threadIdx.x * kRowWords;
  int64_t i = int64_t(blockIdx.x) * kKnnThreads + threadIdx.x;
  if (i >= n) return;
  float x = q[i], y = q[n + i], z = q[2 * n + i];
  TopK<K> top;
  top.init();
  int64_t kx, ky, kz;
  if (isfinite(x) && isfinite(y) && isfinite(z) && voxel_index(double(x), m.v, &kx) &&
      voxel_index(double(y), m.v, &ky) && voxel_index(double(z), m.v, &kz)) {
    int32_t cnt;
    const int32_t own = map_find(m, kx, ky, kz, &cnt);
    const int32_t g = own < 0 && m.ghost_ok ? ghost_find(m, kx, ky, kz) : -1;
    const uint32_t* row = own >= 0 ? m.vox_nbr + int64_t(own) * 26
                                   : (g >= 0 ? m.gnbr + int64_t(g) * 26 : nullptr);
    if (row) {
      load_row(row, lrow);
      map_knn_row<K>(m, double(x), double(y), double(z), int32_t(kx), int32_t(ky), int32_t(kz),
                     own >= 0 ? own * m.nmax : 0, cnt, lrow, r2, top);
    } else if (!m.ghost_ok) {
      map_knn_query<K>(m, double(x), double(y), double(z), r2, top);
    }
  }
  int f = top.found();
  int c = f < k ? f : k;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    if (s < k) {
      idx[i * k + s] = s < c ? top.id[s] : -1;
      if (d2) d2[i * k + s] = s < c ? float(top.d[s]) : -1.0f;
    }
  }
  if (count) count[i] = c;
}

// ---------------------------------------------------------------- scan grid
// Each scan's own voxel grid is CSR: the points of all scans sorted by (scan,
// voxel key) (sorted[j] = x, y, z, original index bits), runs [run_start,
// run_end) of equal (scan, key), and a hash table from (scan, key) to a run's
// start and length (a scan's cells are hashed into its own stretch of slots).
constexpr uint32_t kNoRun = 0xFFFFFFFFu;

struct GridView {
  const Slot* slots;
  const float4* sorted;
  double v;          // neighbourhood radius (the voxel edge)
  double c;          // grid cell edge (v / 2 when v is a power of two, else v)
  double inv_c;
  int32_t pow2;
  const int64_t* part;        // scan offsets: the slots of each scan (NULL: one scan)
  uint32_t n_slots;           // two per point
  double mx;         // runs sorted by x up to a quantum: how far a later point of
                     // a run can lie below an earlier one along x (infinity:
                     // runs unordered)
  // The runs, numbered inside eight ranges of sorted positions, one per XCD:
  // the runs that start in range x are x * run_chunk up to x * run_chunk +
  // n_runs[16 x] (in no particular order), so that an XCD works through the
  // cells of its own scans.
  int64_t run_chunk;
  const uint32_t* n_runs;
  const uint64_t* run_key;
  const uint32_t* run_sid;    // (NULL: one scan)
  const uint32_t* run_start;
  const uint32_t* run_end;
  uint32_t* run_id;           // per sorted point, its run (kNoRun: a non-finite point)
  const uint2* nbt;           // per run, its 27 cells (code (ox+1)*9 + (oy+1)*3 + oz+1) as
                              // (start, count) in sorted; count 0: no run there
  float4* pk_B;               // the source packed for the align by sorted position
  float2* pk_C;               // (B, C as the align's pack writes them), or null
};

// The align's packed covariance words of sorted point j: B = (xx, or -1 when
// invalid, xy, xz, yy), C = (yz, zz), from the values written to cov6.
__device__ inline void write_packed(const GridView& g, int64_t j, const float c[6], bool ok) {
  if (!g.pk_B) return;
  g.pk_B[j] = make_float4(ok ? c[0] : -1.0f, c[1], c[2], c[3]);
  g.pk_C[j] = make_float2(c[4], c[5]);
}

// Slots of scan sc: two per point of the scan (its points are positions
// offsets[sc] .. offsets[sc + 1] of the sorted order, so at most half of its
// slots fill), or the whole table for a single scan.  Each scan's cells are
// hashed into its own stretch, so that the lookups of one scan, which the
// sorted order brings together, stay in a few MB of the table (one XCD's L2).
__device__ inline void grid_part(const GridView& g, uint32_t sc, uint32_t* base,
                                 uint32_t* size) {
  if (g.part) {
    const int64_t a = g.part[sc], b = g.part[sc + 1];
    *base = uint32_t(2 * a);
    *size = uint32_t(2 * (b - a));
  } else {
    *base = 0;
    *size = g.n_slots;
  }
}

__device__ inline uint32_t grid_hash(int64_t kx, int64_t ky, int64_t kz, uint32_t size) {
  const uint32_t h = (uint32_t(kx) * 73856093u) ^ (uint32_t(ky) * 19349669u) ^
                     (uint32_t(kz) * 83492791u);
  const uint32_t m = uint32_t((uint64_t(h) * 0x9E3779B97F4A7C15ull) >> 32);
  return uint32_t((uint64_t(m) * size) >> 32);
}

// Run of cell (kx, ky, kz) of scan sid: its start in sorted (or -1) and in
// *cnt its length.  A slot holds the cell's key, the run's start and its
// length (the scan is implied by the stretch of slots).
__device__ inline int32_t grid_find(const GridView& g, int64_t kx, int64_t ky, int64_t kz,
                                    uint32_t sid, int32_t* cnt) {
  *cnt = 0;
  if (!key_ok(kx) || !key_ok(ky) || !key_ok(kz)) return -1;
  const uint64_t key = pack_key(kx, ky, kz);
  uint32_t base, size;
  grid_part(g, sid, &base, &size);
  uint32_t s = grid_hash(kx, ky, kz, size);
  for (uint32_t probe = 0; probe < size; ++probe) {
    const Slot sl = load_slot(&g.slots[base + s]);
    if (sl.key == key) {
      *cnt = sl.aux;
      return sl.vox;
    }
    if (sl.key == kEmptyKey) return -1;
    s = s + 1 == size ? 0 : s + 1;
  }
  return -1;
}

// Scan id of each key-sorted point (binary search of its original index in
// the scan offsets); the result is the key of a second, stable sort.
__global__ __launch_bounds__(kT) void k_scan_ids(const uint32_t* vals, int64_t n,
                                                 const int64_t* offsets, int32_t S,
                                                 uint64_t* sid_key, uint32_t* pos) {
  int64_t j = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (j >= n) return;
  int64_t i = vals[j];
  int32_t lo = 0, hi = S;            // find s with offsets[s] <= i < offsets[s+1]
  while (hi - lo > 1) {
    int32_t mid = (lo + hi) >> 1;
    if (offsets[mid] <= i) lo = mid; else hi = mid;
  }
  sid_key[j] = uint64_t(lo);
  pos[j] = uint32_t(j);
}

__global__ __launch_bounds__(kT) void k_apply_perm(const uint32_t* perm, int64_t n,
                                                   const uint64_t* keys_in,
                                                   const uint32_t* vals_in, uint64_t* keys_out,
                                                   uint32_t* vals_out, const uint64_t* sid_key,
                                                   uint32_t* sid_out) {
  int64_t m = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (m >= n) return;
  uint32_t j = perm[m];
  keys_out[m] = keys_in[j];
  vals_out[m] = vals_in[j];
  sid_out[m] = uint32_t(sid_key[m]);
}

// ---------------------------------------------------------------- compact grid keys
// A batch's scan grid sorts its points by (scan, voxel key).  Keys limited to
// the batch's own range per axis need few bits (a sensor-frame scan of 120 m
// range at v = 1: 8 per axis), so one radix sort of (scan, kx - min, ky - min,
// kz - min) replaces a 63-bit sort followed by a sort by scan: the same
// order (both are lexicographic, stable on input order), in about half the
// passes.  The range comes from one launch, whose blocks raise seven shared words
// by an atomic each; points without a finite, in-range key sort last in their scan.
constexpr int kRangeBlocks = 1024;

// floor(x / v) as voxel_index computes it, through an exact multiply by 1/v
// when v is a power of two.
__device__ inline bool voxel_index_p2(double x, double v, double inv_v, bool pow2, int64_t* k) {
  const double f = floor(pow2 ? x * inv_v : x / v);
  if (!(f >= -double(kKeyBias) && f < double(kKeyBias))) return false;
  *k = int64_t(f);
  return true;
}

// Scan s of point i: offsets[s] <= i < offsets[s + 1].
__device__ inline int32_t scan_of(const int64_t* offsets, int32_t S, int64_t i) {
  int32_t lo = 0, hi = S;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (offsets[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// How crowded a batch's scans are, by one block: kCrowdSample of its points (drawn by a
// hash, with repeats) are counted by (scan, cell) in a table in LDS, and out receives
// the sum over them of the others drawn in their cell.  Times n / kCrowdSample^2 that
// is the mean number of points in a point's own cell, up to the draw (36 of 28k
// points a cell: within 3 %) and to cells that share a word of the table (n /
// kCrowdCells, taken off by the caller).
constexpr int kCrowdSample = 1024, kCrowdLog2 = 13, kCrowdCells = 1 << kCrowdLog2;

__device__ inline void count_crowd(const float* xyz, int64_t n, double v, double inv_v,
                                   int32_t pow2, const int64_t* offsets, int32_t S,
                                   uint32_t* out) {
  constexpr int kPer = kCrowdSample / kT;
  constexpr uint64_t kMix = 0x9E3779B97F4A7C15ull;
  __shared__ uint4 cnt4[kCrowdCells / 4];
  uint32_t* cnt = reinterpret_cast<uint32_t*>(cnt4);
  float p[kPer][3];
  int32_t sid[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    uint64_t x = uint64_t(u * kT + int(threadIdx.x) + 1) * kMix;
    x = (x ^ (x >> 29)) * kMix;
    const int64_t i = int64_t(((x >> 32) * uint64_t(n)) >> 32);   // n < 2^31
    p[u][0] = xyz[i];
    p[u][1] = xyz[n + i];
    p[u][2] = xyz[2 * n + i];
    sid[u] = offsets ? scan_of(offsets, S, i) : 0;
  }
#pragma unroll
  for (int c = 0; c < kCrowdCells / 4 / kT; ++c)   // (while the loads are in flight)
    cnt4[c * kT + threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  int32_t at[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    int64_t kx, ky, kz;
    at[u] = -1;
    if (!isfinite(p[u][0]) || !isfinite(p[u][1]) || !isfinite(p[u][2]) ||
        !voxel_index_p2(double(p[u][0]), v, inv_v, pow2, &kx) ||
        !voxel_index_p2(double(p[u][1]), v, inv_v, pow2, &ky) ||
        !voxel_index_p2(double(p[u][2]), v, inv_v, pow2, &kz))
      continue;
    at[u] = int32_t((voxel_hash(kx, ky, kz, kCrowdLog2) + uint32_t(sid[u]) * 0x9E3779B1u) &
                    uint32_t(kCrowdCells - 1));
    atomicAdd(&cnt[at[u]], 1u);
  }
  __syncthreads();
  uint32_t others = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) others += at[u] >= 0 ? cnt[at[u]] - 1u : 0u;
  others = block_total(others);
  if (threadIdx.x == 0) *out = others;
}

// Key ranges of the finite points, kRangeBlocks blocks at most: out[a] the
// minimum of axis a as 2^21 - (key + 2^20), out[3 + a] the maximum as key +
// 2^20 + 1 (both raised from 0 by one atomic per block and axis), out[6] the
// number of out-of-range points.  out starts as zeros.  (Per-block results
// reduced by a second launch cost 5 us more on a scan of 100k points.)
// kCrowd: the last block counts the crowd into out[7] instead.
template <bool kCrowd>
__global__ __launch_bounds__(kT) void k_key_range(const float* xyz, int64_t n, double v,
                                                  double inv_v, int32_t pow2,
                                                  const int64_t* offsets, int32_t S,
                                                  uint32_t* out) {
  if constexpr (kCrowd) {
    if (blockIdx.x == gridDim.x - 1) {
      count_crowd(xyz, n, v, inv_v, pow2, offsets, S, out + 7);
      return;
    }
  }
  __shared__ int32_t s_r[kT / 64][6];
  __shared__ uint32_t s_o[kT / 64];
  int32_t r[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN};
  uint32_t oor = 0;
  const int64_t step = int64_t(gridDim.x - (kCrowd ? 1 : 0)) * kT;
  for (int64_t i0 = int64_t(blockIdx.x) * kT + threadIdx.x; i0 < n; i0 += 4 * step) {
    float p[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u) {   // four points' loads in flight
      const int64_t i = min(i0 + u * step, n - 1);
      p[u][0] = xyz[i];
      p[u][1] = xyz[n + i];
      p[u][2] = xyz[2 * n + i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (i0 + u * step >= n) continue;
      const float x = p[u][0], y = p[u][1], z = p[u][2];
      if (!(isfinite(x) && isfinite(y) && isfinite(z))) continue;
      int64_t kx, ky, kz;
      if (voxel_index_p2(double(x), v, inv_v, pow2, &kx) &&
          voxel_index_p2(double(y), v, inv_v, pow2, &ky) &&
          voxel_index_p2(double(z), v, inv_v, pow2, &kz)) {
        r[0] = min(r[0], int32_t(kx)); r[3] = max(r[3], int32_t(kx));
        r[1] = min(r[1], int32_t(ky)); r[4] = max(r[4], int32_t(ky));
        r[2] = min(r[2], int32_t(kz)); r[5] = max(r[5], int32_t(kz));
      } else {
        ++oor;
      }
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    for (int a = 0; a < 3; ++a) {
      r[a] = min(r[a], __shfl_xor(r[a], d));
      r[3 + a] = max(r[3 + a], __shfl_xor(r[3 + a], d));
    }
    oor += uint32_t(__shfl_xor(int(oor), d));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    for (int a = 0; a < 6; ++a) s_r[w][a] = r[a];
    s_o[w] = oor;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    int32_t x = s_r[0][threadIdx.x];
    for (int q = 1; q < kT / 64; ++q)
      x = threadIdx.x < 3 ? min(x, s_r[q][threadIdx.x]) : max(x, s_r[q][threadIdx.x]);
    if (threadIdx.x < 3 ? x != INT_MAX : x != INT_MIN)
      atomicMax(&out[threadIdx.x], threadIdx.x < 3 ? uint32_t(kKeyBias - x)
                                                   : uint32_t(x + kKeyBias + 1));
  }
  if (threadIdx.x == 6) {
    uint32_t o = 0;
    for (int q = 0; q < kT / 64; ++q) o += s_o[q];
    if (o) atomicAdd(&out[6], o);
  }
}

// Compact cell key: the cell's offsets from the batch's per-axis minima,
// bx, by, bz bits (each at least 2), laid out as 4 x 4 x 4 blocks of cells -
// the block's offsets (bx-2, by-2, bz-2 bits, x major) above the cell's place
// in the block (2 + 2 + 2 bits, x major) - so that sorted points fill whole
// blocks in turn: a stretch of the order is a compact patch of space.
struct CompactKey {
  int32_t mx, my, mz;   // per-axis minimum
  int32_t bx, by, bz;   // bits of x, y and z (>= 2)
  int32_t kb;           // key bits (x, y, z); 1 << kb marks an empty key
  int32_t fb;           // bits of the point's x within its cell, below the key
};

__device__ inline uint64_t compact_cell(const CompactKey& ck, int64_t cx, int64_t cy,
                                        int64_t cz) {
  const uint64_t hi = (uint64_t(cx >> 2) << (ck.by + ck.bz - 4)) |
                      (uint64_t(cy >> 2) << (ck.bz - 2)) | uint64_t(cz >> 2);
  return (hi << 6) | (uint64_t(cx & 3) << 4) | (uint64_t(cy & 3) << 2) | uint64_t(cz & 3);
}

__global__ __launch_bounds__(kT) void k_keys_compact(const float* xyz, int64_t n, double v,
                                                     double inv_v, int32_t pow2,
                                                     const int64_t* offsets, int32_t S,
                                                     CompactKey ck, uint64_t* keys,
                                                     uint32_t* vals, uint32_t* zero,
                                                     Slot* slots) {
  const int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i >= n) return;
  if (zero) zero[i] = 0u;
  if (slots) {   // the scan grid's two slots per point, empty
    const uint4 e = make_uint4(~0u, ~0u, ~0u, ~0u);
    reinterpret_cast<uint4*>(slots)[2 * i] = e;
    reinterpret_cast<uint4*>(slots)[2 * i + 1] = e;
  }
  const int32_t s = offsets ? scan_of(offsets, S, i) : 0;
  uint64_t key = uint64_t(1) << (ck.kb + ck.fb);
  const float x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
  int64_t kx, ky, kz;
  if (isfinite(x) && isfinite(y) && isfinite(z) &&
      voxel_index_p2(double(x), v, inv_v, pow2, &kx) &&
      voxel_index_p2(double(y), v, inv_v, pow2, &ky) &&
      voxel_index_p2(double(z), v, inv_v, pow2, &kz)) {
    // x / v less its floor is exact and non-decreasing in x within a cell,
    // so the fb bits below the key sort each run by x up to 2^-fb cells
    const double t = pow2 ? double(x) * inv_v : double(x) / v;
    const uint64_t xq = uint64_t(fmin((t - floor(t)) * ldexp(1.0, ck.fb), ldexp(1.0, ck.fb) - 1.0));
    key = (compact_cell(ck, kx - ck.mx, ky - ck.my, kz - ck.mz) << ck.fb) | xq;
  }
  keys[i] = (uint64_t(s) << (ck.kb + ck.fb + 1)) | key;
  vals[i] = uint32_t(i);
}

// The sorted keys of a scan grid: compact ones, or full keys beside scan ids.
struct GridKeys {
  const uint64_t* k;
  const uint32_t* sid;   // full keys of several scans
  int32_t compact, multi;
  CompactKey ck;
  __device__ bool same(int64_t a, int64_t b) const {
    if (compact) return k[a] >> ck.fb == k[b] >> ck.fb;
    return k[a] == k[b] && (!sid || sid[a] == sid[b]);
  }
  __device__ bool empty(int64_t j) const {
    return compact ? ((k[j] >> (ck.fb + ck.kb)) & 1u) != 0 : k[j] == kEmptyKey;
  }
  __device__ uint32_t scan(int64_t j) const {
    if (!multi) return 0u;
    return compact ? uint32_t(k[j] >> (ck.fb + ck.kb + 1)) : sid[j];
  }
  __device__ uint64_t key(int64_t j) const {
    if (!compact) return k[j];
    const uint64_t c = (k[j] >> ck.fb) & ((uint64_t(1) << ck.kb) - 1);
    const uint64_t hi = c >> 6;
    const int64_t hx = int64_t(hi >> (ck.by + ck.bz - 4));
    const int64_t hy = int64_t((hi >> (ck.bz - 2)) & ((uint64_t(1) << (ck.by - 2)) - 1));
    const int64_t hz = int64_t(hi & ((uint64_t(1) << (ck.bz - 2)) - 1));
    return pack_key(((hx << 2) | int64_t((c >> 4) & 3)) + ck.mx,
                    ((hy << 2) | int64_t((c >> 2) & 3)) + ck.my,
                    ((hz << 2) | int64_t(c & 3)) + ck.mz);
  }
};

// From the sorted keys to the grid in one launch (blocks dealt to the XCDs in
// contiguous ranges; a scan's points stay in the scan's index range, so each
// XCD gathers from, and claims in, the few MB of its own scans): the sorted
// points as float4 (and, when order is not null, the sorted order itself), the
// runs of equal (scan, cell), and each run's slot in its scan's stretch of the
// hash.  A run's end is the next change of cell: in the block's ballots, or,
// for a run that leaves the block, by doubling steps past it.  (As key
// expansion, heads, prefix sum, bounds, gather, clearing and claim: ten
// launches, 28 us at 5k points and 250 us at 4.9M; 9 and 161 us.)
template <int kPer>
__global__ __launch_bounds__(kT) void k_grid_runs(GridView g, GridKeys gk, const float* xyz,
                                                  int64_t n, const uint32_t* vals, Slot* slots,
                                                  float4* sorted, uint32_t* order,
                                                  uint32_t* n_runs, uint64_t* run_key,
                                                  uint32_t* run_sid, uint32_t* run_start,
                                                  uint32_t* run_end) {
  constexpr int kWords = kPer * kT / 64;
  __shared__ uint64_t starts[kWords];
  __shared__ uint32_t heads[kWords];
  __shared__ uint32_t base;
  const int64_t nb = (n + kT * kPer - 1) / (kT * kPer), chunk = (nb + 7) >> 3;
  const int x = int(blockIdx.x & 7);
  const int64_t b = x * chunk + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= chunk || b >= nb) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j0 = b * (kT * kPer), j1 = min(j0 + int64_t(kT) * kPer, n);
  uint64_t hb[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const int64_t j = j0 + r * kT + threadIdx.x;
    const bool st = j < n && (j == 0 || !gk.same(j, j - 1));
    const bool hd = st && !gk.empty(j);
    const uint64_t sb = __ballot(st);
    hb[r] = __ballot(hd);
    if (lane == 0) {
      starts[r * 4 + wave] = sb;
      heads[r * 4 + wave] = uint32_t(__popcll(hb[r]));
    }
    if (j < n) {
      const uint32_t i = vals[j];
      sorted[j] = make_float4(xyz[i], xyz[n + i], xyz[2 * n + i], __int_as_float(int32_t(i)));
      if (order) order[j] = i;
      if (gk.empty(j)) g.run_id[j] = kNoRun;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (int w = 0; w < kWords; ++w) total += heads[w];
    base = uint32_t(x * g.run_chunk) + (total ? atomicAdd(&n_runs[16 * x], total) : 0u);
  }
  __syncthreads();
  uint32_t before = base;
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    uint32_t id = before;
    for (int w = 0; w < 4; ++w) {
      id += w < wave ? heads[r * 4 + w] : 0u;
      before += heads[r * 4 + w];
    }
    if (!((hb[r] >> lane) & 1u)) continue;
    id += uint32_t(__popcll(hb[r] & ((uint64_t(1) << lane) - 1)));
    const int64_t j = j0 + r * kT + threadIdx.x;
    // the next start in the block's ballots
    int w = r * 4 + wave;
    uint64_t m = lane == 63 ? 0ull : starts[w] & (~0ull << (lane + 1));
    while (!m && ++w < kWords) m = starts[w];
    int64_t e = m ? j0 + w * 64 + __builtin_ctzll(m) : j1;
    if (!m && j1 < n && gk.same(j, j1)) {
      int64_t ok = j1, step = 1;             // ok: in the run
      while (ok + step < n && gk.same(j, ok + step)) {
        ok += step;
        step <<= 1;
      }
      for (; step >= 1; step >>= 1)
        if (ok + step < n && gk.same(j, ok + step)) ok += step;
      e = ok + 1;
    }
    const uint64_t key = gk.key(j);
    const uint32_t sc = gk.scan(j), cnt = uint32_t(e - j);
    run_start[id] = uint32_t(j);
    run_end[id] = uint32_t(e);
    run_key[id] = key;
    if (run_sid) run_sid[id] = sc;
    uint32_t sb, size;
    grid_part(g, sc, &sb, &size);
    uint32_t h = grid_hash(key_x(key), key_y(key), key_z(key), size);
    // every run is a different cell, so a slot is claimed on its length word
    // alone (a 32-bit compare-and-swap; a length is at least 1, never the empty
    // word); key and start follow as plain stores, read only by later kernels
    for (uint32_t probe = 0; probe < size; ++probe) {
      const uint32_t old = atomicCAS(reinterpret_cast<uint32_t*>(&slots[sb + h].aux),
                                     0xFFFFFFFFu, cnt);
      if (old == 0xFFFFFFFFu) {
        slots[sb + h].key = key;
        slots[sb + h].vox = int32_t(j);
        break;
      }
      h = h + 1 == size ? 0 : h + 1;
    }
  }
}

// Persistent grids over the runs: at most kGridBlocks blocks, a multiple of 8,
// each taking the items of its XCD's range of runs in turn.
constexpr int kGridBlocks = 8 * 1024;
inline unsigned grid_blocks(int64_t items) {
  const int64_t nb = ((items + kT - 1) / kT + 7) / 8 * 8;
  return unsigned(std::min<int64_t>(nb < 8 ? 8 : nb, kGridBlocks));
}

// Neighbour table of the runs: per run, the (start, count) of the run of the
// same scan in each of its 27 cells, so that a point's search reads its
// cells from its run's row instead of probing the hash for each.  One thread
// per (run, cell) entry t, the entries in XCD ranges (one XCD probes one
// scan's stretch of slots at a time); the rows are written with non-temporal
// stores so that they stream past the L2 holding the slots.
constexpr uint32_t kLongRun = 1024;
__device__ inline void grid_nbr_entry(const GridView& g, uint2* nbt, uint32_t r, int code) {
  const uint32_t s0 = g.run_start[r], s1 = g.run_end[r];
  uint32_t a = s0, c = s1 - s0;
  if (code != 13) {
    const uint64_t key = g.run_key[r];
    const uint32_t sc = g.run_sid ? g.run_sid[r] : 0u;
    int32_t cnt;
    const int32_t f = grid_find(g, key_x(key) + code / 9 - 1, key_y(key) + (code / 3) % 3 - 1,
                                key_z(key) + code % 3 - 1, sc, &cnt);
    a = f < 0 ? 0u : uint32_t(f);
    c = f < 0 ? 0u : uint32_t(cnt);
  }
  const int64_t t = int64_t(r) * 27 + code;
  __builtin_nontemporal_store(a, &nbt[t].x);
  __builtin_nontemporal_store(c, &nbt[t].y);
  // the run's points learn their run: the 27 threads of its row in turn or, of a long
  // run, the wave's lanes together, four points a store (27 threads took 170 us for a
  // run of 200k points and 580 us for one of 600k)
  const bool alone = s1 - s0 > kLongRun;
  if (!alone)
    for (uint32_t j = s0 + uint32_t(code); j < s1; j += 27) g.run_id[j] = r;
  uint64_t rest = __ballot(alone && code == 13);
  if (!rest) return;
  const uint64_t here = __ballot(true);
  const uint32_t lanes = uint32_t(__popcll(here));
  const uint32_t me = uint32_t(__popcll(here & ((uint64_t(1) << (threadIdx.x & 63)) - 1)));
  for (; rest; rest &= rest - 1) {
    const int src = __builtin_ctzll(rest);
    const uint32_t id = uint32_t(__shfl(int(r), src)), a = uint32_t(__shfl(int(s0), src)),
                   b = uint32_t(__shfl(int(s1), src));
    const uint32_t a4 = (a + 3) >> 2, b4 = b >> 2;   // whole groups of four
#pragma unroll 8
    for (uint32_t q = a4 + me; q < b4; q += lanes)
      reinterpret_cast<uint4*>(g.run_id)[q] = make_uint4(id, id, id, id);
    for (uint32_t j = a + me; j < 4 * a4; j += lanes) g.run_id[j] = id;
    for (uint32_t j = 4 * b4 + me; j < b; j += lanes) g.run_id[j] = id;
  }
}

__global__ __launch_bounds__(kT) void k_grid_nbr_table(GridView g, uint2* nbt) {
  const int x = int(blockIdx.x & 7);
  const int64_t total = int64_t(g.n_runs[16 * x]) * 27, step = int64_t(gridDim.x >> 3) * kT;
  for (int64_t t = int64_t(blockIdx.x >> 3) * kT + threadIdx.x; t < total; t += step) {
    const int64_t q = t / 27;
    grid_nbr_entry(g, nbt, uint32_t(x * g.run_chunk + q), int(t - q * 27));
  }
}

// Squared face distance as a float never above the FP64 value (rounded
// down, shrunk by 2^-20 to cover the float sums of three terms).
__device__ inline float face_lb(double g) { return __double2float_rd(g * g) * (1.0f - 0x1p-20f); }

// Covariances, one wave per grid run (the points of one scan in one voxel of
// edge v).  All of a run's queries share one 27-voxel neighbourhood (every
// point within v of them lies in it), so the wave reads the run's row of the
// neighbour table once and walks each needed voxel's points at wave-uniform
// addresses, every lane testing the same candidate against its own query; a
// voxel that no lane's current k-th distance can reach is skipped.  Exact,
// like the per-point search: ranking by (d2, id) over a superset of the
// candidates.  Only runs of at least `dense` points are taken: in sparse runs
// most lanes would idle while the wave walks the neighbourhood.
template <int K>
__device__ inline void grid_cov_run(const GridView& g, int64_t sg, int32_t dense, int64_t n,
                                    int32_t k, int32_t reg, float* cov6, uint8_t* valid,
                                    int32_t* nb_start, int32_t* nb_cnt) {
  const int lane = threadIdx.x;
  __syncthreads();   // the previous run's readers of nb_start and nb_cnt are done
  const uint32_t s0 = g.run_start[sg], s1 = g.run_end[sg];
  if (int64_t(s1 - s0) < dense) return;   // sparse runs: the per-point search
  const uint64_t key = g.run_key[sg];
  const int64_t kx = key_x(key), ky = key_y(key), kz = key_z(key);
  if (lane < 27) {   // the run's row of the neighbour table
    const uint2 e = g.nbt[sg * 27 + lane];
    nb_start[lane] = e.y ? int32_t(e.x) : -1;
    nb_cnt[lane] = int32_t(e.y);
  }
  __syncthreads();
  const double v = g.v, r2 = v * v, slack = 1e-7 * v;
  const double bx = double(kx) * v, by = double(ky) * v, bz = double(kz) * v;
  for (uint32_t q0 = s0; q0 < s1; q0 += 64) {
    const uint32_t j = q0 + uint32_t(lane);
    const bool act = j < s1;
    const float4 me = g.sorted[act ? j : s0];
    const double qx = me.x, qy = me.y, qz = me.z;
    float gl2[3], gh2[3];
    gl2[0] = face_lb(fmax(qx - bx - slack, 0.0)); gh2[0] = face_lb(fmax(bx + v - qx - slack, 0.0));
    gl2[1] = face_lb(fmax(qy - by - slack, 0.0)); gh2[1] = face_lb(fmax(by + v - qy - slack, 0.0));
    gl2[2] = face_lb(fmax(qz - bz - slack, 0.0)); gh2[2] = face_lb(fmax(bz + v - qz - slack, 0.0));
    Query q = make_query(qx, qy, qz, r2);
    TopK<K> top;
    top.init();
    for (int rank = 0; rank < 27; ++rank) {
      const int code = rank == 0 ? 13 : nbr_code(rank);
      const int32_t cnt = __builtin_amdgcn_readfirstlane(nb_cnt[code]);
      if (cnt == 0) continue;
      bool need = act;
      if (rank > 0) {
        const int ox = code / 9 - 1, oy = (code / 3) % 3 - 1, oz = code % 3 - 1;
        const float lb = (ox < 0 ? gl2[0] : (ox > 0 ? gh2[0] : 0.0f)) +
                         (oy < 0 ? gl2[1] : (oy > 0 ? gh2[1] : 0.0f)) +
                         (oz < 0 ? gl2[2] : (oz > 0 ? gh2[2] : 0.0f));
        need = need && double(lb) <= fmin(r2, top.bound());
      }
      if (!__any(need)) continue;
      const int32_t st = __builtin_amdgcn_readfirstlane(nb_start[code]);
      scan_voxel_points<K>(g.sorted, st, cnt, q, r2, top);
    }
    if (act) {
      double c6[6] = {0, 0, 0, 0, 0, 0};
      const bool ok = top.found() >= k;
      if (ok) regularised_cov<K>(top, k, [&](int32_t pos) { return g.sorted[pos]; }, c6, reg);
      const int64_t i = __float_as_int(me.w);
      float cf[6];
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        cf[t] = float(c6[t]);
        cov6[t * n + i] = cf[t];
      }
      valid[i] = ok ? 1 : 0;
      write_packed(g, j, cf, ok);
    }
  }
}

template <int K>
__global__ __launch_bounds__(64) void k_grid_cov_wave(GridView g, int32_t dense, int64_t n,
                                                      int32_t k, int32_t reg, float* cov6,
                                                      uint8_t* valid) {
  __shared__ int32_t nb_start[27];
  __shared__ int32_t nb_cnt[27];
  // each block of an XCD takes every (gridDim / 8)-th run of its range
  const int x = int(blockIdx.x & 7);
  const int64_t lo = x * g.run_chunk, hi = lo + g.n_runs[16 * x];
  for (int64_t sg = lo + (blockIdx.x >> 3); sg < hi; sg += gridDim.x >> 3)
    grid_cov_run<K>(g, sg, dense, n, k, reg, cov6, valid, nb_start, nb_cnt);
}

// Covariance of every scan point from its k nearest points of the same scan
// within v, one point per lane over the 27 voxels (processed in sorted order
// for locality; written at the original index).  Points of runs with at
// least `dense` points (dense > 0) are left to k_grid_cov_wave.  Non-finite
// points get the zero covariance and the invalid flag.
// Waves per SIMD asked of the per-point covariance search (latency-bound
// gathers, as in the linearisation).
constexpr int kCovMinWaves = 5;

template <int K>
__global__ __launch_bounds__(kT, kCovMinWaves) void k_grid_cov(GridView g, int32_t dense, int64_t n,
                                                               int32_t k, int32_t reg,
                                                               float* cov6, uint8_t* valid) {
  // blocks dealt to the eight XCDs in contiguous ranges of the sorted
  // points: the neighbour voxels a block reads are those of the blocks
  // around it, which then share that XCD's L2
  const int64_t nb = (n + kT - 1) / kT, chunk = (nb + 7) >> 3;
  const int64_t b = int64_t(blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  const int64_t j = b * kT + threadIdx.x;
  if ((blockIdx.x >> 3) >= chunk || j >= n) return;
  const float4 me = g.sorted[j];
  const uint32_t rid = g.run_id[j];
  if (rid == kNoRun) {   // a non-finite point: zero covariance, invalid
    const int64_t i = __float_as_int(me.w);
#pragma unroll
    for (int t = 0; t < 6; ++t) cov6[t * n + i] = 0.0f;
    valid[i] = 0;
    const float z[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    write_packed(g, j, z, false);
    return;
  }
  const double qx = me.x, qy = me.y, qz = me.z;
  // the cells around the point's own cell (the cell of its run's key: the
  // same coordinates and cell edge) from its run's row of the neighbour table
  const uint2* row = g.nbt + int64_t(rid) * 27;
  if (dense > 0 && int32_t(row[13].y) >= dense) return;
  TopK<K> top;
  knn_cells27<K>(qx, qy, qz, g.c, g.inv_c, g.pow2 != 0, g.v * g.v, g.sorted, int32_t(j), g.mx,
                 [&](int code, int32_t* cnt) {
                   const uint2 e = row[code];
                   *cnt = int32_t(e.y);
                   return e.y ? int32_t(e.x) : int32_t(-1);
                 },
                 top);
  double c6[6] = {0, 0, 0, 0, 0, 0};
  const bool ok = top.found() >= k;
  if (ok) regularised_cov<K>(top, k, [&](int32_t pos) { return g.sorted[pos]; }, c6, reg);
  const int64_t i = __float_as_int(me.w);
  const float f0 = float(c6[0]), f1 = float(c6[1]), f2 = float(c6[2]), f3 = float(c6[3]),
              f4 = float(c6[4]), f5 = float(c6[5]);
  if (g.pk_B) {   // the align's packed words at the sorted position (n < 2^31)
    const uint32_t j32 = uint32_t(j);
    g.pk_B[j32] = make_float4(ok ? f0 : -1.0f, f1, f2, f3);
    g.pk_C[j32] = make_float2(f4, f5);
  }
  cov6[i] = f0;
  cov6[n + i] = f1;
  cov6[2 * n + i] = f2;
  cov6[3 * n + i] = f3;
  cov6[4 * n + i] = f4;
  cov6[5 * n + i] = f5;
  valid[i] = ok ? 1 : 0;
}

// Covariances of a small scan, 32 lanes per point.  One lane per point leaves
// most of the chip idle below about 30k points (5000 points are 79 waves, each
// as long as its slowest chain of cells: 60 us; 15.3 us here; k = 5 at 20k
// points 54 -> 34 us, k = 10 at 13k points 86 -> 45 us).  First the lanes share
// the points of the own cell, each keeping its own K best, and the group merges
// them; then every lane ranks one of the other 26 cells against the merged K-th
// best (entries it holds from the start, with no place, so only better points
// enter), and the group merges again.
// The list is the K best by (d2, id) of the same candidates, so the results
// are those of k_grid_cov, bit for bit.
// The lines.  Points: one scan of 16000, 24000, 32000 and 48000 points took 98, 114,
// 133 and 164 us a call at k = 5 (125, 130, 128 and 135 by one lane per point), 123,
// 151, 186 and 263 at k = 10 (220, 204, 207 and 205).  Crowd: without x order a lane
// ranks all points of a neighbour cell, and the chip all pairs of points in a
// cell.  On a plane, k = 5, wide against one lane per point: 2000 points with 100, 200
// and 300 a cell 108, 132 and 163 us (128, 127 and 133); 8000 with 1000 397 (198);
// 16000 with 20, 100 and 300 121, 158 and 249 (130, 136 and 154); 28000 with 10, 50, 300
// and 1000 137, 165, 344 and 756 (131, 126, 158 and 211).  At k = 10 the cell may be
// half as full again.  (crowd is the mean number of points in a point's cell, by
// sample: 0.3 us of the range pass; scans of up to kWideCovFew points gain by the wide
// search whatever their crowd.)
constexpr int64_t kWideCovMax = 28 * 1024, kWideCovFew = 512;
inline bool wide_cov_pays(int64_t n, int32_t k, double crowd) {
  return crowd <= (k <= 5 ? 200.0 : 300.0) && crowd * double(n) <= 1.2e6;
}

template <int K>
__global__ __launch_bounds__(kT) void k_grid_cov_wide(GridView g, int64_t n, int32_t k,
                                                      int32_t reg, float* cov6, uint8_t* valid) {
  constexpr int kPts = kT / kGroup;
  __shared__ int32_t s_pos[kPts][K];   // the K nearest of the block's points (-1: none)
  const int64_t j = int64_t(blockIdx.x) * kPts + threadIdx.x / kGroup;
  const int lane = threadIdx.x & (kGroup - 1);
  float4 me = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (j < n) me = g.sorted[j];
  const bool fin = j < n && isfinite(me.x) && isfinite(me.y) && isfinite(me.z);
  TopK<K> top;
  top.init();
  if (fin) {
    const uint2* row = g.nbt + int64_t(g.run_id[j]) * 27;
    const double px = me.x, py = me.y, pz = me.z, c = g.c, r2 = g.v * g.v;
    const double tx = g.pow2 ? px * g.inv_c : px / c;
    const double fx = floor(tx), fy = floor(g.pow2 ? py * g.inv_c : py / c),
                 fz = floor(g.pow2 ? pz * g.inv_c : pz / c);
    // the own cell, its points dealt to the lanes
    TopK<K> own;
    own.init();
    Query q = make_query(px, py, pz, r2);
    const uint2 me_run = row[13];
    for (uint32_t u = me_run.x + uint32_t(lane); u < me_run.x + me_run.y; u += kGroup) {
      const float4 p = g.sorted[u];
      const double d = dist2(double(p.x), double(p.y), double(p.z), px, py, pz);
      if (d <= r2) own.push(d, __float_as_int(p.w), int32_t(u));
    }
    merge_lists<kGroup>(own, top);
    // one other cell per lane, from the list's last entry on
    const double bound = fmin(r2, top.bound());
    const double slack = 1e-7 * c;
    const int ox = lane / 9 - 1, oy = (lane / 3) % 3 - 1, oz = lane % 3 - 1;
    auto gap = [&](int o, double p, double f) {
      return o == 0 ? 0.0f
                    : lb_down_sq(fmax(o < 0 ? p - f * c - slack : (f + 1.0) * c - p - slack, 0.0));
    };
    const float lb = (gap(ox, px, fx) + gap(oy, py, fy)) + gap(oz, pz, fz);
#pragma unroll
    for (int s = 0; s < K; ++s) {
      own.d[s] = top.d[K - 1];
      own.id[s] = top.id[K - 1];
      own.pos[s] = -1;
    }
    bool any = false;
    if (lane < 27 && lane != 13 && double(lb) <= bound) {
      const uint2 e = row[lane];
      if (e.y) {
        q.bound_f = screen_bound(bound, q.m);
        const float w = fminf(fmaxf(float(e.y) * (float(tx - fx) - float(ox)), 0.0f), float(e.y));
        scan_run_x<K>(g.sorted, int32_t(e.x), int32_t(e.y),
                      int32_t(e.x) + min(int32_t(w), int32_t(e.y)), q, r2, g.mx, own);
        any = own.pos[0] >= 0;
      }
    }
    // (a ballot of the group's half of the wave)
    if ((__ballot(any) >> (threadIdx.x & 32)) & 0xFFFFFFFFull) {
      if (lane == 31) own = top;   // the first list takes part as a lane of its own
      merge_lists<kGroup>(own, top);
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int s = 0; s < K; ++s) s_pos[threadIdx.x / kGroup][s] = top.pos[s];
  }
  __syncthreads();
  // the FP64 covariances by one lane per point, all in the first wave (by every
  // wave for its own points they would take four times the issue slots)
  const int64_t jj = int64_t(blockIdx.x) * kPts + threadIdx.x;
  if (threadIdx.x >= kPts || jj >= n) return;
  int found = 0;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    top.pos[s] = s_pos[threadIdx.x][s];
    found += top.pos[s] >= 0 ? 1 : 0;
  }
  double c6[6] = {0, 0, 0, 0, 0, 0};
  const bool ok = found >= k;
  if (ok) regularised_cov<K>(top, k, [&](int32_t pos) { return g.sorted[pos]; }, c6, reg);
  const int64_t i = __float_as_int(g.sorted[jj].w);
  float cf[6];
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    cf[t] = float(c6[t]);
    cov6[t * n + i] = cf[t];
  }
  valid[i] = ok ? 1 : 0;
  write_packed(g, jj, cf, ok);
}

// Probe lengths of the held keys: summed per block before the two atomics (one
// pair per held slot, all on one address, took 200 us for 0.2M voxels in a
// table of 1M slots; 13 us now).
__global__ __launch_bounds__(kT) void k_probe_stats(const Slot* slots, int64_t n_slots,
                                                    uint32_t slot_mask, int log2_slots,
                                                    unsigned long long* sum,
                                                    uint32_t* maxp) {
  uint32_t total = 0, longest = 0;
  for (int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x; s < n_slots;
       s += int64_t(gridDim.x) * kT) {
    const uint64_t key = slots[s].key;
    if (key == kEmptyKey) continue;
    const uint32_t h = voxel_hash(key_x(key), key_y(key), key_z(key), log2_slots);
    const uint32_t len = ((uint32_t(s) - h) & slot_mask) + 1;
    total += len;
    longest = max(longest, len);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    total += uint32_t(__shfl_xor(int(total), d));
    longest = max(longest, uint32_t(__shfl_xor(int(longest), d)));
  }
  __shared__ uint32_t s_t[kT / 64], s_l[kT / 64];
  if ((threadIdx.x & 63) == 0) {
    s_t[threadIdx.x >> 6] = total;
    s_l[threadIdx.x >> 6] = longest;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long t = 0;
  for (int w = 0; w < kT / 64; ++w) {
    t += s_t[w];
    longest = max(longest, s_l[w]);
  }
  if (!t) return;
  atomicAdd(sum, t);
  atomicMax(maxp, longest);
}

__global__ __launch_bounds__(kT) void k_export(const float4* cov, const float* pt_xyz,
                                               int64_t point_cap, int64_t N, float* xyz,
                                               float* cov6, uint8_t* valid) {
  int64_t i = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (i >= N) return;
  if (xyz) {
    xyz[i] = pt_xyz[i];
    xyz[N + i] = pt_xyz[point_cap + i];
    xyz[2 * N + i] = pt_xyz[2 * point_cap + i];
  }
  float4 a = cov[2 * i], b = cov[2 * i + 1];
  if (cov6) {
    cov6[i] = a.x;
    cov6[N + i] = a.y;
    cov6[2 * N + i] = a.z;
    cov6[3 * N + i] = a.w;
    cov6[4 * N + i] = b.x;
    cov6[5 * N + i] = b.y;
  }
  if (valid) valid[i] = b.z != 0.0f ? 1 : 0;
}

// ---------------------------------------------------------------- fine index
// Fine cell key of every map point (cells of v/2, exact: v is a power of
// two); a key outside the 21-bit range is counted and disables the index.
__global__ __launch_bounds__(kT) void k_fine_keys(const float* pt_xyz, int64_t point_cap,
                                                  int64_t n, double inv_fc, uint64_t* keys,
                                                  uint32_t* vals, uint32_t* counters) {
  int64_t id = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (id >= n) return;
  const double x = pt_xyz[id], y = pt_xyz[point_cap + id], z = pt_xyz[2 * point_cap + id];
  const double fx = floor(x * inv_fc), fy = floor(y * inv_fc), fz = floor(z * inv_fc);
  const double lim = double(kKeyBias);
  uint64_t key = kEmptyKey;
  if (fx >= -lim && fx < lim && fy >= -lim && fy < lim && fz >= -lim && fz < lim)
    key = pack_key(int64_t(fx), int64_t(fy), int64_t(fz));
  else
    atomicAdd(&counters[1], 1u);
  keys[id] = key;
  vals[id] = uint32_t(id);
}

__global__ __launch_bounds__(kT) void k_fine_fill(const float* pt_xyz, int64_t point_cap,
                                                  int64_t n, const uint32_t* vals,
                                                  float4* fine_pts) {
  int64_t j = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (j >= n) return;
  const uint32_t id = vals[j];
  fine_pts[j] = make_float4(pt_xyz[id], pt_xyz[point_cap + id], pt_xyz[2 * point_cap + id],
                            __int_as_float(int32_t(id)));
}

__global__ __launch_bounds__(kT) void k_fine_claim(Slot* slots, uint32_t slot_mask,
                                                   int log2_slots, const uint64_t* keys,
                                                   const uint32_t* seg_start,
                                                   const uint32_t* seg_end, int64_t n_seg) {
  int64_t s = int64_t(blockIdx.x) * kT + threadIdx.x;
  if (s >= n_seg) return;
  const uint64_t key = keys[seg_start[s]];
  uint32_t h = voxel_hash(key_x(key), key_y(key), key_z(key), log2_slots);
  for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
    unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(&slots[h].key),
                                       (unsigned long long)kEmptyKey,
                                       (unsigned long long)key);
    if (old == kEmptyKey) {
      slots[h].vox = int32_t(seg_start[s]);
      slots[h].aux = int32_t(seg_end[s] - seg_start[s]);
      return;
    }
    h = (h + 1) & slot_mask;
  }
}

template <class F>
far_status_t dispatch_k(int32_t k, F&& f) {
  if (k <= 1) return f(std::integral_constant<int, 1>());
  if (k <= 4) return f(std::integral_constant<int, 4>());
  if (k == 5) return f(std::integral_constant<int, 5>());
  if (k <= 8) return f(std::integral_constant<int, 8>());
  if (k <= 10) return f(std::integral_constant<int, 10>());
  if (k <= 16) return f(std::integral_constant<int, 16>());
  return f(std::integral_constant<int, 32>());
}

// Points sorted (stably) by full voxel key: the path of key ranges too wide for
// compact keys.
far_status_t sort_full_keys(const float* xyz, int64_t n, double v, hipStream_t st, Scratch& scr,
                            uint64_t** keys, uint32_t** vals) {
  uint64_t* keys_alt;
  uint32_t *vals_alt, *counters;
  FAR_TRY(scr.get(keys, size_t(n)));
  FAR_TRY(scr.get(vals, size_t(n)));
  FAR_TRY(scr.get(&keys_alt, size_t(n)));
  FAR_TRY(scr.get(&vals_alt, size_t(n)));
  FAR_TRY(scr.get(&counters, 2));
  FAR_HIP(hipMemsetAsync(counters, 0, 2 * sizeof(uint32_t), st));
  k_keys<<<blocks_for(n), kT, 0, st>>>(xyz, n, v, *keys, *vals, counters);
  FAR_HIP(hipGetLastError());
  bool alt = false;
  FAR_TRY(radix_sort_pairs(*keys, *vals, keys_alt, vals_alt, n, 64, st, scr, &alt));
  if (alt) {
    *keys = keys_alt;
    *vals = vals_alt;
  }
  return FAR_OK;
}

// Blocks for n items one per thread, at most per_cu per CU (the kernel strides).
inline unsigned blocks_upto(int64_t n, int per_cu) {
  return unsigned(std::min<int64_t>(blocks_for(n), int64_t(per_cu) * device_cu_count()));
}

inline int ceil_log2(int64_t x) {
  int l = 0;
  while ((int64_t(1) << l) < x) ++l;
  return l;
}

}  // namespace

// Covariance regularisation of every covariance computed from now on
// (far_set_covariance_regularisation): FAR_REG_EQ1 or FAR_REG_PLANE.
int32_t g_cov_reg = FAR_REG_EQ1;

far_status_t fine_build(far_map_s* m, hipStream_t st) {
  if (m->fine_ok || m->n_points == 0) return FAR_OK;
  int e2 = 0;
  if (std::frexp(m->p.voxel_size, &e2) != 0.5) return FAR_OK;   // not a power of two
  const int64_t n = m->n_points;
  Scratch scr(st);
  uint64_t *keys, *keys_alt;
  uint32_t *vals, *vals_alt, *seg_start, *seg_end, *counters;
  FAR_TRY(scr.get(&keys, size_t(n)));
  FAR_TRY(scr.get(&keys_alt, size_t(n)));
  FAR_TRY(scr.get(&vals, size_t(n)));
  FAR_TRY(scr.get(&vals_alt, size_t(n)));
  FAR_TRY(scr.get(&seg_start, size_t(n)));
  FAR_TRY(scr.get(&seg_end, size_t(n)));
  FAR_TRY(scr.get(&counters, 4));
  FAR_HIP(hipMemsetAsync(counters, 0, 4 * sizeof(uint32_t), st));
  const double inv_fc = 2.0 / m->p.voxel_size;
  k_fine_keys<<<blocks_for(n), kT, 0, st>>>(m->pt_xyz, m->p.point_capacity, n, inv_fc, keys,
                                            vals, counters);
  FAR_HIP(hipGetLastError());
  FAR_TRY(radix_sort_pairs(keys, vals, keys_alt, vals_alt, n, kKeyBits, st, scr));
  FAR_TRY(scan_flags(RunFlags{SortedKeys{keys, kEmptyKey}, n, seg_start, seg_end}, n,
                     counters + 2, st, scr));
  uint32_t h_cnt[4];
  FAR_HIP(hipMemcpyAsync(h_cnt, counters, sizeof(h_cnt), hipMemcpyDeviceToHost, st));
  FAR_HIP(hipStreamSynchronize(st));
  if (h_cnt[1] > 0) return FAR_OK;                    // out of the fine key range
  const int64_t n_seg = h_cnt[2];
  FAR_HIP(hipMemsetAsync(m->fine_slots, 0xFF, size_t(m->fine_nslots) * sizeof(Slot), st));
  k_fine_claim<<<blocks_for(n_seg), kT, 0, st>>>(m->fine_slots, uint32_t(m->fine_nslots - 1),
                                                 m->fine_log2, keys, seg_start, seg_end, n_seg);
  FAR_HIP(hipGetLastError());
  k_fine_fill<<<blocks_for(n), kT, 0, st>>>(m->pt_xyz, m->p.point_capacity, n, vals,
                                            m->fine_pts);
  FAR_HIP(hipGetLastError());
  m->fine_ok = true;
  return FAR_OK;
}

// Certificates of the points of the voxels marked with gen (of all n_vox
// voxels when mark is null; at most n_pts points), and with cov given the
// covariances of the counts->n_acc (at most n_add) points with ids from id0
// on: in the same search when its list is long enough for the map's k_cov (up
// to 10), else by a search of their own.
far_status_t certs_build(far_map_s* m, int64_t n_vox, int64_t n_pts, const uint32_t* mark,
                         uint32_t gen, InsertCounts* counts, float4* cov, int64_t id0,
                         int64_t n_add, hipStream_t st, Scratch& scr) {
  if (n_vox == 0 || n_pts == 0) return FAR_OK;
  uint32_t* list;
  FAR_TRY(scr.get(&list, size_t(n_pts)));
  k_cert_list<<<blocks_for(n_vox), kT, 0, st>>>(n_vox, m->p.max_pts_per_voxel, m->vox_count,
                                                mark, gen, list, &counts->n_cert);
  FAR_HIP(hipGetLastError());
  const int32_t k = m->p.k_cov;
  const uint32_t* n_cert = &counts->n_cert;
  const unsigned nb = blocks_upto(n_pts, 16);
  float4* const c = k <= 10 ? cov : nullptr;
  // (an insert lists the points around the added ones too: two to three times
  // as many in a map that fills up)
  const int64_t listed = mark ? 2 * n_add : n_pts;
  auto go = [&](auto KK) {
    constexpr int K = decltype(KK)::value;
    if (listed <= kCertQuadMax)
      k_cert_build_quad<K><<<blocks_upto(n_pts * 4, 32), kT, 0, st>>>(
          m->view(), list, n_cert, m->cert, c, m->vox_cov, id0, k, g_cov_reg);
    else
      k_cert_build<K><<<nb, kT, 0, st>>>(m->view(), list, n_cert, m->cert, c, m->vox_cov, id0, k,
                                         g_cov_reg);
  };
  if (k <= kCertK + 2 || k > 10)
    go(std::integral_constant<int, kCertK + 2>());
  else
    go(std::integral_constant<int, 10>());
  FAR_HIP(hipGetLastError());
  if (!cov || k <= 10 || n_add <= 0) return FAR_OK;
  return dispatch_k(k, [&](auto KK) -> far_status_t {
    constexpr int K = decltype(KK)::value;
    k_map_cov<K><<<blocks_upto(n_add, 16), kT, 0, st>>>(m->view(), cov, m->vox_cov, m->pt_loc,
                                                        id0, &counts->n_acc, k, g_cov_reg);
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  });
}

// An empty map: the hash of the voxels, the counts of the first n_vox, the ghosts'
// hash and count (ghosts on), cleared in one launch.
far_status_t voxels_reset(far_map_s* m, hipStream_t st) {
  // (four slots a thread; 8192 striding blocks took 364 us for 1.3 GB, this 283)
  const int64_t n = std::max(m->slots, m->gslots_n);
  k_clear_voxels<<<blocks_for(n, 4 * kT), kT, 0, st>>>(m->slots_d, m->slots, m->gslots,
                                                       m->gslots_n, m->vox_count, m->n_voxels,
                                                       m->gcount);
  FAR_HIP(hipGetLastError());
  m->n_ghosts = 0;
  m->ghost_ok = true;
  return FAR_OK;
}

// Neighbour rows, marks and ghosts after the voxels of the runs seg_vox (at
// most n_max, counts->n_seg in fact) changed; all of them are new when is_new
// is null.  counts->ghosts receives the ghost count.
far_status_t links_update(far_map_s* m, int64_t n_max, int64_t vox_room, InsertCounts* counts,
                          const int32_t* seg_vox, const uint32_t* is_new,
                          const uint32_t* seg_changed, hipStream_t st) {
  const MapView mv = m->view();
  k_links<<<blocks_upto(n_max * 26, 32), kT, 0, st>>>(mv, counts, vox_room, seg_vox, is_new,
                                                     seg_changed, m->vox_key, m->vox_nbr,
                                                     m->cert_mark, m->cert_gen, m->gslots,
                                                     m->gkey, m->gcount, m->ghost_cap);
  FAR_HIP(hipGetLastError());
  // (a surface map has about two ghosts per voxel; the kernel reads how many)
  k_ghost_fill<<<blocks_upto(n_max * 52, 16), kT, 0, st>>>(
      mv, m->gkey, m->gcount, m->n_ghosts, m->ghost_ok ? m->ghost_cap : 0, m->gnbr,
      &counts->ghosts);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

// Layout of compact keys (no x bits) for the points' range: *fits = false when
// no point is finite (*none) or a key with the scan id needs more than 62 bits;
// *oor receives the points whose keys leave [-2^20, 2^20), *crowd (if not null) the
// mean number of points in a point's cell, by sample.  One small copy and one wait.
static far_status_t compact_layout(const float* xyz, const int64_t* offsets, int64_t n,
                                   double cell, int32_t S_, hipStream_t st, Scratch& scr, CompactKey* ck, bool* fits,
                                   uint32_t* oor, bool* none, double* crowd = nullptr) {
  *fits = false;
  *oor = 0;
  if (none) *none = false;
  uint32_t* rng;
  FAR_TRY(scr.get(&rng, 8));
  FAR_HIP(hipMemsetAsync(rng, 0, 8 * sizeof(uint32_t), st));
  int e2 = 0;
  const int32_t pow2 = std::frexp(cell, &e2) == 0.5 ? 1 : 0;
  const unsigned nb = unsigned(std::min<int64_t>(blocks_for(n, 4 * kT), kRangeBlocks));
  if (crowd)
    k_key_range<true><<<nb + 1, kT, 0, st>>>(xyz, n, cell, 1.0 / cell, pow2, offsets, S_, rng);
  else
    k_key_range<false><<<nb, kT, 0, st>>>(xyz, n, cell, 1.0 / cell, pow2, nullptr, 1, rng);
  FAR_HIP(hipGetLastError());
  uint32_t h[8];
  FAR_TRY(fetch(st, h, rng, sizeof(h)));
  if (crowd)
    *crowd = double(n) * (double(h[7]) / (double(kCrowdSample) * kCrowdSample) - 1.0 / kCrowdCells);
  *oor = h[6];
  if (h[6] > 0) return FAR_OK;
  if (h[0] == 0) {
    if (none) *none = true;
    return FAR_OK;
  }
  int32_t lo[3], hi[3];
  for (int a = 0; a < 3; ++a) {
    lo[a] = int32_t(kKeyBias) - int32_t(h[a]);
    hi[a] = int32_t(h[3 + a]) - int32_t(kKeyBias) - 1;
  }
  ck->mx = lo[0];
  ck->my = lo[1];
  ck->mz = lo[2];
  ck->bx = std::max(ceil_log2(int64_t(hi[0]) - lo[0] + 1), 2);
  ck->by = std::max(ceil_log2(int64_t(hi[1]) - lo[1] + 1), 2);
  ck->bz = std::max(ceil_log2(int64_t(hi[2]) - lo[2] + 1), 2);
  ck->kb = ck->bx + ck->by + ck->bz;
  ck->fb = 0;
  *fits = (S_ > 1 ? ceil_log2(S_) : 0) + ck->kb + 1 <= 62;
  return FAR_OK;
}

// The ghost count the device reached: beyond the capacity the ghosts go off.
void ghosts_take(far_map_s* m, uint32_t ghosts) {
  m->n_ghosts = ghosts;
  if (int64_t(ghosts) > m->ghost_cap) m->ghost_ok = false;
}

}  // namespace far

using namespace far;

extern "C" {

const char* far_status_str(far_status_t s) {
  switch (s) {
    case FAR_OK: return "ok";
    case FAR_E_INVALID: return "invalid argument";
    case FAR_E_CAPACITY: return "capacity exceeded";
    case FAR_E_HIP: return "HIP runtime error";
    case FAR_E_NOT_PD: return "H not positive definite";
    case FAR_E_FEW_CORR: return "too few correspondences";
    case FAR_E_UNSUPPORTED: return "unsupported";
  }
  return "unknown status";
}

const char* far_last_error(void) { return g_err; }

far_status_t far_map_create(const far_map_params_t* params, far_stream_t stream,
                            far_map_t* out) {
  if (!params || !out) {
    set_error("far_map_create: null argument");
    return FAR_E_INVALID;
  }
  *out = nullptr;
  far_map_params_t p = *params;
  if (!(p.voxel_size > 0.0) || !std::isfinite(p.voxel_size) || p.max_pts_per_voxel < 1 ||
      p.max_pts_per_voxel > 64 || p.point_capacity < 1 || p.point_capacity >= (int64_t(1) << 31) ||
      p.k_cov < 1 || p.k_cov > 32 || !std::isfinite(p.min_spacing)) {
    set_error("far_map_create: parameter out of range");
    return FAR_E_INVALID;
  }
  // the neighbour table packs a voxel index into 25 bits
  if (p.voxel_capacity <= 0)
    p.voxel_capacity = std::min<int64_t>(p.point_capacity, (int64_t(1) << 25) - 1);
  if (p.voxel_capacity >= (int64_t(1) << 25) ||
      p.voxel_capacity * p.max_pts_per_voxel >= (int64_t(1) << 31)) {
    set_error("far_map_create: need voxel_capacity < 2^25 and voxel_capacity * "
              "max_pts_per_voxel < 2^31");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  far_map_s* m = new far_map_s();
  m->p = p;
  m->dmin = p.min_spacing < 0 ? p.voxel_size / std::sqrt(double(p.max_pts_per_voxel))
                              : p.min_spacing;
  m->voxel_cap = p.voxel_capacity;
  m->log2_slots = ceil_log2(2 * p.voxel_capacity);
  if (m->log2_slots < 10) m->log2_slots = 10;
  m->slots = int64_t(1) << m->log2_slots;
  if (hipGetDevice(&m->device) != hipSuccess) m->device = 0;
  auto fail = [&](hipError_t e, const char* what) {
    far_map_destroy(m);
    return hip_fail(e, what, __FILE__, __LINE__);
  };
  hipError_t e;
  size_t b_slots = size_t(m->slots) * sizeof(Slot);
  size_t b_cnt = size_t(m->voxel_cap) * sizeof(int32_t);
  size_t b_key = size_t(m->voxel_cap) * sizeof(uint64_t);
  size_t b_pts = size_t(m->voxel_cap) * p.max_pts_per_voxel * sizeof(float4);
  size_t b_cov = size_t(p.point_capacity) * 2 * sizeof(float4);
  size_t b_vcov = size_t(m->voxel_cap) * p.max_pts_per_voxel * 2 * sizeof(float4);
  size_t b_nbr = size_t(m->voxel_cap) * 26 * sizeof(uint32_t);
  size_t b_xyz = size_t(p.point_capacity) * 3 * sizeof(float);
  size_t b_loc = size_t(p.point_capacity) * sizeof(int32_t);
  size_t b_vslot = size_t(m->voxel_cap) * sizeof(int32_t);
  size_t b_cert = size_t(m->voxel_cap) * p.max_pts_per_voxel * sizeof(CertRow);
  size_t b_mark = size_t(m->voxel_cap) * sizeof(uint32_t);
  // ghosts: four per voxel of capacity (a surface map has about two)
  m->ghost_cap = 4 * m->voxel_cap;
  m->glog2 = ceil_log2(2 * m->ghost_cap);
  if (m->glog2 < 10) m->glog2 = 10;
  m->gslots_n = int64_t(1) << m->glog2;
  size_t b_gslots = size_t(m->gslots_n) * sizeof(Slot);
  size_t b_gkey = size_t(m->ghost_cap) * sizeof(uint64_t);
  size_t b_gnbr = size_t(m->ghost_cap) * 26 * sizeof(uint32_t);
  m->fine_log2 = ceil_log2(2 * p.point_capacity);
  if (m->fine_log2 < 10) m->fine_log2 = 10;
  m->fine_nslots = int64_t(1) << m->fine_log2;
  size_t b_fpts = size_t(p.point_capacity) * sizeof(float4);
  size_t b_fslots = size_t(m->fine_nslots) * sizeof(Slot);
  if ((e = hipMalloc(&m->slots_d, b_slots)) != hipSuccess) return fail(e, "hipMalloc slots");
  if ((e = hipMalloc(&m->vox_count, b_cnt)) != hipSuccess) return fail(e, "hipMalloc counts");
  if ((e = hipMalloc(&m->vox_key, b_key)) != hipSuccess) return fail(e, "hipMalloc keys");
  if ((e = hipMalloc(&m->vox_pts, b_pts)) != hipSuccess) return fail(e, "hipMalloc points");
  if ((e = hipMalloc(&m->cov, b_cov)) != hipSuccess) return fail(e, "hipMalloc cov");
  if ((e = hipMalloc(&m->vox_cov, b_vcov)) != hipSuccess) return fail(e, "hipMalloc cov");
  if ((e = hipMalloc(&m->vox_nbr, b_nbr)) != hipSuccess) return fail(e, "hipMalloc nbr");
  if ((e = hipMalloc(&m->pt_xyz, b_xyz)) != hipSuccess) return fail(e, "hipMalloc xyz");
  if ((e = hipMalloc(&m->pt_loc, b_loc)) != hipSuccess) return fail(e, "hipMalloc loc");
  if ((e = hipMalloc(&m->vox_slot, b_vslot)) != hipSuccess) return fail(e, "hipMalloc vslot");
  if ((e = hipMalloc(&m->cert, b_cert)) != hipSuccess) return fail(e, "hipMalloc cert");
  if ((e = hipMalloc(&m->cert_mark, b_mark)) != hipSuccess) return fail(e, "hipMalloc mark");
  if ((e = hipMalloc(&m->gslots, b_gslots)) != hipSuccess) return fail(e, "hipMalloc ghosts");
  if ((e = hipMalloc(&m->gkey, b_gkey)) != hipSuccess) return fail(e, "hipMalloc ghosts");
  if ((e = hipMalloc(&m->gnbr, b_gnbr)) != hipSuccess) return fail(e, "hipMalloc ghosts");
  if ((e = hipMalloc(&m->gcount, sizeof(uint32_t))) != hipSuccess) return fail(e, "hipMalloc ghosts");
  if ((e = hipMalloc(&m->fine_pts, b_fpts)) != hipSuccess) return fail(e, "hipMalloc fine");
  if ((e = hipMalloc(&m->fine_slots, b_fslots)) != hipSuccess) return fail(e, "hipMalloc fine");
  m->bytes = int64_t(b_slots + b_cnt + b_key + b_pts + b_cov + b_vcov + b_nbr + b_xyz + b_loc + b_vslot +
                     b_cert + b_mark + b_gslots + b_gkey + b_gnbr + sizeof(uint32_t) + b_fpts +
                     b_fslots);
  if ((e = hipMemsetAsync(m->slots_d, 0xFF, b_slots, st)) != hipSuccess) return fail(e, "memset");
  if ((e = hipMemsetAsync(m->vox_count, 0, b_cnt, st)) != hipSuccess) return fail(e, "memset");
  if ((e = hipMemsetAsync(m->cert_mark, 0, b_mark, st)) != hipSuccess) return fail(e, "memset");
  if ((e = hipMemsetAsync(m->gslots, 0xFF, b_gslots, st)) != hipSuccess) return fail(e, "memset");
  if ((e = hipMemsetAsync(m->gcount, 0, sizeof(uint32_t), st)) != hipSuccess)
    return fail(e, "memset");
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail(e, "sync");
  *out = m;
  return FAR_OK;
}

far_status_t far_map_destroy(far_map_t m) {
  if (!m) return FAR_OK;
  hipError_t e = hipDeviceSynchronize();
  free_ws(m->ws);
  m->ws = nullptr;
  void* ptrs[] = {m->slots_d, m->vox_count, m->vox_key, m->vox_pts, m->cov, m->vox_cov,
                  m->vox_nbr, m->pt_xyz,
                  m->pt_loc, m->vox_slot, m->cert, m->cert_mark, m->gslots, m->gkey,
                  m->gnbr, m->gcount, m->fine_pts, m->fine_slots};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  delete m;
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize", __FILE__, __LINE__);
  return FAR_OK;
}

far_status_t far_map_insert(far_map_t m, const float* xyz, int64_t n, const int32_t* caps,
                            far_stream_t stream, int64_t* n_accepted) {
  if (n_accepted) *n_accepted = 0;
  if (!m || n < 0 || n >= (int64_t(1) << 31) || (n > 0 && !xyz)) {
    set_error("far_map_insert: invalid argument");
    return FAR_E_INVALID;
  }
  if (n == 0) return FAR_OK;
  hipStream_t st = S(stream);
  Scratch scr(st);
  const double v = m->p.voxel_size;
  m->fine_ok = false;
  // the one wait before the last: the points' key range gives the sort's keys
  CompactKey ck;
  bool fits = false, none = false;
  uint32_t oor = 0;
  FAR_TRY(compact_layout(xyz, nullptr, n, v, 1, st, scr, &ck, &fits, &oor, &none));
  if (oor > 0) {
    set_error("far_map_insert: %u points have voxel keys outside [-2^20, 2^20)", oor);
    return FAR_E_INVALID;
  }
  if (none) return FAR_OK;
  uint64_t* keys;
  uint32_t *vals, *seg_start, *seg_end, *is_new, *acc_flag, *id_local, *seg_changed;
  int32_t *seg_vox, *acc_pos, *seg_newcount;
  InsertCounts* counts;
  const size_t nn = size_t(n);
  FAR_TRY(scr.get(&counts, 1));
  FAR_TRY(scr.get(&seg_start, nn));
  FAR_TRY(scr.get(&seg_end, nn));
  FAR_TRY(scr.get(&seg_vox, nn));
  FAR_TRY(scr.get(&is_new, nn));
  FAR_TRY(scr.get(&acc_flag, nn));
  FAR_TRY(scr.get(&acc_pos, nn));
  FAR_TRY(scr.get(&id_local, nn));
  FAR_TRY(scr.get(&seg_newcount, nn));
  FAR_TRY(scr.get(&seg_changed, nn));
  FAR_HIP(hipMemsetAsync(counts, 0, sizeof(InsertCounts), st));
  if (fits) {
    uint64_t* keys_alt;
    uint32_t* vals_alt;
    FAR_TRY(scr.get(&keys, nn));
    FAR_TRY(scr.get(&keys_alt, nn));
    FAR_TRY(scr.get(&vals, nn));
    FAR_TRY(scr.get(&vals_alt, nn));
    int e2 = 0;
    const int32_t pow2 = std::frexp(v, &e2) == 0.5 ? 1 : 0;
    k_keys_compact<<<blocks_for(n), kT, 0, st>>>(xyz, n, v, 1.0 / v, pow2, nullptr, 1, ck, keys,
                                                  vals, acc_flag, nullptr);
    FAR_HIP(hipGetLastError());
    bool alt = false;
    FAR_TRY(radix_sort_pairs(keys, vals, keys_alt, vals_alt, n, ck.kb + 1, st, scr, &alt));
    if (alt) {
      keys = keys_alt;
      vals = vals_alt;
    }
  } else {   // a range that needs the full keys
    FAR_HIP(hipMemsetAsync(acc_flag, 0, nn * sizeof(uint32_t), st));
    FAR_TRY(sort_full_keys(xyz, n, v, st, scr, &keys, &vals));
  }
  const SortedKeys sk{keys, fits ? uint64_t(1) << ck.kb : kEmptyKey};
  FAR_TRY(scan_flags(RunFlags{sk, n, seg_start, seg_end}, n, &counts->n_seg, st, scr));
  const int64_t vox_room = m->voxel_cap - m->n_voxels;
  const int64_t room = m->p.point_capacity - m->n_points;
  FAR_TRY(scan_flags(NewVoxelFlags{m->view(), xyz, n, v, vals, seg_start, counts, m->n_voxels,
                                   vox_room, seg_vox, is_new, m->slots_d, m->vox_key,
                                   m->vox_slot},
                     n, &counts->n_new, st, scr));
  const double dmin2 = m->dmin > 0 ? m->dmin * m->dmin : 0.0;
  k_greedy<<<blocks_upto(n * kGreedyLanes, 16), kT, 0, st>>>(
      xyz, n, caps, m->p.max_pts_per_voxel, dmin2, vals, seg_start, seg_end, counts, vox_room,
      seg_vox, m->vox_count, m->vox_pts, acc_flag, acc_pos, seg_newcount);
  FAR_HIP(hipGetLastError());
  FAR_TRY(scan_flags(CommitFlags{xyz, n, acc_flag, acc_pos, id_local, m->n_points,
                                 m->p.point_capacity, m->vox_pts, m->pt_xyz, m->pt_loc},
                     n, &counts->n_acc, st, scr));
  k_counts<<<blocks_upto(n, 8), kT, 0, st>>>(counts, vox_room, room, seg_vox, seg_newcount, vals,
                                              seg_start, seg_end, acc_flag, id_local,
                                              m->vox_count, m->vox_slot, m->slots_d, seg_changed);
  FAR_HIP(hipGetLastError());
  // certificates of the points within v of an added point
  if (++m->cert_gen == 0) {
    FAR_HIP(hipMemsetAsync(m->cert_mark, 0, size_t(m->voxel_cap) * sizeof(uint32_t), st));
    m->cert_gen = 1;
  }
  FAR_TRY(links_update(m, n, vox_room, counts, seg_vox, is_new, seg_changed, st));
  const int64_t n_add = std::min(n, room);
  FAR_TRY(certs_build(m, m->n_voxels + std::min(n, vox_room), m->n_points + n_add, m->cert_mark,
                      m->cert_gen, counts, m->cov, m->n_points, n_add, st, scr));
  InsertCounts h;
  FAR_TRY(fetch(st, &h, counts, sizeof(h)));
  if (int64_t(h.n_new) > vox_room) {
    set_error("far_map_insert: %lld new voxels exceed the voxel capacity %lld",
              (long long)h.n_new, (long long)m->voxel_cap);
    return FAR_E_CAPACITY;
  }
  const int64_t n_commit = std::min<int64_t>(h.n_acc, room);
  ghosts_take(m, h.ghosts);
  m->n_points += n_commit;
  m->n_voxels += h.n_new;
  if (n_accepted) *n_accepted = n_commit;
  if (int64_t(h.n_acc) > n_commit) {
    set_error("far_map_insert: point capacity %lld reached; %lld accepted points dropped",
              (long long)m->p.point_capacity, (long long)(int64_t(h.n_acc) - n_commit));
    return FAR_E_CAPACITY;
  }
  return FAR_OK;
}

far_status_t far_map_knn(far_map_t m, const float* q, int64_t n, int32_t k, double radius,
                         int32_t* idx, float* d2, int32_t* count, far_stream_t stream) {
  if (!m || n < 0 || k < 1 || k > 32 || !(radius > 0.0) || radius > m->p.voxel_size ||
      (n > 0 && (!q || !idx))) {
    set_error("far_map_knn: invalid argument (need 1 <= k <= 32, 0 < radius <= v)");
    return FAR_E_INVALID;
  }
  if (n == 0) return FAR_OK;
  hipStream_t st = S(stream);
  MapView mv = m->view();
  double r2 = radius * radius;
  return dispatch_k(k, [&](auto KK) -> far_status_t {
    constexpr int K = decltype(KK)::value;
    k_map_knn<K><<<blocks_for(n, kKnnThreads), kKnnThreads, 0, st>>>(mv, q, n, k, r2, idx, d2,
                                                                     count);
    FAR_HIP(hipGetLastError());
    return FAR_OK;
  });
}

// Voxel grid of a batch of scans with cells of edge `cell`: the points sorted
// by (scan, cell, x), through compact keys (see k_key_range) or, when the
// batch's key range needs more than 62 bits with the scan id, by full keys and
// then by scan (runs not ordered by x, as without by_x); the runs, a hash of
// them, and each run's neighbour cells.  *oor receives the points whose keys
// leave [-2^20, 2^20) (the grid is then not built).  *wide (given as whether the wide
// covariances of k neighbours come into question) receives whether they are taken;
// without by_x the grid of those has no x order.
static far_status_t build_grid(const float* xyz, const int64_t* offsets, int32_t S_, int64_t n,
                               double v, double cell, hipStream_t st, Scratch& scr,
                               int32_t k, bool by_x, bool* wide, GridView* out, uint32_t* oor,
                               uint32_t* order = nullptr, float4* sorted_in = nullptr) {
  CompactKey ck{};
  bool compact = false, none = false;
  // per point: two slots (32 B), 27 cells (216), run arrays (24), keys and
  // values twice (24), sorted point (16), and the sort's tables and small words
  FAR_TRY(scr.reserve(size_t(n) * (32 + 216 + 24 + 24 + 16 + 2) + (size_t(1) << 20)));
  double crowd = 0.0;
  FAR_TRY(compact_layout(xyz, S_ > 1 ? offsets : nullptr, n, cell, S_, st, scr, &ck, &compact, oor, &none,
                         *wide && n > kWideCovFew ? &crowd : nullptr));
  if (*oor > 0) return FAR_OK;
  *wide = *wide && wide_cov_pays(n, k, crowd);
  by_x = by_x || !*wide;
  int e2 = 0;
  const int32_t pow2 = std::frexp(cell, &e2) == 0.5 ? 1 : 0;
  const size_t nn = size_t(n);
  const int64_t n_slots = 2 * n;   // two slots per point, each scan's in its own stretch
  Slot* slots;
  uint64_t *keys, *run_key;
  uint32_t *vals, *run_start, *run_end, *run_id, *n_runs, *run_sid = nullptr, *sid = nullptr;
  uint2* nbt;
  FAR_TRY(scr.get(&n_runs, 8 * 16));
  FAR_TRY(scr.get(&slots, size_t(n_slots)));
  FAR_TRY(scr.get(&run_key, nn));
  FAR_TRY(scr.get(&run_start, nn));
  FAR_TRY(scr.get(&run_end, nn));
  FAR_TRY(scr.get(&run_id, nn));
  if (S_ > 1) FAR_TRY(scr.get(&run_sid, nn));
  FAR_HIP(hipMemsetAsync(n_runs, 0, 8 * 16 * sizeof(uint32_t), st));
  float4* sorted = sorted_in;   // the caller's packed A words: the sorted points are exactly those
  if (!sorted) FAR_TRY(scr.get(&sorted, nn));
  if (compact) {
    uint64_t* keys_alt;
    uint32_t* vals_alt;
    FAR_TRY(scr.get(&keys, nn));
    FAR_TRY(scr.get(&keys_alt, nn));
    FAR_TRY(scr.get(&vals, nn));
    FAR_TRY(scr.get(&vals_alt, nn));
    const int key_bits = (S_ > 1 ? ceil_log2(S_) : 0) + ck.kb + 1;
    // x bits: one more radix pass of 8 bits (8 to 15 bits), within 62 in all
    ck.fb = by_x ? std::min(((key_bits + 15) / 8) * 8 - key_bits, 62 - key_bits) : 0;
    k_keys_compact<<<blocks_for(n), kT, 0, st>>>(xyz, n, cell, 1.0 / cell, pow2,
                                                  S_ > 1 ? offsets : nullptr, S_, ck, keys, vals,
                                                  nullptr, slots);
    FAR_HIP(hipGetLastError());
    bool alt = false;
    FAR_TRY(radix_sort_pairs(keys, vals, keys_alt, vals_alt, n, key_bits + ck.fb, st, scr, &alt));
    if (alt) {
      keys = keys_alt;
      vals = vals_alt;
    }
  } else {
    FAR_HIP(hipMemsetAsync(slots, 0xFF, size_t(n_slots) * sizeof(Slot), st));
    FAR_TRY(sort_full_keys(xyz, n, cell, st, scr, &keys, &vals));
    if (S_ > 1) {
      // second stable sort, by scan id, keeps the key order inside every scan
      uint64_t *sid_key, *sid_alt, *keys2;
      uint32_t *perm, *perm_alt, *vals2;
      FAR_TRY(scr.get(&sid_key, nn));
      FAR_TRY(scr.get(&sid_alt, nn));
      FAR_TRY(scr.get(&perm, nn));
      FAR_TRY(scr.get(&perm_alt, nn));
      FAR_TRY(scr.get(&keys2, nn));
      FAR_TRY(scr.get(&vals2, nn));
      FAR_TRY(scr.get(&sid, nn));
      k_scan_ids<<<blocks_for(n), kT, 0, st>>>(vals, n, offsets, S_, sid_key, perm);
      FAR_HIP(hipGetLastError());
      FAR_TRY(radix_sort_pairs(sid_key, perm, sid_alt, perm_alt, n, ceil_log2(S_), st, scr));
      k_apply_perm<<<blocks_for(n), kT, 0, st>>>(perm, n, keys, vals, keys2, vals2, sid_key, sid);
      FAR_HIP(hipGetLastError());
      keys = keys2;
      vals = vals2;
    }
  }
  FAR_TRY(scr.get(&nbt, nn * 27));
  // a later point of an x-sorted run lies at most one quantum (2^-fb cells,
  // plus the rounding of x / cell) below an earlier one; twice that is kept
  const double mx = compact && ck.fb > 0 ? std::ldexp(cell, 1 - ck.fb) : HUGE_VAL;
  // four positions a lane where the blocks' adds on the run counts would
  // otherwise be many
  const int per = n > (1 << 20) ? 4 : 1;
  const int64_t nb = (n + kT * per - 1) / (kT * per);
  *out = GridView{slots, sorted, v, cell, 1.0 / cell, pow2, S_ > 1 ? offsets : nullptr,
                  uint32_t(n_slots), mx, ((nb + 7) >> 3) * kT * per, n_runs, run_key, run_sid,
                  run_start, run_end, run_id, nbt, nullptr, nullptr};
  const GridKeys gk{keys, sid, compact ? 1 : 0, S_ > 1 ? 1 : 0, ck};
  const unsigned grid = unsigned(((nb + 7) / 8) * 8);
  if (per == 4)
    k_grid_runs<4><<<grid, kT, 0, st>>>(*out, gk, xyz, n, vals, slots, sorted, order, n_runs,
                                        run_key, run_sid, run_start, run_end);
  else
    k_grid_runs<1><<<grid, kT, 0, st>>>(*out, gk, xyz, n, vals, slots, sorted, order, n_runs,
                                        run_key, run_sid, run_start, run_end);
  FAR_HIP(hipGetLastError());
  k_grid_nbr_table<<<grid_blocks(n * 27), kT, 0, st>>>(*out, nbt);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

// Points per voxel run from which the covariance search takes one wave per
// run (k_grid_cov_wave) instead of one lane per point; 0 = never.
static int32_t g_dense_threshold = 0;

static far_status_t scan_cov_impl(const float* xyz, const int64_t* offsets, int32_t S_,
                                  int64_t n, double voxel_size, int32_t k, float* cov6,
                                  uint8_t* valid, hipStream_t st, const char* who,
                                  uint32_t* order = nullptr, void* packed = nullptr) {
  Scratch scr(st);
  TimedScope ts(FAR_TIME_COVARIANCES, st);
  GridView g{};
  uint32_t oor = 0;
  char* pk = static_cast<char*>(packed);
  const int32_t dense = g_dense_threshold;
  // the wide search deals a cell's few points to its lanes and gains less from
  // runs in x order than their radix pass costs; an order the caller receives
  // keeps it
  bool wide = dense == 0 && k <= 10 && n <= kWideCovMax;
  FAR_TRY(build_grid(xyz, offsets, S_, n, voxel_size, voxel_size, st, scr, k, order || packed,
                     &wide, &g, &oor, order, reinterpret_cast<float4*>(pk)));
  if (pk) {
    g.pk_B = reinterpret_cast<float4*>(pk + 16 * n);
    g.pk_C = reinterpret_cast<float2*>(pk + 32 * n);
  }
  if (oor > 0) {
    set_error("%s: %u points have voxel keys outside [-2^20, 2^20)", who, oor);
    return FAR_E_INVALID;
  }
  // (a batch with no finite point has no runs: every point takes the
  // non-finite branch of k_grid_cov, zero covariance and invalid)
  return dispatch_k(k, [&](auto KK) -> far_status_t {
    constexpr int K = decltype(KK)::value;
    if constexpr (K <= 10) {
      if (wide) {
        k_grid_cov_wide<K><<<blocks_for(n * kGroup), kT, 0, st>>>(g, n, k, g_cov_reg, cov6,
                                                                     valid);
        FAR_HIP(hipGetLastError());
        return FAR_OK;
      }
    }
    const int64_t cov_grid = ((blocks_for(n) + 7) / 8) * 8;
    k_grid_cov<K><<<unsigned(cov_grid), kT, 0, st>>>(g, dense, n, k, g_cov_reg, cov6, valid);
    FAR_HIP(hipGetLastError());
    if (dense > 0) {   // a persistent grid of 64 waves per CU over the runs
      k_grid_cov_wave<K><<<256 * 64, 64, 0, st>>>(g, dense, n, k, g_cov_reg, cov6, valid);
      FAR_HIP(hipGetLastError());
    }
    return FAR_OK;
  });
}

far_status_t far_scan_covariances(const float* xyz, int64_t n, double voxel_size, int32_t k,
                                  float* cov6, uint8_t* valid, far_stream_t stream) {
  if (n < 0 || n >= (int64_t(1) << 31) || !(voxel_size > 0.0) || k < 1 || k > 32 ||
      (n > 0 && (!xyz || !cov6 || !valid))) {
    set_error("far_scan_covariances: invalid argument");
    return FAR_E_INVALID;
  }
  if (n == 0) return FAR_OK;
  return scan_cov_impl(xyz, nullptr, 1, n, voxel_size, k, cov6, valid, S(stream),
                       "far_scan_covariances");
}

far_status_t far_scan_covariances_batch(const float* xyz, const int64_t* offsets, int32_t S_,
                                        int64_t n_total, double voxel_size, int32_t k,
                                        float* cov6, uint8_t* valid, far_stream_t stream) {
  if (S_ < 1 || !offsets || n_total < 0 || n_total >= (int64_t(1) << 31) ||
      !(voxel_size > 0.0) || k < 1 || k > 32 || (n_total > 0 && (!xyz || !cov6 || !valid))) {
    set_error("far_scan_covariances_batch: invalid argument");
    return FAR_E_INVALID;
  }
  if (n_total == 0) return FAR_OK;
  return scan_cov_impl(xyz, offsets, S_, n_total, voxel_size, k, cov6, valid, S(stream),
                       "far_scan_covariances_batch");
}

far_status_t far_scan_covariances_batch_order(const float* xyz, const int64_t* offsets,
                                              int32_t S_, int64_t n_total, double voxel_size,
                                              int32_t k, float* cov6, uint8_t* valid,
                                              uint32_t* order, far_stream_t stream) {
  if (S_ < 1 || !offsets || n_total < 0 || n_total >= (int64_t(1) << 31) ||
      !(voxel_size > 0.0) || k < 1 || k > 32 ||
      (n_total > 0 && (!xyz || !cov6 || !valid || !order))) {
    set_error("far_scan_covariances_batch_order: invalid argument");
    return FAR_E_INVALID;
  }
  if (n_total == 0) return FAR_OK;
  return scan_cov_impl(xyz, offsets, S_, n_total, voxel_size, k, cov6, valid, S(stream),
                       "far_scan_covariances_batch_order", order);
}

far_status_t far_scan_covariances_batch_packed(const float* xyz, const int64_t* offsets,
                                               int32_t S_, int64_t n_total, double voxel_size,
                                               int32_t k, float* cov6, uint8_t* valid,
                                               void* packed, far_stream_t stream) {
  if (S_ < 1 || !offsets || n_total < 0 || n_total >= (int64_t(1) << 31) ||
      !(voxel_size > 0.0) || k < 1 || k > 32 ||
      (n_total > 0 && (!xyz || !cov6 || !valid || !packed)) ||
      (reinterpret_cast<uintptr_t>(packed) & 15) != 0) {
    set_error("far_scan_covariances_batch_packed: invalid argument");
    return FAR_E_INVALID;
  }
  if (n_total == 0) return FAR_OK;
  return scan_cov_impl(xyz, offsets, S_, n_total, voxel_size, k, cov6, valid, S(stream),
                       "far_scan_covariances_batch_packed", nullptr, packed);
}

far_status_t far_voxel_downsample(const float* xyz, int64_t n, double v, float* out,
                                  int32_t* keep, int64_t* n_out, far_stream_t stream) {
  if (n_out) *n_out = 0;
  if (!n_out || n < 0 || n >= (int64_t(1) << 31) || !(v > 0.0) || !std::isfinite(v) ||
      (n > 0 && (!xyz || !out)) || (n > 0 && out == xyz)) {
    set_error("far_voxel_downsample: invalid argument");
    return FAR_E_INVALID;
  }
  if (n == 0) return FAR_OK;
  hipStream_t st = S(stream);
  Scratch scr(st);
  const int log2_slots = std::max(10, ceil_log2(2 * n));
  const int64_t n_slots = int64_t(1) << log2_slots;
  Slot* slots;
  uint32_t *slot_of, *cnt;   // cnt: points out of range, points kept
  FAR_TRY(scr.get(&cnt, 2));
  FAR_TRY(scr.get(&slot_of, size_t(n)));
  FAR_TRY(scr.get(&slots, size_t(n_slots)));
  FAR_HIP(hipMemsetAsync(cnt, 0, 2 * sizeof(uint32_t), st));
  FAR_HIP(hipMemsetAsync(slots, 0xFF, size_t(n_slots) * sizeof(Slot), st));
  k_ds_claim<<<blocks_for(n), kT, 0, st>>>(xyz, n, v, slots, uint32_t(n_slots - 1), log2_slots,
                                           slot_of, cnt);
  FAR_HIP(hipGetLastError());
  FAR_TRY(scan_flags(DownsampleFlags{xyz, n, slots, slot_of, cnt, out, keep}, n, cnt + 1, st,
                     scr));
  uint32_t h[2];
  FAR_TRY(fetch(st, h, cnt, sizeof(h)));
  if (h[0] > 0) {
    set_error("far_voxel_downsample: %u points have voxel keys outside [-2^20, 2^20)", h[0]);
    return FAR_E_INVALID;
  }
  *n_out = h[1];
  return FAR_OK;
}

far_status_t far_transform_points(const float* xyz, int64_t n, const double T[16], float* out,
                                  far_stream_t stream) {
  if (n < 0 || !T || (n > 0 && (!xyz || !out))) {
    set_error("far_transform_points: invalid argument");
    return FAR_E_INVALID;
  }
  Rigid R;
  for (int i = 0; i < 12; ++i) {
    R.r[i] = T[i];
    if (!std::isfinite(T[i])) {
      set_error("far_transform_points: non-finite pose");
      return FAR_E_INVALID;
    }
  }
  if (n == 0) return FAR_OK;
  k_transform<<<blocks_for(n), kT, 0, S(stream)>>>(xyz, n, R, out);
  FAR_HIP(hipGetLastError());
  return FAR_OK;
}

far_status_t far_set_covariance_schedule(int32_t dense_threshold) {
  if (dense_threshold < 0) {
    set_error("far_set_covariance_schedule: dense_threshold must be >= 0");
    return FAR_E_INVALID;
  }
  g_dense_threshold = dense_threshold;
  return FAR_OK;
}

far_status_t far_set_covariance_regularisation(int32_t mode) {
  if (mode != FAR_REG_EQ1 && mode != FAR_REG_PLANE) {
    set_error("far_set_covariance_regularisation: unknown mode %d", mode);
    return FAR_E_INVALID;
  }
  g_cov_reg = mode;
  return FAR_OK;
}

far_status_t far_get_covariance_regularisation(int32_t* mode) {
  if (!mode) {
    set_error("far_get_covariance_regularisation: null argument");
    return FAR_E_INVALID;
  }
  *mode = g_cov_reg;
  return FAR_OK;
}

far_status_t far_get_covariance_schedule(int32_t* dense_threshold) {
  if (!dense_threshold) {
    set_error("far_get_covariance_schedule: null argument");
    return FAR_E_INVALID;
  }
  *dense_threshold = g_dense_threshold;
  return FAR_OK;
}

far_status_t far_autotune_covariances(const float* xyz, const int64_t* offsets, int32_t S_,
                                      int64_t n_total, double voxel_size, int32_t k,
                                      float* cov6, uint8_t* valid, int32_t reps, int32_t* best,
                                      double* ms, far_stream_t stream) {
  if (!best || reps < 1 || reps > 100) {
    set_error("far_autotune_covariances: invalid argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  const int32_t saved = g_dense_threshold;
  const int32_t cands[5] = {0, 16, 32, 64, 128};
  double times[5];
  int32_t win = saved;
  double win_ms = -1.0;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  far_status_t rs = FAR_OK;
  hipError_t e;
  if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess)
    rs = hip_fail(e, "far_autotune_covariances setup", __FILE__, __LINE__);
  for (int c = 0; c < 5 && rs == FAR_OK; ++c) {
    g_dense_threshold = cands[c];
    double bestc = 1e300;
    for (int r = 0; r <= reps && rs == FAR_OK; ++r) {
      if ((e = hipEventRecord(e0, st)) != hipSuccess) {
        rs = hip_fail(e, "far_autotune_covariances", __FILE__, __LINE__);
        break;
      }
      rs = far_scan_covariances_batch(xyz, offsets, S_, n_total, voxel_size, k, cov6, valid,
                                      stream);
      if (rs != FAR_OK) break;
      float t = 0.0f;
      if ((e = hipEventRecord(e1, st)) != hipSuccess ||
          (e = hipEventSynchronize(e1)) != hipSuccess ||
          (e = hipEventElapsedTime(&t, e0, e1)) != hipSuccess) {
        rs = hip_fail(e, "far_autotune_covariances timing", __FILE__, __LINE__);
        break;
      }
      if (r > 0 && t < bestc) bestc = t;
    }
    times[c] = bestc;
    if (rs == FAR_OK && (win_ms < 0.0 || bestc < win_ms)) {
      win_ms = bestc;
      win = cands[c];
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (rs != FAR_OK) {
    g_dense_threshold = saved;
    return rs;
  }
  // the threshold in place stays unless a candidate beats it by more than 2 %
  for (int c = 0; c < 5; ++c)
    if (cands[c] == saved && times[c] <= 1.02 * win_ms) win = saved;
  g_dense_threshold = win;
  *best = win;
  if (ms)
    for (int c = 0; c < 5; ++c) ms[c] = times[c];
  return FAR_OK;
}

far_status_t far_asmd_caps(const float* xyz_sensor, const float* xyz_map, int64_t n, double v,
                           int32_t k, int32_t nmax, double r_near, double r_max, int32_t* caps,
                           double* mean_near, far_stream_t stream) {
  if (n < 0 || n >= (int64_t(1) << 31) || !(v > 0.0) || !std::isfinite(v) || k < 1 ||
      nmax < k || nmax > 64 || !(r_near >= 0.0) || !(r_max > 0.0) ||
      (n > 0 && (!xyz_sensor || !xyz_map || !caps))) {
    set_error("far_asmd_caps: invalid argument");
    return FAR_E_INVALID;
  }
  double mean = double(nmax);
  if (n > 0) {
    hipStream_t st = S(stream);
    Scratch scr(st);
    const int set_log2 = std::max(6, ceil_log2(2 * n));
    const int64_t set_n = int64_t(1) << set_log2;
    uint64_t* set;
    uint32_t* counters;
    FAR_TRY(scr.get(&set, size_t(set_n)));
    FAR_TRY(scr.get(&counters, 3));
    {
      TimedScope ts(FAR_TIME_ASMD, st);
      FAR_HIP(hipMemsetAsync(set, 0xFF, size_t(set_n) * sizeof(uint64_t), st));
      FAR_HIP(hipMemsetAsync(counters, 0, 3 * sizeof(uint32_t), st));
      k_asmd_count<<<blocks_for(n), kT, 0, st>>>(xyz_sensor, xyz_map, n, v, r_near * r_near,
                                                 set, uint32_t(set_n - 1), set_log2, counters);
      FAR_HIP(hipGetLastError());
      k_asmd_caps<<<blocks_for(n), kT, 0, st>>>(xyz_sensor, n, counters, r_max, k, nmax, caps);
      FAR_HIP(hipGetLastError());
    }
    uint32_t h[3];
    FAR_TRY(fetch(st, h, counters, sizeof(h)));
    if (h[2] > 0) {
      set_error("far_asmd_caps: %u near points have voxel keys outside [-2^20, 2^20)", h[2]);
      return FAR_E_INVALID;
    }
    if (h[1] > 0) mean = double(h[0]) / double(h[1]);
  }
  if (mean_near) *mean_near = mean;
  return FAR_OK;
}

far_status_t far_map_evict(far_map_t m, const double c[3], double radius, int64_t* n_removed,
                           far_stream_t stream) {
  if (n_removed) *n_removed = 0;
  if (!m || !c || !(radius >= 0.0) || !std::isfinite(c[0]) || !std::isfinite(c[1]) ||
      !std::isfinite(c[2])) {
    set_error("far_map_evict: invalid argument");
    return FAR_E_INVALID;
  }
  const int64_t n = m->n_points;
  hipStream_t st = S(stream);
  const double v = m->p.voxel_size;
  if (n == 0) {
    // only empty voxels can be held: drop them too (the map is rebuilt from
    // its surviving points)
    if (m->n_voxels > 0) {
      FAR_TRY(voxels_reset(m, st));
      FAR_HIP(hipStreamSynchronize(st));
      m->n_voxels = 0;
      m->fine_ok = false;
    }
    return FAR_OK;
  }
  Scratch scr(st);
  const int64_t nv = m->n_voxels;
  const int32_t nmax = m->p.max_pts_per_voxel;
  uint32_t *vkeep, *nvox;
  uint64_t* kkey;
  float* xyz;
  float4* cv;
  int32_t *loc, *kcount, *seg_vox;
  InsertCounts* counts;   // n_seg: voxels kept, n_acc: points kept
  FAR_TRY(scr.get(&counts, 1));
  FAR_TRY(scr.get(&vkeep, size_t(nv)));
  FAR_TRY(scr.get(&nvox, size_t(nv)));
  FAR_TRY(scr.get(&kkey, size_t(nv)));
  FAR_TRY(scr.get(&kcount, size_t(nv)));
  FAR_TRY(scr.get(&seg_vox, size_t(nv)));
  FAR_TRY(scr.get(&xyz, size_t(3 * n)));
  FAR_TRY(scr.get(&cv, size_t(2 * n)));
  FAR_TRY(scr.get(&loc, size_t(n)));
  InsertCounts h;
  {
    TimedScope ts(FAR_TIME_EVICT, st);
    FAR_HIP(hipMemsetAsync(counts, 0, sizeof(InsertCounts), st));
    FAR_TRY(scan_flags(EvictVoxels{m->vox_key, m->vox_count, v, c[0], c[1], c[2],
                                   radius * radius, vkeep, nvox, kkey, kcount,
                                   &counts->leaves},
                       nv, &counts->n_seg, st, scr));
    FAR_TRY(scan_flags(EvictPoints{m->pt_xyz, m->cov, m->pt_loc, m->p.point_capacity, nmax,
                                   vkeep, nvox, xyz, cv, loc, &counts->leaves},
                       n, &counts->n_acc, st, scr));
  }
  FAR_TRY(fetch(st, &h, counts, sizeof(h)));
  const int64_t n_keep = h.n_acc, v_keep = h.n_seg;
  if (n_keep == n) return FAR_OK;
  TimedScope ts2(FAR_TIME_EVICT, st);
  // clear the voxel structures, then store the survivors and rebuild them
  FAR_TRY(voxels_reset(m, st));
  m->n_points = 0;
  m->n_voxels = 0;
  m->fine_ok = false;
  if (n_removed) *n_removed = n - n_keep;
  if (n_keep == 0) {
    ts2.stop();
    FAR_HIP(hipStreamSynchronize(st));
    return FAR_OK;
  }
  k_evict_store<<<blocks_for(n_keep), kT, 0, st>>>(
      xyz, cv, loc, n_keep, m->p.point_capacity, kkey, kcount, v_keep, m->pt_xyz, m->cov,
      m->pt_loc, m->vox_pts, m->vox_cov, m->slots_d, uint32_t(m->slots - 1), m->log2_slots,
      m->vox_key, m->vox_count, m->vox_slot, seg_vox);
  FAR_HIP(hipGetLastError());
  // every slot changed: all rows, ghosts and certificates again
  FAR_TRY(links_update(m, v_keep, m->voxel_cap, counts, seg_vox, nullptr, nullptr, st));
  FAR_TRY(certs_build(m, v_keep, n_keep, nullptr, 0, counts, nullptr, 0, 0, st, scr));
  ts2.stop();
  FAR_TRY(fetch(st, &h, counts, sizeof(h)));
  ghosts_take(m, h.ghosts);
  m->n_points = n_keep;
  m->n_voxels = v_keep;
  return FAR_OK;
}

far_status_t far_map_stats(far_map_t m, far_map_stats_t* out, far_stream_t stream) {
  if (!m || !out) {
    set_error("far_map_stats: null argument");
    return FAR_E_INVALID;
  }
  hipStream_t st = S(stream);
  Scratch scr(st);
  unsigned long long* sum;
  uint32_t* maxp;
  FAR_TRY(scr.get(&sum, 1));
  FAR_TRY(scr.get(&maxp, 1));
  FAR_HIP(hipMemsetAsync(sum, 0, sizeof(unsigned long long), st));
  FAR_HIP(hipMemsetAsync(maxp, 0, sizeof(uint32_t), st));
  const unsigned nb = unsigned(std::min<int64_t>(blocks_for(m->slots), 2 * device_cu_count()));
  k_probe_stats<<<nb, kT, 0, st>>>(m->slots_d, m->slots,
                                                     uint32_t(m->slots - 1), m->log2_slots,
                                                     sum, maxp);
  FAR_HIP(hipGetLastError());
  unsigned long long h_sum = 0;
  uint32_t h_max = 0;
  FAR_TRY(fetch(st, &h_sum, sum, sizeof(h_sum), &h_max, maxp, sizeof(h_max)));
  out->n_points = m->n_points;
  out->n_voxels = m->n_voxels;
  out->table_slots = m->slots;
  out->load_factor = double(m->n_voxels) / double(m->slots);
  out->mean_probe = m->n_voxels ? double(h_sum) / double(m->n_voxels) : 0.0;
  out->max_probe = int32_t(h_max);
  out->max_pts_per_voxel = m->p.max_pts_per_voxel;
  out->voxel_size = m->p.voxel_size;
  out->min_spacing = m->dmin;
  out->bytes_device = m->bytes;
  return FAR_OK;
}

far_status_t far_map_export(far_map_t m, float* xyz, float* cov6, uint8_t* valid,
                            int64_t capacity, int64_t* n_out, far_stream_t stream) {
  if (!m || !n_out) {
    set_error("far_map_export: null argument");
    return FAR_E_INVALID;
  }
  *n_out = m->n_points;
  if (m->n_points > capacity) {
    set_error("far_map_export: map holds %lld points, buffers hold %lld",
              (long long)m->n_points, (long long)capacity);
    return FAR_E_CAPACITY;
  }
  if (m->n_points == 0) return FAR_OK;
  hipStream_t st = S(stream);
  k_export<<<blocks_for(m->n_points), kT, 0, st>>>(m->cov, m->pt_xyz, m->p.point_capacity,
                                                   m->n_points, xyz, cov6, valid);
  FAR_HIP(hipGetLastError());
  FAR_HIP(hipStreamSynchronize(st));
  return FAR_OK;
}

}  // extern "C"
