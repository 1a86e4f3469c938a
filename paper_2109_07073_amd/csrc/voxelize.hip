// Voxel-map construction on gfx950 (Sec. III-A, VGICP voxel data association).
//
// Each voxel carries the mean of its points and the mean of their
// covariances (the VGICP aggregation of point distributions), accumulated in
// FP64 in point order and rounded once to FP32.  Voxels are stored densely,
// brick after brick (bricks of 4 x 4 x 4 voxels), and found through an
// open-addressed table of brick records holding each brick's occupancy mask.
//
// Clouds of at most kGroupMaxPoints points are grouped by brick in a hash
// table (group.hpp): six launches and one wait of the host.
// Larger clouds, and the few whose bricks do not fit the table or that put
// more than kVoxelMax points in one voxel, are sorted instead: keys -> radix
// sort of (key, point index) -> segment heads -> scan -> segment starts ->
// [host sync: voxel count] -> per voxel its brick-major sort key -> radix sort
// of (brick key and bit, voxel ordinal) -> brick heads -> scan -> brick starts
// -> [host sync: brick count] -> brick table insertion and FP64 voxel sums.
// Both give the same map.  This runs once per cloud, off the per-iteration
// path.

#include <algorithm>
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "group.hpp"

namespace vgicp {

// The voxel key of point i (zeros on an axis it is refused on) and the error
// bits of its coordinates.
__device__ __forceinline__ uint32_t point_key(const float *__restrict__ xyz, int64_t n, int64_t i,
                                              float s, int32_t k[3]) {
  uint32_t bad = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float x = xyz[a * n + i];
    const float v = x * s;
    if (!isfinite(x)) {
      bad |= kErrNonFinite;
      k[a] = 0;
    } else if (!(v >= -kKeyLimitF && v < kKeyLimitF)) {
      bad |= kErrRange;
      k[a] = 0;
    } else {
      k[a] = int32_t(floorf(v));
    }
  }
  return bad;
}

__global__ void __launch_bounds__(256)
k_voxel_keys(const float *__restrict__ xyz, int64_t n, float s, uint64_t *__restrict__ keys,
             uint32_t *__restrict__ idx, uint32_t *__restrict__ err) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int32_t k[3];
  const uint32_t bad = point_key(xyz, n, i, s, k);
  if (bad) atomicOr(err, bad);
  keys[i] = pack_key(k[0], k[1], k[2]);
  idx[i] = uint32_t(i);
}

__global__ void __launch_bounds__(256)
k_segment_heads(const uint64_t *__restrict__ sorted_keys, int64_t n, uint32_t *__restrict__ head) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  head[i] = (i == 0 || sorted_keys[i] != sorted_keys[i - 1]) ? 1u : 0u;
}

// What the host waits for in the sorted construction (pinned): the points'
// error bits and the number of segments; `seq` is written last.
struct SegmentCounts {
  uint32_t err, n, seq;
};
static_assert(sizeof(SegmentCounts) <= kCountsWord * sizeof(uint32_t), "words of their own");

// ord1[i] is the inclusive scan of head: the 1-based ordinal of element i.  err
// (may be NULL) holds the points' error bits.
__global__ void __launch_bounds__(256)
k_segment_starts(const uint32_t *__restrict__ head, const uint32_t *__restrict__ ord1, int64_t n,
                 uint32_t *__restrict__ seg, const uint32_t *__restrict__ err, SegmentCounts *host,
                 uint32_t seq) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (head[i]) seg[ord1[i] - 1] = uint32_t(i);
  if (i == n - 1) {
    seg[ord1[i]] = uint32_t(n);
    host->err = err ? *err : 0u;
    host->n = ord1[i];
    __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Record i of an empty table, and word i of its bitset.
__device__ __forceinline__ void fill_empty(int64_t i, BrickRecord *__restrict__ bricks,
                                           int64_t cap, uint32_t *__restrict__ occ,
                                           uint32_t occ_words) {
  if (i < cap) {
    BrickRecord r;
    r.key = kEmptyKey;
    r.mask = 0;
    r.base = 0;
    r.pad[0] = r.pad[1] = r.pad[2] = 0;
    bricks[i] = r;
  }
  if (i < int64_t(occ_words)) occ[i] = 0u;
}

__global__ void __launch_bounds__(256)
k_fill_empty(BrickRecord *__restrict__ bricks, int64_t cap, uint32_t *__restrict__ occ,
             uint32_t occ_words) {
  fill_empty(int64_t(blockIdx.x) * blockDim.x + threadIdx.x, bricks, cap, occ, occ_words);
}

// Per voxel (in lexicographic order): its packed key and its brick-major sort
// key (brick key above the 6-bit position in the brick).
__global__ void __launch_bounds__(256)
k_brick_sortkeys(const uint64_t *__restrict__ sorted_keys, const uint32_t *__restrict__ seg,
                 int64_t n_voxels, uint64_t *__restrict__ vkey, uint64_t *__restrict__ bsort,
                 uint32_t *__restrict__ vord) {
  const int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (v >= n_voxels) return;
  const uint64_t key = sorted_keys[seg[v]];
  const int32_t kx = key_field(key, 0), ky = key_field(key, 1), kz = key_field(key, 2);
  vkey[v] = key;
  bsort[v] = brick_sort_key(kx, ky, kz);
  vord[v] = uint32_t(v);
}

__global__ void __launch_bounds__(256)
k_brick_heads(const uint64_t *__restrict__ bsort, int64_t n_voxels, uint32_t *__restrict__ head) {
  const int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (d >= n_voxels) return;
  head[d] = (d == 0 || (bsort[d] >> 6) != (bsort[d - 1] >> 6)) ? 1u : 0u;
}

// Linear-probing insertion of a brick's record (`brick` in key order) and its
// occupancy bit.
__device__ __forceinline__ void insert_record(uint64_t brick, uint64_t mask, uint32_t base,
                                              BrickRecord *__restrict__ bricks, uint32_t log2cap,
                                              uint32_t *__restrict__ occ, uint32_t occ_mask) {
  const uint32_t cmask = (1u << log2cap) - 1u;
  const int32_t bx = brick_coord(brick, 0), by = brick_coord(brick, 1), bz = brick_coord(brick, 2);
  const uint64_t key = record_key(bx, by, bz);
  uint32_t h = brick_slot(bx, by, bz, log2cap);
  // the records of one position in the lines: cap / kProbeStep of them
  for (uint32_t probe = 0; probe <= (cmask >> 2); ++probe) {
    const unsigned long long prev =
        atomicCAS(reinterpret_cast<unsigned long long *>(&bricks[h].key),
                  (unsigned long long)kEmptyKey, (unsigned long long)key);
    if (prev == kEmptyKey) break;
    h = (h + kProbeStep) & cmask;
  }
  bricks[h].mask = mask;
  bricks[h].base = base;
  const uint32_t bit = h & occ_mask;
  atomicOr(&occ[bit >> 5], 1u << (bit & 31u));
}

// One thread per brick: its occupancy mask from its voxels' bits, then its
// record.
__global__ void __launch_bounds__(256)
k_build_bricks(const uint64_t *__restrict__ bsort, const uint32_t *__restrict__ bstart,
               int64_t n_bricks, int64_t n_voxels, BrickRecord *__restrict__ bricks,
               uint32_t log2cap, uint32_t *__restrict__ occ, uint32_t occ_mask) {
  const int64_t b = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (b >= n_bricks) return;
  const uint32_t d0 = bstart[b];
  const uint32_t d1 = (b + 1 < n_bricks) ? bstart[b + 1] : uint32_t(n_voxels);
  uint64_t mask = 0;
  for (uint32_t d = d0; d < d1; ++d) mask |= 1ull << (bsort[d] & 63u);
  insert_record(brick_key_of_sort_key(bsort[d0]), mask, d0, bricks, log2cap, occ, occ_mask);
}

// Coordinates and covariance of point p.
__device__ __forceinline__ void gather_point(const float *__restrict__ xyz,
                                             const float *__restrict__ cov, uint32_t n, uint32_t p,
                                             float v[9]) {
  v[0] = xyz[p], v[1] = xyz[uint64_t(n) + p], v[2] = xyz[2ull * n + p];
  const float2 *c = reinterpret_cast<const float2 *>(cov + 6ull * p);
#pragma unroll
  for (int a = 0; a < 3; ++a) v[3 + 2 * a] = c[a].x, v[4 + 2 * a] = c[a].y;
}

// One thread per voxel, by dense (brick-major) position d: sequential FP64
// sums over the voxel's points in point order, one FP64 division, one
// rounding to FP32.  Bound by the fullest voxels, whose points are gathered one
// dependent pair of loads after the other: kPayloadPoints are in flight at once.
constexpr uint32_t kPayloadPoints = 8;
__global__ void __launch_bounds__(256)
k_build_payload(const float *__restrict__ xyz, const float *__restrict__ cov, int64_t n,
                const uint32_t *__restrict__ sorted_idx, const uint32_t *__restrict__ seg,
                const uint32_t *__restrict__ vord, const uint64_t *__restrict__ vkey,
                int64_t n_voxels, VoxelStats *__restrict__ stats,
                VoxelInfo *__restrict__ info) {
  const int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (d >= n_voxels) return;
  const uint32_t v = vord[d];
  const uint32_t b = seg[v], e = seg[v + 1];
  double sm[3] = {0.0, 0.0, 0.0};
  double sc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  auto add = [&](const float *p) {
#pragma unroll
    for (int a = 0; a < 3; ++a) sm[a] += double(p[a]);
#pragma unroll
    for (int a = 0; a < 6; ++a) sc[a] += double(p[3 + a]);
  };
  uint32_t j = b;
  for (; j + kPayloadPoints <= e; j += kPayloadPoints) {
    uint32_t p[kPayloadPoints];
    float x[kPayloadPoints][9];
#pragma unroll
    for (uint32_t u = 0; u < kPayloadPoints; ++u) p[u] = sorted_idx[j + u];
#pragma unroll
    for (uint32_t u = 0; u < kPayloadPoints; ++u) gather_point(xyz, cov, uint32_t(n), p[u], x[u]);
#pragma unroll
    for (uint32_t u = 0; u < kPayloadPoints; ++u) add(x[u]);
  }
  for (; j < e; ++j) {
    float x[9];
    gather_point(xyz, cov, uint32_t(n), sorted_idx[j], x);
    add(x);
  }
  const double cnt = double(e - b);
  VoxelStats st;
#pragma unroll
  for (int a = 0; a < 3; ++a) st.mean[a] = float(sm[a] / cnt);
#pragma unroll
  for (int a = 0; a < 6; ++a) st.cov[a] = float(sc[a] / cnt);
  stats[d] = st;
  VoxelInfo in;
  in.key = vkey[v];
  in.ordinal = int32_t(v);
  in.count = int32_t(e - b);
  info[d] = in;
}

// ---------------------------------------------------------------- grouped construction
// group.hpp's steps with cells = voxels, and then
//   number   per brick: its rank and the voxels before it (against every
//            other brick), so the dense position of its voxels.  Its first
//            thread hands the counts to the host, which meanwhile allocates
//            the map (the same launch scatters the points);
//   finish   per voxel: its points put back in point order, gathered, and
//            summed in that order in FP64; per brick: the lexicographic
//            ordinals of its voxels; the table's empty records;
//   records  per brick: its record.
// A call on 20,011 returns takes 46 us (185 us by sorting), on a merged submap
// of 320,000 points at 0.5 m 84 us (480 us; 7 us more with four other bricks in a
// lane's flight while numbering and each brick's own loads one after the other).
// What can tell that a cloud does not fit is the insert, so a cloud that is
// sorted in the end pays for it, most where it has too many bricks: 320,000
// points at 0.05 m (60,600) take 505 us, sorted at once 400, and 2^20 at 0.1 m
// (38,400) 620 and 530.  From about 18,000 bricks at 32,768 slots on it is one or
// the other; there grouping takes 280 us (320,000 points at 0.1 m) and sorting
// 365.
constexpr uint32_t kVoxelMax = 4096;  // points of a voxel at most: they are ordered in LDS
constexpr uint32_t kNumberBlocks = 512;
constexpr uint32_t kNumberBricks = 4;  // bricks a wave numbers at once
constexpr uint32_t kNumberLoads = 8;   // other bricks a lane has in flight

// What the host waits for (pinned); `seq` is written last.
struct GroupCounts {
  uint32_t err, n_voxels, n_bricks, n_heavy, max_count, seq;
};

struct VoxelGroup : Group {
  uint64_t *skey, *smask;  // [bricks] in key order
  uint32_t *sbase;         // voxels in earlier bricks
  uint2 *sseg;             // the bricks with the same x field
  uint2 *vox;              // [voxels] start in the list, points
  uint32_t *heavy;         // voxels of more than kLightMax points
};

// The brick and cell of a point, as group.hpp asks for them.
struct VoxelOfPoint {
  const float *xyz;
  uint32_t n;
  float s;
  __device__ uint32_t operator()(uint32_t i, uint64_t &brick, uint32_t &cell) const {
    int32_t k[3];
    const uint32_t bad = point_key(xyz, n, i, s, k);
    brick = brick_key(brick_field(k[0]), brick_field(k[1]), brick_field(k[2]));
    cell = brick_bit(k[0], k[1], k[2]);
    return bad;
  }
};

__global__ void __launch_bounds__(256)
k_group_clear(VoxelGroup g, uint32_t *__restrict__ err_word) {
  group_clear(g, blockIdx.x);
  if (blockIdx.x == 0 && threadIdx.x == 0) *err_word = 0;  // for a sorted construction
}

__global__ void __launch_bounds__(256)
k_group_insert(VoxelGroup g, VoxelOfPoint key) {
  group_insert(g, blockIdx.x, key.n, kVoxelMax, key);
}

__global__ void __launch_bounds__(kCompactThreads)
k_group_compact(VoxelGroup g) {
  group_compact(g, blockIdx.x);
}

// Blocks [0, number_blocks): bricks; the others: points.
__global__ void __launch_bounds__(256)
k_group_number(VoxelGroup g, uint32_t number_blocks, uint32_t n, GroupCounts *host,
               uint32_t seq) {
  if (blockIdx.x >= number_blocks) {
    group_scatter(g, (blockIdx.x - number_blocks) * 256 + threadIdx.x, n);
    return;
  }
  const uint64_t totals = g.hdr->totals;
  const uint32_t nb = uint32_t(totals >> kBricksShift);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    host->err = g.hdr->err;
    host->n_voxels = uint32_t(totals >> kCellsShift) & kTotalsMask;
    host->n_bricks = nb;
    host->n_heavy = g.hdr->n_heavy;
    host->max_count = g.hdr->max_count;
    __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (uint32_t i0 = w * kNumberBricks; i0 < nb; i0 += number_blocks * 4 * kNumberBricks) {
    uint64_t key[kNumberBricks], mask[kNumberBricks];
    uint32_t slot[kNumberBricks], rank[kNumberBricks], base[kNumberBricks], lt[kNumberBricks],
        le[kNumberBricks];
#pragma unroll
    for (uint32_t q = 0; q < kNumberBricks; ++q) {
      const uint32_t i = min(i0 + q, nb - 1);
      key[q] = g.bkey[i];
      mask[q] = g.bmask[i];
      slot[q] = g.bslot[i];
      rank[q] = base[q] = lt[q] = le[q] = 0;
    }
    for (uint32_t j0 = lane; j0 < nb; j0 += 64 * kNumberLoads) {
      uint64_t k[kNumberLoads], m[kNumberLoads];
#pragma unroll
      for (uint32_t u = 0; u < kNumberLoads; ++u) {
        const uint32_t j = min(j0 + 64 * u, nb - 1);
        k[u] = g.bkey[j];
        m[u] = g.bmask[j];
      }
#pragma unroll
      for (uint32_t u = 0; u < kNumberLoads; ++u) {
        if (j0 + 64 * u >= nb) k[u] = ~0ull;  // after every brick
        const uint32_t pop = uint32_t(__popcll(m[u]));
        const uint32_t x = uint32_t(k[u] >> (2 * kBrickBits));
#pragma unroll
        for (uint32_t q = 0; q < kNumberBricks; ++q) {
          const uint32_t xq = uint32_t(key[q] >> (2 * kBrickBits));
          rank[q] += k[u] < key[q] ? 1u : 0u;
          base[q] += k[u] < key[q] ? pop : 0u;
          lt[q] += x < xq ? 1u : 0u;
          le[q] += x <= xq ? 1u : 0u;
        }
      }
    }
    uint32_t c[kNumberBricks], at[kNumberBricks];
#pragma unroll
    for (uint32_t q = 0; q < kNumberBricks; ++q) {
      c[q] = at[q] = 0;
      if ((mask[q] >> lane) & 1ull) {
        const uint32_t at64 = (slot[q] << 6) | lane;
        c[q] = g.count[at64];
        at[q] = g.first[slot[q]] + g.rel[at64];
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kNumberBricks; ++q) {
      if (i0 + q >= nb) break;
      const uint32_t r = wave_total(rank[q]), b = wave_total(base[q]);
      const uint32_t s0 = wave_total(lt[q]), s1 = wave_total(le[q]);
      if (lane == 0) {
        g.skey[r] = key[q];
        g.smask[r] = mask[q];
        g.sbase[r] = b;
        g.sseg[r] = make_uint2(s0, s1);
      }
      if ((mask[q] >> lane) & 1ull) {
        const uint32_t d = b + uint32_t(__popcll(mask[q] & ((1ull << lane) - 1ull)));
        g.vox[d] = make_uint2(at[q], c[q]);
        if (c[q] > kLightMax) g.heavy[atomicAdd(&g.hdr->heavy_at, 1u)] = d;
      }
    }
  }
}

// Adds m values to acc one after the other.
__device__ __forceinline__ double add_in_order(double acc, const float *v, uint32_t m) {
  uint32_t r = 0;
  for (; r + 8 <= m; r += 8) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = v[r + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += double(x[u]);
  }
  for (; r < m; ++r) acc += double(v[r]);
  return acc;
}

constexpr uint32_t kGatherStride = 260;  // lists after nine rows are 16-byte aligned
constexpr uint32_t kLightStride = kLightMax + 1;

// Entries of the sorted list of a voxel of m points.
__host__ __device__ inline uint32_t list_size(uint32_t m) {
  uint32_t m2 = 128;
  while (m2 < m) m2 <<= 1;
  return m2;
}

// LDS of a finish block: the gathered points of a heavy voxel and its list
// (the fullest voxel's, so that blocks take no more than they need), or the
// points of four light ones.
static size_t finish_lds(uint32_t max_count) {
  if (max_count <= kLightMax) return 4 * 9 * kLightStride * sizeof(float);
  return (9 * kGatherStride + list_size(max_count)) * sizeof(float);
}
static_assert(9 * kGatherStride % 4 == 0, "aligned lists");
static_assert(9 * kGatherStride + 128 >= 4 * 9 * kLightStride, "light points fit a heavy block");

// A voxel of more than kLightMax points, by one block.  Up to 256 points take
// the place that counting the smaller indices gives them, while they are
// gathered; more are sorted in LDS first, then gathered 256 at a time while
// nine lanes of the first wave add the previous ones.
__device__ void finish_heavy(float *lds, const VoxelGroup &g, uint32_t d,
                             const float *__restrict__ xyz, const float *__restrict__ cov,
                             uint32_t n, float *__restrict__ stats) {
  const uint32_t tid = threadIdx.x;
  const uint2 vx = g.vox[d];
  const uint32_t m = vx.y;
  const uint32_t m2 = list_size(m);
  uint32_t *idx = reinterpret_cast<uint32_t *>(lds + 9 * kGatherStride);
  for (uint32_t i = tid; i < m2; i += 256) idx[i] = i < m ? g.list[vx.x + i] : 0xffffffffu;
  __syncthreads();
  double acc = 0.0;
  if (m <= 256) {
    float v[9];
    const uint32_t p = tid < m ? idx[tid] : 0u;
    if (tid < m) gather_point(xyz, cov, n, p, v);
    uint32_t rank = 0;
    for (uint32_t l = 0; l < m2; l += 4) {
      const uint4 o = *reinterpret_cast<const uint4 *>(idx + l);
      rank += (o.x < p ? 1u : 0u) + (o.y < p ? 1u : 0u) + (o.z < p ? 1u : 0u) + (o.w < p ? 1u : 0u);
    }
    if (tid < m) {
#pragma unroll
      for (uint32_t a = 0; a < 9; ++a) lds[a * kGatherStride + rank] = v[a];
    }
    __syncthreads();
    if (tid < 9) acc = add_in_order(0.0, lds + tid * kGatherStride, m);
  } else {
    for (uint32_t k = 2; k <= m2; k <<= 1)
      for (uint32_t j = k >> 1; j > 0; j >>= 1) {
        for (uint32_t t = tid; t < m2 / 2; t += 256) {
          const uint32_t lo = 2 * t - (t & (j - 1)), hi = lo + j;
          const uint32_t a = idx[lo], b = idx[hi];
          if ((a > b) == ((lo & k) == 0)) {
            idx[lo] = b;
            idx[hi] = a;
          }
        }
        __syncthreads();
      }
    for (uint32_t c0 = 0; c0 < m; c0 += 256) {
      float v[9];
      if (c0 + tid < m) gather_point(xyz, cov, n, idx[c0 + tid], v);
      __syncthreads();  // the previous points have been added
      if (c0 + tid < m) {
#pragma unroll
        for (uint32_t a = 0; a < 9; ++a) lds[a * kGatherStride + tid] = v[a];
      }
      __syncthreads();
      if (tid < 9) acc = add_in_order(acc, lds + tid * kGatherStride, min(m - c0, 256u));
    }
  }
  if (tid < 9) stats[9ull * d + tid] = float(acc / double(m));
}

// A voxel of at most kLightMax points, by one wave.
__device__ __forceinline__ void finish_light(float *lds, const VoxelGroup &g, uint32_t d,
                                             const float *__restrict__ xyz,
                                             const float *__restrict__ cov, uint32_t n,
                                             float *__restrict__ stats) {
  const uint32_t lane = threadIdx.x & 63;
  const uint2 vx = g.vox[d];
  const uint32_t m = __builtin_amdgcn_readfirstlane(vx.y);
  if (m > kLightMax) return;
  uint32_t p = 0, rank = 0;
  float v[9];
  if (lane < m) {
    p = g.list[vx.x + lane];
    gather_point(xyz, cov, n, p, v);
  }
  for (uint32_t l = 0; l < m; ++l)
    rank += uint32_t(__builtin_amdgcn_readlane(int(p), int(l))) < p ? 1u : 0u;
  if (lane < m) {
#pragma unroll
    for (uint32_t a = 0; a < 9; ++a) lds[a * kLightStride + rank] = v[a];
  }
  __builtin_amdgcn_wave_barrier();
  if (lane < 9) stats[9ull * d + lane] = float(add_in_order(0.0, lds + lane * kLightStride, m) / double(m));
}

// The voxels of brick s (in key order), a lane per voxel of the brick.  A
// voxel's ordinal counts the voxels whose key comes first, axis after axis:
// every voxel of the bricks with a smaller x field, and in the bricks with the
// same x field (neighbours in key order) those its own bits select.
__device__ __forceinline__ void finish_brick(const VoxelGroup &g, uint32_t s,
                                             VoxelInfo *__restrict__ info) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t key = g.skey[s], mask = g.smask[s];
  const uint2 seg = g.sseg[s];
  // bits of a brick whose position on an axis (its bits h1 h0) equals this
  // lane's, and is less
  auto axis = [&](uint32_t b1, uint32_t b0, uint64_t h1, uint64_t h0, uint64_t &eq, uint64_t &lt) {
    const bool v1 = (lane >> b1) & 1u, v0 = (lane >> b0) & 1u;
    const uint64_t e1 = v1 ? h1 : ~h1;
    eq = e1 & (v0 ? h0 : ~h0);
    lt = (v1 ? ~h1 : 0ull) | (v0 ? e1 & ~h0 : 0ull);
  };
  uint64_t xeq, xlt, yeq, ylt, zeq, zlt;
  axis(5, 2, 0xffffffff00000000ull, 0xf0f0f0f0f0f0f0f0ull, xeq, xlt);
  axis(4, 1, 0xffff0000ffff0000ull, 0xccccccccccccccccull, yeq, ylt);
  axis(3, 0, 0xff00ff00ff00ff00ull, 0xaaaaaaaaaaaaaaaaull, zeq, zlt);
  (void)zeq;
  const uint32_t fmask = (1u << kBrickBits) - 1u;
  const uint32_t y = uint32_t(key >> kBrickBits) & fmask, z = uint32_t(key) & fmask;
  uint32_t ordinal = g.sbase[seg.x];
  for (uint32_t j0 = seg.x; j0 < seg.y; j0 += 64) {
    const uint32_t j = min(j0 + lane, seg.y - 1);
    const uint64_t kj = g.skey[j], mj = g.smask[j];
    const uint32_t cnt = min(seg.y - j0, 64u);
    for (uint32_t l = 0; l < cnt; ++l) {
      const uint32_t klo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(kj)), int(l)));
      const uint32_t khi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(kj >> 32)), int(l)));
      const uint32_t mlo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(mj)), int(l)));
      const uint32_t mhi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(mj >> 32)), int(l)));
      const uint64_t k = (uint64_t(khi) << 32) | klo;
      const uint32_t yj = uint32_t(k >> kBrickBits) & fmask, zj = uint32_t(k) & fmask;
      uint64_t sel = xlt;
      if (yj < y) {
        sel |= xeq;
      } else if (yj == y) {
        sel |= xeq & (ylt | (zj < z ? yeq : zj == z ? (yeq & zlt) : 0ull));
      }
      ordinal += uint32_t(__popcll(sel & ((uint64_t(mhi) << 32) | mlo)));
    }
  }
  if ((mask >> lane) & 1ull) {
    const uint32_t d = g.sbase[s] + uint32_t(__popcll(mask & ((1ull << lane) - 1ull)));
    const int32_t x4 = (int32_t(uint32_t(key >> (2 * kBrickBits))) - kBrickBias) * 4;
    const int32_t y4 = (int32_t(y) - kBrickBias) * 4, z4 = (int32_t(z) - kBrickBias) * 4;
    const int32_t a = int32_t((lane >> 4) & 2u) | int32_t((lane >> 2) & 1u);
    const int32_t b = int32_t((lane >> 3) & 2u) | int32_t((lane >> 1) & 1u);
    const int32_t c = int32_t((lane >> 2) & 2u) | int32_t(lane & 1u);
    VoxelInfo in;
    in.key = pack_key(x4 + a, y4 + b, z4 + c);
    in.ordinal = int32_t(ordinal);
    in.count = int32_t(g.vox[d].y);
    info[d] = in;
  }
}

// Blocks: one per heavy voxel (they take longest), then fill_blocks empty the
// table, then four bricks a block, then four light voxels a block.
__global__ void __launch_bounds__(256)
k_group_finish(VoxelGroup g, uint32_t n_bricks, uint32_t n_voxels, uint32_t n_heavy,
               uint32_t fill_blocks, const float *__restrict__ xyz,
               const float *__restrict__ cov, uint32_t n,
               BrickRecord *__restrict__ bricks, int64_t cap, uint32_t *__restrict__ occ,
               uint32_t occ_words, VoxelStats *__restrict__ stats, VoxelInfo *__restrict__ info) {
  extern __shared__ float lds[];
  uint32_t blk = blockIdx.x;
  const uint32_t wave = threadIdx.x >> 6;
  float *st = reinterpret_cast<float *>(stats);
  if (blk < n_heavy) {
    finish_heavy(lds, g, g.heavy[blk], xyz, cov, n, st);
    return;
  }
  blk -= n_heavy;
  if (blk < fill_blocks) {
    fill_empty(int64_t(blk) * 256 + threadIdx.x, bricks, cap, occ, occ_words);
    return;
  }
  blk -= fill_blocks;
  const uint32_t brick_blocks = (n_bricks + 3) / 4;
  if (blk < brick_blocks) {
    const uint32_t s = __builtin_amdgcn_readfirstlane(blk * 4 + wave);
    if (s < n_bricks) finish_brick(g, s, info);
    return;
  }
  const uint32_t d = __builtin_amdgcn_readfirstlane((blk - brick_blocks) * 4 + wave);
  if (d < n_voxels) finish_light(lds + wave * 9 * kLightStride, g, d, xyz, cov, n, st);
}

__global__ void __launch_bounds__(256)
k_group_records(VoxelGroup g, uint32_t n_bricks, BrickRecord *__restrict__ bricks, uint32_t log2cap,
                uint32_t *__restrict__ occ, uint32_t occ_mask, uint32_t *host, uint32_t seq) {
  const uint32_t s = blockIdx.x * 256 + threadIdx.x, at = min(s, n_bricks - 1);
  const uint64_t key = g.skey[at], mask = g.smask[at];
  const uint32_t base = g.sbase[at];
  // The last block to have read the workspace says so.  (Every wave has its
  // values before the barrier; nothing written is to be seen with the word, so
  // it needs no release.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0 && atomicAdd(&g.hdr->done, 1u) == gridDim.x - 1)
    __hip_atomic_store(host, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (s < n_bricks) insert_record(key, mask, base, bricks, log2cap, occ, occ_mask);
}

__global__ void __launch_bounds__(256)
k_export(const VoxelStats *__restrict__ stats, const VoxelInfo *__restrict__ info,
         int64_t n_voxels, int32_t *__restrict__ keys, float *__restrict__ mean,
         float *__restrict__ cov, int32_t *__restrict__ count) {
  const int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (d >= n_voxels) return;
  const VoxelStats s = stats[d];
  const VoxelInfo in = info[d];
  const int64_t o = in.ordinal;
  if (keys) {
#pragma unroll
    for (int a = 0; a < 3; ++a) keys[3 * o + a] = key_field(in.key, a);
  }
  if (mean) {
#pragma unroll
    for (int a = 0; a < 3; ++a) mean[3 * o + a] = s.mean[a];
  }
  if (cov) {
#pragma unroll
    for (int a = 0; a < 6; ++a) cov[6 * o + a] = s.cov[a];
  }
  if (count) count[o] = in.count;
}

static inline unsigned grid_for(int64_t n, int block = 256) {
  return unsigned((n + block - 1) / block);
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Scratch layout for n points; returns total bytes (rocPRIM temp included).
// After the point sort, keys_in, idx_in, head, ord1 and spare are reused for
// the per-voxel arrays (V <= n): vkey, vord_in, bhead, bord1, vord_out;
// bsort_in/out hold the brick-major sort keys and bstart the brick starts.
struct VoxScratch {
  uint64_t *keys_in, *keys_out, *bsort_in, *bsort_out;
  uint32_t *idx_in, *idx_out, *head, *ord1, *spare, *seg, *bstart;
  void *temp;
  size_t temp_bytes;
};

static hipError_t plan_scratch(int64_t n, hipStream_t stream, size_t *total, size_t *sort_bytes,
                               size_t *scan_bytes) {
  size_t sb = 0, cb = 0;
  hipError_t err = rocprim::radix_sort_pairs(nullptr, sb, (uint64_t *)nullptr, (uint64_t *)nullptr,
                                             (uint32_t *)nullptr, (uint32_t *)nullptr, size_t(n), 0,
                                             63, stream);
  if (err != hipSuccess) return err;
  err = rocprim::inclusive_scan(nullptr, cb, (uint32_t *)nullptr, (uint32_t *)nullptr, size_t(n),
                                rocprim::plus<uint32_t>(), stream);
  if (err != hipSuccess) return err;
  const size_t nn = size_t(n);
  *total = 4 * align256(8 * nn) + 5 * align256(4 * nn) + 2 * align256(4 * (nn + 1)) +
           align256(std::max(sb, cb));
  *sort_bytes = sb;
  *scan_bytes = cb;
  return hipSuccess;
}

static VoxScratch carve(void *base, int64_t n, size_t temp_bytes) {
  char *p = static_cast<char *>(base);
  const size_t nn = size_t(n);
  VoxScratch s;
  s.keys_in = reinterpret_cast<uint64_t *>(p);
  p += align256(8 * nn);
  s.keys_out = reinterpret_cast<uint64_t *>(p);
  p += align256(8 * nn);
  s.bsort_in = reinterpret_cast<uint64_t *>(p);
  p += align256(8 * nn);
  s.bsort_out = reinterpret_cast<uint64_t *>(p);
  p += align256(8 * nn);
  s.idx_in = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * nn);
  s.idx_out = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * nn);
  s.head = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * nn);
  s.ord1 = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * nn);
  s.spare = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * nn);
  s.seg = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * (nn + 1));
  s.bstart = reinterpret_cast<uint32_t *>(p);
  p += align256(4 * (nn + 1));
  s.temp = p;
  s.temp_bytes = temp_bytes;
  return s;
}

// Host driver used by vgicp_voxelize.  Returns a status code and fills *map.
int voxelize_impl(vgicp_ctx ctx, const vgicp_cloud *cloud, double resolution, vgicp_map *out,
                  std::string &msg);

}  // namespace vgicp

// ---------------------------------------------------------------------------

#define HIP_TRY(expr)                                                         \
  do {                                                                        \
    hipError_t _e = (expr);                                                   \
    if (_e != hipSuccess) {                                                   \
      msg = std::string(#expr) + ": " + hipGetErrorString(_e);                \
      return _e == hipErrorOutOfMemory ? VGICP_ENOMEM : VGICP_EHIP;           \
    }                                                                         \
  } while (0)

namespace vgicp {

hipError_t claim_scratch(vgicp_ctx ctx) {
  if (!ctx->stream_set) return hipSuccess;
  const uint32_t *word = ctx->host_pinned + kScratchWord;
  auto done = [&] { return __atomic_load_n(word, __ATOMIC_ACQUIRE) == ctx->scratch_seq; };
  if (ctx->scratch_left == kScratchWordFollows) {
    for (int spin = 0; spin < 20000 && !done(); ++spin) __builtin_ia32_pause();
    if (done()) ctx->scratch_left = kScratchFree;
  }
  if (ctx->scratch_left != kScratchFree) {
    const hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    ctx->scratch_left = kScratchFree;
  }
  ctx->stream_set = false;
  return hipSuccess;
}

// A call's use of the scratch, which a call that returns early ends itself.
struct ScratchUse {
  vgicp_ctx ctx;
  const bool any;  // an empty cloud uses none
  int left = kScratchFree;
  ScratchUse(vgicp_ctx c, bool used) : ctx(c), any(used) {
    if (any) __atomic_store_n(ctx->host_pinned + kScratchWord, ~++ctx->scratch_seq, __ATOMIC_RELAXED);
  }
  ~ScratchUse() {
    if (!any) return;
    if (left == kScratchFree) (void)hipStreamSynchronize(ctx->stream);
    ctx->scratch_left = left;
  }
};

int ensure_scratch(vgicp_ctx ctx, size_t bytes, std::string &msg) {
  if (ctx->scratch_bytes >= bytes) return VGICP_OK;
  if (ctx->scratch) {
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    HIP_TRY(hipFree(ctx->scratch));
    ctx->scratch = nullptr;
    ctx->scratch_bytes = 0;
  }
  const size_t want = std::max(bytes, size_t(1) << 20);
  HIP_TRY(hipMalloc(&ctx->scratch, want));
  ctx->scratch_bytes = want;
  return VGICP_OK;
}

// Lays the workspace of a grouped construction for n points out at base (NULL:
// only sizes it).
static size_t carve_voxel_group(char *base, size_t n, VoxelGroup *g) {
  size_t at = 0;
  carve_group(base, at, n, g);
  const size_t slots = size_t(1) << g->log2slots;
  carve_piece(base, at, &g->skey, slots);
  carve_piece(base, at, &g->smask, slots);
  carve_piece(base, at, &g->sbase, slots);
  carve_piece(base, at, &g->sseg, slots);
  carve_piece(base, at, &g->vox, n);
  carve_piece(base, at, &g->heavy, n / kLightMax + 1);
  return at;
}

// Groups the cloud's points (the launches up to `number`) and waits for the
// counts.  *taken is false when the cloud has to be sorted instead.  pinned_dev
// is the device's address of ctx's pinned words.
static int group_points(vgicp_ctx ctx, const vgicp_cloud *cloud, float s, uint32_t *pinned_dev,
                        VoxelGroup *g, GroupCounts *counts, bool *taken, std::string &msg) {
  const hipStream_t st = ctx->stream;
  const uint32_t n = uint32_t(cloud->n);
  const int rc = ensure_scratch(ctx, carve_voxel_group(nullptr, n, g), msg);
  if (rc != VGICP_OK) return rc;
  carve_voxel_group(static_cast<char *>(ctx->scratch), n, g);
  const uint32_t slots = 1u << g->log2slots;
  auto *host = reinterpret_cast<GroupCounts *>(ctx->host_pinned + kCountsWord);
  auto *host_dev = reinterpret_cast<GroupCounts *>(pinned_dev + kCountsWord);
  // the words may be new to this context and hold another one's counts
  const uint32_t seq = ++ctx->group_seq;
  __atomic_store_n(&host->seq, ~seq, __ATOMIC_RELAXED);
  const uint32_t points = grid_for(n), number = std::min(kNumberBlocks, grid_for(n, 16));
  const VoxelOfPoint key{cloud->xyz, n, s};
  k_group_clear<<<slots / 16, 256, 0, st>>>(*g, ctx->err_word);
  k_group_insert<<<insert_grid(n), 256, 0, st>>>(*g, key);
  k_group_compact<<<slots / kCompactSlots, kCompactThreads, 0, st>>>(*g);
  k_group_number<<<number + points, 256, 0, st>>>(*g, number, n, host_dev, seq);
  HIP_TRY(hipGetLastError());
  // the kernel's first thread writes the counts, so the host need not wait for
  // its end
  HIP_TRY(wait_for_host_words(
      st, [&] { return __atomic_load_n(&host->seq, __ATOMIC_ACQUIRE) == seq; }));
  *counts = *host;
  *taken = !(counts->err & kErrFull);
  return VGICP_OK;
}

static int point_error(uint32_t err, std::string &msg) {
  if (err & kErrNonFinite) {
    msg = "vgicp_voxelize: a point coordinate is not finite";
    return VGICP_ENONFINITE;
  }
  if (err & kErrRange) {
    msg = "vgicp_voxelize: a voxel key lies outside [-2^20, 2^20)";
    return VGICP_ERANGE;
  }
  return VGICP_OK;
}

int voxelize_impl(vgicp_ctx ctx, const vgicp_cloud *cloud, double resolution, vgicp_map *out,
                  std::string &msg) {
  const int64_t n = cloud->n;
  const float s = float(1.0 / resolution);
  const hipStream_t st = ctx->stream;

  int64_t n_voxels = 0, n_bricks = 0;
  VoxScratch sc{};
  VoxelGroup group{};
  GroupCounts counts{};
  bool grouped = false;
  void *pinned = nullptr;
  HIP_TRY(hipHostGetDevicePointer(&pinned, ctx->host_pinned, 0));
  uint32_t *const pinned_dev = static_cast<uint32_t *>(pinned);
  if (n > 0) HIP_TRY(claim_scratch(ctx));
  ScratchUse use(ctx, n > 0);
  // the sorted construction's counts
  auto *segments = reinterpret_cast<SegmentCounts *>(ctx->host_pinned);
  auto *segments_dev = reinterpret_cast<SegmentCounts *>(pinned_dev);
  auto next_seq = [&] {
    const uint32_t seq = ++ctx->group_seq;
    __atomic_store_n(&segments->seq, ~seq, __ATOMIC_RELAXED);
    return seq;
  };
  auto segments_arrive = [&](uint32_t seq) {
    return wait_for_host_words(
        st, [&] { return __atomic_load_n(&segments->seq, __ATOMIC_ACQUIRE) == seq; });
  };
  if (n > 0 && n <= kGroupMaxPoints) {
    int rc = group_points(ctx, cloud, s, pinned_dev, &group, &counts, &grouped, msg);
    // (of a cloud that is sorted instead, not every point has been looked at)
    if (rc == VGICP_OK && grouped) rc = point_error(counts.err, msg);
    if (rc != VGICP_OK) return rc;
    if (grouped) {
      n_voxels = counts.n_voxels;
      n_bricks = counts.n_bricks;
    }
  }
  if (n > 0 && !grouped) {
    size_t total = 0, sort_bytes = 0, scan_bytes = 0;
    HIP_TRY(plan_scratch(n, st, &total, &sort_bytes, &scan_bytes));
    int rc = ensure_scratch(ctx, total, msg);
    if (rc != VGICP_OK) return rc;
    sc = carve(ctx->scratch, n, std::max(sort_bytes, scan_bytes));

    if (n > kGroupMaxPoints) HIP_TRY(hipMemsetAsync(ctx->err_word, 0, sizeof(uint32_t), st));
    k_voxel_keys<<<grid_for(n), 256, 0, st>>>(cloud->xyz, n, s, sc.keys_in, sc.idx_in,
                                               ctx->err_word);
    HIP_TRY(hipGetLastError());
    size_t tb = sc.temp_bytes;
    HIP_TRY(rocprim::radix_sort_pairs(sc.temp, tb, sc.keys_in, sc.keys_out, sc.idx_in, sc.idx_out,
                                      size_t(n), 0, 63, st));
    k_segment_heads<<<grid_for(n), 256, 0, st>>>(sc.keys_out, n, sc.head);
    HIP_TRY(hipGetLastError());
    tb = sc.temp_bytes;
    HIP_TRY(rocprim::inclusive_scan(sc.temp, tb, sc.head, sc.ord1, size_t(n),
                                    rocprim::plus<uint32_t>(), st));
    const uint32_t seq = next_seq();
    k_segment_starts<<<grid_for(n), 256, 0, st>>>(sc.head, sc.ord1, n, sc.seg, ctx->err_word,
                                                   segments_dev, seq);
    HIP_TRY(hipGetLastError());
    HIP_TRY(segments_arrive(seq));
    const int prc = point_error(segments->err, msg);
    if (prc != VGICP_OK) return prc;
    n_voxels = int64_t(segments->n);
  }

  // Brick order: sort the voxels by (brick key, position in the brick).
  uint64_t *vkey = sc.keys_in;
  uint32_t *vord_in = sc.idx_in, *bhead = sc.head, *bord1 = sc.ord1, *vord_out = sc.spare;
  if (n_voxels > 0 && !grouped) {
    size_t need_sort = 0, need_scan = 0;
    HIP_TRY(rocprim::radix_sort_pairs(nullptr, need_sort, (uint64_t *)nullptr,
                                      (uint64_t *)nullptr, (uint32_t *)nullptr,
                                      (uint32_t *)nullptr, size_t(n_voxels), 0, 63, st));
    HIP_TRY(rocprim::inclusive_scan(nullptr, need_scan, (uint32_t *)nullptr, (uint32_t *)nullptr,
                                    size_t(n_voxels), rocprim::plus<uint32_t>(), st));
    // rocPRIM's temporary storage for V <= n elements normally fits in the
    // storage planned for n; if it does not, this phase gets its own.
    void *temp = sc.temp;
    size_t temp_bytes = sc.temp_bytes;
    void *own_temp = nullptr;
    if (need_sort > temp_bytes || need_scan > temp_bytes) {
      temp_bytes = std::max(need_sort, need_scan);
      HIP_TRY(hipMalloc(&own_temp, temp_bytes));
      temp = own_temp;
    }
    const int64_t V = n_voxels;
    k_brick_sortkeys<<<grid_for(V), 256, 0, st>>>(sc.keys_out, sc.seg, V, vkey, sc.bsort_in,
                                                   vord_in);
    HIP_TRY(hipGetLastError());
    size_t tb = temp_bytes;
    hipError_t pe = rocprim::radix_sort_pairs(temp, tb, sc.bsort_in, sc.bsort_out, vord_in,
                                              vord_out, size_t(V), 0, 63, st);
    if (pe == hipSuccess) {
      k_brick_heads<<<grid_for(V), 256, 0, st>>>(sc.bsort_out, V, bhead);
      pe = hipGetLastError();
    }
    tb = temp_bytes;
    if (pe == hipSuccess)
      pe = rocprim::inclusive_scan(temp, tb, bhead, bord1, size_t(V), rocprim::plus<uint32_t>(),
                                   st);
    if (pe == hipSuccess) {
      const uint32_t seq = next_seq();
      k_segment_starts<<<grid_for(V), 256, 0, st>>>(bhead, bord1, V, sc.bstart, nullptr,
                                                     segments_dev, seq);
      pe = hipGetLastError();
      if (pe == hipSuccess) pe = segments_arrive(seq);
    }
    if (own_temp) {
      (void)hipStreamSynchronize(st);
      (void)hipFree(own_temp);
    }
    HIP_TRY(pe);
    n_bricks = int64_t(segments->n);
  }

  // Load factor at most 1/8: a lookup in an empty brick (most misses of a
  // partial overlap) almost always stops at an empty home record or one
  // probe later.  At most kMaxMapBricks bricks, so the table (at most 2^27
  // records) stays within 32-bit byte offsets.
  if (n_bricks > kMaxMapBricks) {
    msg = "vgicp_voxelize: more than 2^24 occupied bricks in one map";
    return VGICP_EINVAL;
  }
  int64_t cap = 16;
  uint32_t log2cap = 4;
  while (cap < 8 * n_bricks) {
    cap <<= 1;
    ++log2cap;
  }
  vgicp_map m = new (std::nothrow) vgicp_voxelmap_s();
  if (!m) {
    msg = "vgicp_voxelize: out of host memory";
    return VGICP_ENOMEM;
  }
  m->device = ctx->device;
  m->n_voxels = n_voxels;
  m->n_bricks = n_bricks;
  m->capacity = cap;
  m->log2cap = log2cap;
  m->scale = s;
  m->resolution = resolution;
  const size_t brick_bytes = align256(size_t(cap) * sizeof(BrickRecord));
  const uint32_t obits = occ_bits(cap);
  const size_t occ_bytes = align256(size_t(obits / 8));
  const size_t stats_bytes = align256(size_t(n_voxels) * sizeof(VoxelStats));
  hipError_t e = hipMalloc(&m->buffer, brick_bytes + occ_bytes + stats_bytes +
                                           size_t(n_voxels) * sizeof(VoxelInfo));
  if (e == hipSuccess) {
    char *base = static_cast<char *>(m->buffer);
    m->bricks = reinterpret_cast<BrickRecord *>(base);
    m->occ = reinterpret_cast<uint32_t *>(base + brick_bytes);
    m->stats = reinterpret_cast<VoxelStats *>(base + brick_bytes + occ_bytes);
    m->info = reinterpret_cast<VoxelInfo *>(base + brick_bytes + occ_bytes + stats_bytes);
  }
  if (e != hipSuccess) {
    delete m;
    msg = std::string("vgicp_voxelize: hipMalloc of the voxel map: ") + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? VGICP_ENOMEM : VGICP_EHIP;
  }
  const unsigned fill = grid_for(std::max<int64_t>(cap, obits / 32));
  if (grouped) {
    const uint32_t nb = uint32_t(n_bricks), nv = uint32_t(n_voxels);
    k_group_finish<<<counts.n_heavy + fill + grid_for(nb, 4) + grid_for(nv, 4), 256,
                     finish_lds(counts.max_count), st>>>(
        group, nb, nv, counts.n_heavy, fill, cloud->xyz, cloud->cov, uint32_t(n), m->bricks, cap,
        m->occ, obits / 32, m->stats, m->info);
    k_group_records<<<grid_for(nb), 256, 0, st>>>(group, nb, m->bricks, log2cap, m->occ, obits - 1,
                                                  pinned_dev + kScratchWord, ctx->scratch_seq);
  } else {
    k_fill_empty<<<fill, 256, 0, st>>>(m->bricks, cap, m->occ, obits / 32);
  }
  if (n_voxels > 0 && !grouped) {
    k_build_bricks<<<grid_for(n_bricks), 256, 0, st>>>(sc.bsort_out, sc.bstart, n_bricks,
                                                       n_voxels, m->bricks, log2cap, m->occ,
                                                       obits - 1);
    k_build_payload<<<grid_for(n_voxels), 256, 0, st>>>(cloud->xyz, cloud->cov, n, sc.idx_out,
                                                        sc.seg, vord_out, vkey, n_voxels,
                                                        m->stats, m->info);
  }
  e = hipGetLastError();
  if (e != hipSuccess) {
    (void)hipFree(m->buffer);
    delete m;
    msg = std::string("vgicp_voxelize: kernel launch: ") + hipGetErrorString(e);
    return VGICP_EHIP;
  }
  use.left = grouped ? kScratchWordFollows : kScratchInUse;
  *out = m;
  return VGICP_OK;
}

int map_export_impl(vgicp_ctx ctx, vgicp_map m, int32_t *keys, float *mean, float *cov,
                    int32_t *count, std::string &msg) {
  if (m->n_voxels == 0) return VGICP_OK;
  k_export<<<grid_for(m->n_voxels), 256, 0, ctx->stream>>>(m->stats, m->info, m->n_voxels, keys,
                                                           mean,
                                                           cov, count);
  HIP_TRY(hipGetLastError());
  return VGICP_OK;
}

}  // namespace vgicp
