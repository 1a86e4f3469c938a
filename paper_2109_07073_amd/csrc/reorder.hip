// Resident, spatially ordered copies of the source clouds of a factor set.
//
// A linearization round streams every source point once and gathers the
// target voxel of each (Sec. III-A).  Consecutive points of a scan in its
// recorded order can lie far apart (a ring of a rotating sensor, thinned),
// so the 64 lanes of a wave touch many brick records and voxel statistics
// lines.  A factor set therefore keeps its own copy of each source cloud with
// the points in Morton order of cells at the finest resolution among the maps
// the cloud is matched against: neighbours in memory are neighbours in space,
// and a rigid transform keeps them neighbours in the target map.  The copy is
// made once; every round reads it instead of the caller's arrays.  Per-point
// outputs are written at the caller's index through the stored permutation.
// The results are the same up to FP32 summation order (integer outputs are
// identical).

#include "group.hpp"

#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>

namespace vgicp {
namespace {

constexpr int kThreads = 256;
constexpr float kCellLo = -1048576.0f;  // -2^20
constexpr float kCellHi = 1048575.0f;   //  2^20 - 1

// Cell index on one axis, offset to [0, 2^21); NaN and out-of-range values
// clamp to the ends (any order of such points is valid).
__device__ __forceinline__ uint32_t cell21(float x, float inv_cell) {
  const float q = fminf(fmaxf(floorf(x * inv_cell), kCellLo), kCellHi);
  return uint32_t(int32_t(q) + 1048576);
}

// The 21 low bits of v moved to every third bit (bit k to bit 3k).
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | (x << 32)) & 0x001f00000000ffffull;
  x = (x | (x << 16)) & 0x001f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// Morton key (63 bits, x most significant within each bit triple) of the cell
// of point i.
__device__ __forceinline__ uint64_t morton_key(const float *__restrict__ xyz, uint32_t n,
                                               uint32_t i, float inv_cell) {
  const uint32_t cx = cell21(xyz[i], inv_cell);
  const uint32_t cy = cell21(xyz[uint64_t(n) + i], inv_cell);
  const uint32_t cz = cell21(xyz[2ull * n + i], inv_cell);
  return (spread3(cx) << 2) | (spread3(cy) << 1) | spread3(cz);
}

// The Morton key and the point's own index of every point of one cloud.
__global__ void __launch_bounds__(kThreads)
k_morton_keys(const float *__restrict__ xyz, uint32_t n, float inv_cell,
              uint64_t *__restrict__ keys, uint32_t *__restrict__ idx) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  keys[i] = morton_key(xyz, n, i, inv_cell);
  idx[i] = i;
}

// Point j of the cloud to position i of the ordered copy, counting a
// non-finite coordinate (nonfinite[0]) or covariance entry (nonfinite[1]): the
// only full pass over a factor set's inputs.
__device__ __forceinline__ void copy_point(const float *__restrict__ xyz,
                                           const float *__restrict__ cov, uint32_t n, uint64_t j,
                                           uint64_t i, float *__restrict__ xyz_out,
                                           float *__restrict__ cov_out,
                                           unsigned long long *__restrict__ nonfinite) {
  const float x = xyz[j], y = xyz[uint64_t(n) + j], z = xyz[2ull * n + j];
  xyz_out[3 * i] = x;
  xyz_out[3 * i + 1] = y;
  xyz_out[3 * i + 2] = z;
  const float2 *src = reinterpret_cast<const float2 *>(cov + 6 * j);
  float2 *dst = reinterpret_cast<float2 *>(cov_out + 6 * i);
  const float2 c0 = src[0], c1 = src[1], c2 = src[2];
  dst[0] = c0;
  dst[1] = c1;
  dst[2] = c2;
  const bool bad_p = !(isfinite(x) && isfinite(y) && isfinite(z));
  const bool bad_c = !(isfinite(c0.x) && isfinite(c0.y) && isfinite(c1.x) && isfinite(c1.y) &&
                       isfinite(c2.x) && isfinite(c2.y));
  if (bad_p) atomicAdd(&nonfinite[0], 1ull);
  if (bad_c) atomicAdd(&nonfinite[1], 1ull);
}

// Copies point perm[i] of the cloud to position i of the ordered copy.
__global__ void __launch_bounds__(kThreads)
k_gather_points(const float *__restrict__ xyz, const float *__restrict__ cov, uint32_t n,
                const int32_t *__restrict__ perm, float *__restrict__ xyz_out,
                float *__restrict__ cov_out, unsigned long long *__restrict__ nonfinite) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i < n) copy_point(xyz, cov, n, uint32_t(perm[i]), i, xyz_out, cov_out, nonfinite);
}

// ---------------------------------------------------------------- grouped order
// The Morton order of many clouds at once: each is grouped by cells and bricks
// (group.hpp; a brick's key is the Morton key of its cells above their six low
// bits, which are the cell's place in the brick), number counts the points in
// the bricks before each brick, and place puts every point behind the points
// of earlier cells and the earlier points of its own.  Five launches order as
// many clouds as the workspace holds; sorting them one by one took twelve
// launches a cloud (450 us of a 10-scan submap's factor set).  A wave's points
// read the list of their cell once each, so a cell costs the square of its
// points: beyond kOrderCellMax a cloud is sorted (a set over one cloud of
// 320,000 points, 1,072 in its fullest cell: 350 us grouped, 350 sorted; 4,011:
// 680 and 360; of 2^20, 1,527: 1,000 and 425).  Numbering squares the bricks, so
// a cloud that is alone gets all of kOrderBlocks (320,000 points in 18,000
// bricks: 270 us, 545 with 64).
struct OrderJob {
  Group g;
  uint32_t *base;  // [slots] points in earlier bricks
  const float *xyz, *cov;
  float *xyz_out, *cov_out;
  int32_t *perm;
  uint32_t n;
  float inv_cell;
  uint32_t *redo;  // set when the cloud has to be sorted instead
};

constexpr size_t kOrderWorkspace = size_t(192) << 20;  // bytes of grouped clouds at once
constexpr uint32_t kOrderJobs = 256;                   // and clouds
constexpr uint32_t kOrderBlocks = 512;                 // blocks that number bricks,
constexpr uint32_t kOrderCloudBlocks = 64;             // of each cloud at least these
constexpr uint32_t kOrderCellMax = 1024;               // points of a cell at most
constexpr uint32_t kOrderBricks = 4;                   // bricks a wave numbers at once
constexpr uint32_t kOrderLoads = 8;                    // other bricks a lane has in flight

// The brick and cell of a point, as group.hpp asks for them.
struct CellOfPoint {
  const float *xyz;
  uint32_t n;
  float inv_cell;
  __device__ uint32_t operator()(uint32_t i, uint64_t &brick, uint32_t &cell) const {
    const uint64_t k = morton_key(xyz, n, i, inv_cell);
    brick = k >> 6;
    cell = uint32_t(k) & 63u;
    return 0u;
  }
};

__global__ void __launch_bounds__(256)
k_order_clear(const OrderJob *__restrict__ jobs) {
  group_clear(jobs[blockIdx.y].g, blockIdx.x);
}

__global__ void __launch_bounds__(256)
k_order_insert(const OrderJob *__restrict__ jobs) {
  const OrderJob &job = jobs[blockIdx.y];
  if (blockIdx.x >= insert_grid(job.n)) return;
  group_insert(job.g, blockIdx.x, job.n, kOrderCellMax,
               CellOfPoint{job.xyz, job.n, job.inv_cell});
}

__global__ void __launch_bounds__(kCompactThreads)
k_order_compact(const OrderJob *__restrict__ jobs) {
  const Group &g = jobs[blockIdx.y].g;
  if (blockIdx.x * kCompactSlots < (1u << g.log2slots)) group_compact(g, blockIdx.x);
}

// Blocks [0, number_blocks): bricks; the others: points.
__global__ void __launch_bounds__(256)
k_order_number(const OrderJob *__restrict__ jobs, uint32_t number_blocks) {
  const OrderJob &job = jobs[blockIdx.y];
  const Group &g = job.g;
  if (blockIdx.x >= number_blocks) {
    group_scatter(g, (blockIdx.x - number_blocks) * 256 + threadIdx.x, job.n);
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *job.redo = g.hdr->err != 0 ? 1u : 0u;
  const uint32_t nb = uint32_t(g.hdr->totals >> kBricksShift), lane = threadIdx.x & 63;
  const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  for (uint32_t i0 = w * kOrderBricks; i0 < nb; i0 += number_blocks * 4 * kOrderBricks) {
    uint64_t key[kOrderBricks];
    uint32_t slot[kOrderBricks], base[kOrderBricks];
#pragma unroll
    for (uint32_t q = 0; q < kOrderBricks; ++q) {
      const uint32_t i = min(i0 + q, nb - 1);
      key[q] = g.bkey[i];
      slot[q] = g.bslot[i];
      base[q] = 0;
    }
    for (uint32_t j0 = lane; j0 < nb; j0 += 64 * kOrderLoads) {
      uint64_t k[kOrderLoads];
      uint32_t pts[kOrderLoads];
#pragma unroll
      for (uint32_t u = 0; u < kOrderLoads; ++u) {
        const uint32_t j = min(j0 + 64 * u, nb - 1);
        k[u] = g.bkey[j];
        pts[u] = g.bpts[j];
      }
#pragma unroll
      for (uint32_t u = 0; u < kOrderLoads; ++u) {
        if (j0 + 64 * u >= nb) k[u] = ~0ull;  // after every brick
#pragma unroll
        for (uint32_t q = 0; q < kOrderBricks; ++q) base[q] += k[u] < key[q] ? pts[u] : 0u;
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kOrderBricks; ++q) {
      if (i0 + q >= nb) break;
      const uint32_t b = wave_total(base[q]);
      if (lane == 0) job.base[slot[q]] = b;
    }
  }
}

__global__ void __launch_bounds__(256)
k_order_place(const OrderJob *__restrict__ jobs, unsigned long long *__restrict__ nonfinite) {
  const OrderJob &job = jobs[blockIdx.y];
  const uint32_t n = job.n, i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n || *job.redo) return;
  const Group &g = job.g;
  const uint32_t code = g.code[i], slot = code >> 6;
  const uint32_t rel = g.rel[code], m = g.count[code];
  const uint32_t *list = g.list + g.first[slot] + rel;
  uint32_t at = job.base[slot] + rel;
  for (uint32_t l = 0; l < m; l += 4) {
    uint32_t o[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) o[u] = list[min(l + u, m - 1)];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) at += (l + u < m && o[u] < i) ? 1u : 0u;
  }
  copy_point(job.xyz, job.cov, n, i, at, job.xyz_out, job.cov_out, nonfinite);
  job.perm[at] = int32_t(i);
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Position q of the sorted (factor, voxel) keys is point q - corr_offset of
// factor f = key >> 32 in its new copy; it takes point vals[q] of the old
// copy (coordinates, covariance, and the caller's index through the old
// permutation, or vals[q] itself when the old copy is the caller's cloud).
__global__ void __launch_bounds__(kThreads)
k_gather_factor_points(const FactorDesc *__restrict__ old_desc,
                       const FactorDesc *__restrict__ new_desc, const uint64_t *__restrict__ keys,
                       const uint32_t *__restrict__ vals, uint64_t total) {
  const uint64_t q = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
  if (q >= total) return;
  const uint32_t f = uint32_t(keys[q] >> 32);
  const uint64_t i = vals[q];
  const FactorDesc &o = old_desc[f];
  const FactorDesc &d = new_desc[f];
  const uint64_t local = q - uint64_t(d.corr_offset);
  float *xyz = const_cast<float *>(d.xyz);
  xyz[3 * local] = o.xyz[3 * i];
  xyz[3 * local + 1] = o.xyz[3 * i + 1];
  xyz[3 * local + 2] = o.xyz[3 * i + 2];
  const float2 *src = reinterpret_cast<const float2 *>(o.cov + 6 * i);
  float2 *dst = reinterpret_cast<float2 *>(const_cast<float *>(d.cov) + 6 * local);
  dst[0] = src[0];
  dst[1] = src[1];
  dst[2] = src[2];
  const_cast<int32_t *>(d.perm)[local] = o.perm ? o.perm[i] : int32_t(i);
}

}  // namespace

hipError_t launch_voxel_order_keys(const vgicp_factorset_s *fs, const double *poses,
                                   uint64_t *keys, uint32_t *vals, hipStream_t st);

hipError_t reorder_by_target(vgicp_factorset_s *fs, const double *poses, hipStream_t st) {
  const int64_t total = fs->total_points;
  if (fs->n_factors == 0 || total == 0) return hipSuccess;
  // new per-factor copies: covariances [n][6], coordinates [n][3], permutation [n]
  std::vector<FactorDesc> nd = fs->h_factors;
  size_t bytes = 0;
  std::vector<size_t> off(nd.size(), 0);
  for (size_t f = 0; f < nd.size(); ++f) {
    const size_t n = size_t(nd[f].n);
    off[f] = bytes;
    if (n) bytes += align256(24 * n) + align256(12 * n) + align256(4 * n);
  }
  int end_bit = 32;
  while (end_bit < 64 && (uint64_t(fs->n_factors - 1) >> (end_bit - 32)) != 0) ++end_bit;
  size_t sort_bytes = 0;
  hipError_t e = rocprim::radix_sort_pairs(
      nullptr, sort_bytes, static_cast<const uint64_t *>(nullptr), static_cast<uint64_t *>(nullptr),
      static_cast<const uint32_t *>(nullptr), static_cast<uint32_t *>(nullptr), size_t(total), 0,
      end_bit, st);
  if (e != hipSuccess) return e;
  const size_t kb = align256(8 * size_t(total)), vb = align256(4 * size_t(total));
  const size_t db = align256(sizeof(FactorDesc) * nd.size());
  char *buf = nullptr, *tmp = nullptr;
  e = hipMalloc(&buf, std::max<size_t>(bytes, 1));
  if (e == hipSuccess) e = hipMalloc(&tmp, 2 * kb + 2 * vb + db + align256(sort_bytes));
  if (e != hipSuccess) {
    if (buf) (void)hipFree(buf);
    return e;
  }
  for (size_t f = 0; f < nd.size(); ++f) {
    const size_t n = size_t(nd[f].n);
    char *p = buf + off[f];
    nd[f].cov = n ? reinterpret_cast<float *>(p) : nullptr;
    nd[f].xyz = n ? reinterpret_cast<float *>(p + align256(24 * n)) : nullptr;
    nd[f].perm = n ? reinterpret_cast<int32_t *>(p + align256(24 * n) + align256(12 * n)) : nullptr;
  }
  uint64_t *keys_in = reinterpret_cast<uint64_t *>(tmp);
  uint64_t *keys_out = reinterpret_cast<uint64_t *>(tmp + kb);
  uint32_t *vals_in = reinterpret_cast<uint32_t *>(tmp + 2 * kb);
  uint32_t *vals_out = reinterpret_cast<uint32_t *>(tmp + 2 * kb + vb);
  FactorDesc *d_new = reinterpret_cast<FactorDesc *>(tmp + 2 * kb + 2 * vb);
  void *sort_tmp = tmp + 2 * kb + 2 * vb + db;
  e = launch_voxel_order_keys(fs, poses, keys_in, vals_in, st);
  if (e == hipSuccess)
    e = rocprim::radix_sort_pairs(sort_tmp, sort_bytes, keys_in, keys_out, vals_in, vals_out,
                                  size_t(total), 0, end_bit, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(d_new, nd.data(), sizeof(FactorDesc) * nd.size(), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) {
    const uint64_t grid = (uint64_t(total) + kThreads - 1) / kThreads;
    k_gather_factor_points<<<unsigned(grid), kThreads, 0, st>>>(fs->d_factors, d_new, keys_out,
                                                                vals_out, uint64_t(total));
    e = hipGetLastError();
  }
  if (e == hipSuccess)
    e = hipMemcpyAsync(fs->d_factors, nd.data(), sizeof(FactorDesc) * nd.size(),
                       hipMemcpyHostToDevice, st);
  const hipError_t se = hipStreamSynchronize(st);
  if (e == hipSuccess) e = se;
  (void)hipFree(tmp);
  if (e != hipSuccess) {
    // the device descriptors may already name the new copies: put the old ones back
    (void)hipMemcpy(fs->d_factors, fs->h_factors.data(), sizeof(FactorDesc) * nd.size(),
                    hipMemcpyHostToDevice);
    (void)hipFree(buf);
    return e;
  }
  if (fs->d_sorted) (void)hipFree(fs->d_sorted);
  fs->d_sorted = buf;
  fs->h_factors = nd;
  return hipSuccess;
}

namespace {

// ctx's scratch, at least `bytes` of it, free for this call's use.
hipError_t reserve_scratch(vgicp_ctx ctx, size_t bytes) {
  const hipError_t e = claim_scratch(ctx);
  if (e != hipSuccess) return e;
  std::string msg;
  const int rc = ensure_scratch(ctx, bytes, msg);
  return rc == VGICP_OK       ? hipSuccess
         : rc == VGICP_ENOMEM ? hipErrorOutOfMemory
                              : hipErrorUnknown;
}

// Enqueues the ordering of the clouds `which`, one by one, with a radix sort of
// their Morton keys in ctx's scratch, into the copies out names.
hipError_t sort_sources(vgicp_ctx ctx, const vgicp_cloud *sources,
                        const std::vector<int32_t> &which, const std::vector<double> &cell,
                        const std::vector<SortedSource> &out, unsigned long long *d_bad) {
  const hipStream_t st = ctx->stream;
  size_t sort_bytes = 0;
  uint32_t nmax = 0;
  for (int32_t s : which) {
    size_t b = 0;
    const hipError_t e = rocprim::radix_sort_pairs(
        nullptr, b, static_cast<const uint64_t *>(nullptr), static_cast<uint64_t *>(nullptr),
        static_cast<const uint32_t *>(nullptr), static_cast<uint32_t *>(nullptr),
        uint32_t(sources[s].n), 0, 63, st);
    if (e != hipSuccess) return e;
    sort_bytes = std::max(sort_bytes, b);
    nmax = std::max(nmax, uint32_t(sources[s].n));
  }
  const size_t kbytes = align256(8 * size_t(nmax)), ibytes = align256(4 * size_t(nmax));
  hipError_t e = reserve_scratch(ctx, 2 * kbytes + ibytes + align256(sort_bytes));
  if (e != hipSuccess) return e;
  char *tmp = static_cast<char *>(ctx->scratch);
  uint64_t *keys_in = reinterpret_cast<uint64_t *>(tmp);
  uint64_t *keys_out = reinterpret_cast<uint64_t *>(tmp + kbytes);
  uint32_t *idx_in = reinterpret_cast<uint32_t *>(tmp + 2 * kbytes);
  void *sort_tmp = tmp + 2 * kbytes + ibytes;
  for (int32_t s : which) {
    if (e != hipSuccess) break;
    const vgicp_cloud &c = sources[s];
    const SortedSource &o = out[size_t(s)];
    const uint32_t n = uint32_t(c.n), grid = (n + kThreads - 1) / kThreads;
    int32_t *perm = const_cast<int32_t *>(o.perm);
    k_morton_keys<<<grid, kThreads, 0, st>>>(c.xyz, n, float(1.0 / cell[size_t(s)]), keys_in,
                                             idx_in);
    e = hipGetLastError();
    size_t b = align256(sort_bytes);
    if (e == hipSuccess)
      e = rocprim::radix_sort_pairs(sort_tmp, b, keys_in, keys_out, idx_in,
                                    reinterpret_cast<uint32_t *>(perm), n, 0, 63, st);
    if (e == hipSuccess) {
      k_gather_points<<<grid, kThreads, 0, st>>>(c.xyz, c.cov, n, perm, const_cast<float *>(o.xyz),
                                                 const_cast<float *>(o.cov), d_bad);
      e = hipGetLastError();
    }
  }
  return e;
}

// Enqueues the grouping of the clouds order.grouped, as many at once as
// kOrderWorkspace holds, in ctx's scratch on its stream; d_redo's words are set
// for the ones that have to be sorted.
hipError_t group_sources(vgicp_ctx ctx, const vgicp_cloud *sources,
                         const std::vector<double> &cell, SourceOrder &order, uint32_t *d_redo) {
  const hipStream_t st = ctx->stream;
  const std::vector<int32_t> &which = order.grouped;
  const size_t count = which.size();
  // the jobs first, then the batches' workspaces over each other
  size_t head = 0;
  OrderJob *d_jobs = nullptr;
  carve_piece<OrderJob>(nullptr, head, &d_jobs, count);
  std::vector<OrderJob> jobs(count);
  std::vector<size_t> batch;  // first job of each
  size_t most = 0, at = head;
  auto place = [&](char *base) {
    batch.clear();
    at = head;
    for (size_t k = 0; k < count; ++k) {
      const size_t n = size_t(sources[which[k]].n);
      auto carve = [&] {
        carve_group(base, at, n, &jobs[k].g);
        carve_piece(base, at, &jobs[k].base, size_t(1) << jobs[k].g.log2slots);
      };
      const size_t before = at;
      if (k > 0) carve();
      if (k == 0 || at - head > kOrderWorkspace || k - batch.back() >= kOrderJobs) {
        if (k > 0) most = std::max(most, before);
        at = head;
        batch.push_back(k);
        carve();
      }
    }
    most = std::max(most, at);
  };
  place(nullptr);
  hipError_t e = reserve_scratch(ctx, most);
  if (e != hipSuccess) return e;
  char *base = static_cast<char *>(ctx->scratch);
  place(base);
  head = 0;
  carve_piece(base, head, &d_jobs, count);
  for (size_t k = 0; k < count; ++k) {
    const vgicp_cloud &c = sources[which[k]];
    const SortedSource &o = order.out[size_t(which[k])];
    jobs[k].xyz = c.xyz;
    jobs[k].cov = c.cov;
    jobs[k].xyz_out = const_cast<float *>(o.xyz);
    jobs[k].cov_out = const_cast<float *>(o.cov);
    jobs[k].perm = const_cast<int32_t *>(o.perm);
    jobs[k].n = uint32_t(c.n);
    jobs[k].inv_cell = float(1.0 / cell[size_t(which[k])]);
    jobs[k].redo = d_redo + k;
  }
  order.jobs.resize(count * sizeof(OrderJob));
  std::memcpy(order.jobs.data(), jobs.data(), order.jobs.size());
  e = hipMemcpyAsync(d_jobs, order.jobs.data(), order.jobs.size(), hipMemcpyHostToDevice, st);
  for (size_t b = 0; b < batch.size() && e == hipSuccess; ++b) {
    const size_t k0 = batch[b], k1 = b + 1 < batch.size() ? batch[b + 1] : count;
    uint32_t nmax = 0, slots = 0, insert = 0;
    for (size_t k = k0; k < k1; ++k) {
      nmax = std::max(nmax, jobs[k].n);
      slots = std::max(slots, 1u << jobs[k].g.log2slots);
      insert = std::max(insert, insert_grid(jobs[k].n));
    }
    const unsigned nj = unsigned(k1 - k0), points = (nmax + 255) / 256;
    const unsigned number = std::max(kOrderCloudBlocks, kOrderBlocks / nj);
    const OrderJob *d = d_jobs + k0;
    k_order_clear<<<dim3(slots / 16, nj), 256, 0, st>>>(d);
    k_order_insert<<<dim3(insert, nj), 256, 0, st>>>(d);
    k_order_compact<<<dim3(slots / kCompactSlots, nj), kCompactThreads, 0, st>>>(d);
    k_order_number<<<dim3(number + points, nj), 256, 0, st>>>(d, number);
    k_order_place<<<dim3(points, nj), 256, 0, st>>>(d, order.d_bad);
    e = hipGetLastError();
  }
  return e;
}

// Gives scratch back that the ordering has grown beyond kScratchKeep, once
// nothing enqueued uses it.
void trim_scratch(vgicp_ctx ctx, const SourceOrder &order) {
  if (ctx->scratch_bytes <= std::max(kScratchKeep, order.scratch_before)) return;
  (void)hipFree(ctx->scratch);
  ctx->scratch = nullptr;
  ctx->scratch_bytes = 0;
}

// Gives the copies back after an error, once nothing enqueued uses them.
hipError_t drop_copies(vgicp_ctx ctx, SourceOrder &order, hipError_t e) {
  (void)hipStreamSynchronize(ctx->stream);
  trim_scratch(ctx, order);
  if (order.buffer) (void)hipFree(order.buffer);
  order.buffer = nullptr;
  order.out.assign(order.out.size(), SortedSource{});
  return e;
}

}  // namespace

hipError_t begin_sorted_sources(vgicp_ctx ctx, const vgicp_cloud *sources, int32_t n_sources,
                                const std::vector<double> &cell, SourceOrder &order) {
  order.out.assign(size_t(n_sources), SortedSource{});
  order.scratch_before = ctx->scratch_bytes;
  // layout: per used cloud, covariances [n][6], coordinates [n][3], permutation
  // [n]; then the two counts of non-finite points and the grouped clouds' words
  size_t total = 0;
  std::vector<size_t> off(size_t(n_sources), 0);
  for (int32_t s = 0; s < n_sources; ++s) {
    const int64_t n = sources[s].n;
    if (!(cell[size_t(s)] > 0.0) || n <= 0) continue;
    off[size_t(s)] = total;
    total += align256(24 * size_t(n)) + align256(12 * size_t(n)) + align256(4 * size_t(n));
    (n <= kGroupMaxPoints ? order.grouped : order.sorted).push_back(s);
  }
  if (total == 0) return hipSuccess;
  const size_t words = 2 * sizeof(unsigned long long) + order.grouped.size() * sizeof(uint32_t);
  hipError_t e = hipMalloc(&order.buffer, total + words);
  if (e != hipSuccess) {
    order.buffer = nullptr;
    return e;
  }
  char *base = static_cast<char *>(order.buffer);
  for (const auto *list : {&order.grouped, &order.sorted})
    for (int32_t s : *list) {
      const size_t n = size_t(sources[s].n);
      char *p = base + off[size_t(s)];
      order.out[size_t(s)] = SortedSource{
          reinterpret_cast<float *>(p + align256(24 * n)), reinterpret_cast<float *>(p),
          reinterpret_cast<int32_t *>(p + align256(24 * n) + align256(12 * n))};
    }
  order.d_bad = reinterpret_cast<unsigned long long *>(base + total);
  e = hipMemsetAsync(order.d_bad, 0, words, ctx->stream);
  if (e == hipSuccess && !order.grouped.empty())
    e = group_sources(ctx, sources, cell, order, reinterpret_cast<uint32_t *>(order.d_bad + 2));
  return e == hipSuccess ? e : drop_copies(ctx, order, e);
}

hipError_t finish_sorted_sources(vgicp_ctx ctx, const vgicp_cloud *sources,
                                 const std::vector<double> &cell, SourceOrder &order) {
  const hipStream_t st = ctx->stream;
  if (!order.buffer) return hipStreamSynchronize(st);
  // the counts and the grouped clouds' words
  std::vector<unsigned long long> words(2 + (order.grouped.size() + 1) / 2);
  auto fetch = [&](size_t bytes) {
    const hipError_t e =
        hipMemcpyAsync(words.data(), order.d_bad, bytes, hipMemcpyDeviceToHost, st);
    const hipError_t se = hipStreamSynchronize(st);
    return e == hipSuccess ? se : e;
  };
  hipError_t e = hipSuccess;
  if (!order.grouped.empty()) {
    e = fetch(2 * sizeof(unsigned long long) + order.grouped.size() * sizeof(uint32_t));
    if (e != hipSuccess) return drop_copies(ctx, order, e);
    const uint32_t *redo = reinterpret_cast<const uint32_t *>(words.data() + 2);
    for (size_t k = 0; k < order.grouped.size(); ++k)
      if (redo[k]) order.sorted.push_back(order.grouped[k]);
  }
  if (!order.sorted.empty()) {
    e = sort_sources(ctx, sources, order.sorted, cell, order.out, order.d_bad);
    if (e == hipSuccess) e = fetch(2 * sizeof(unsigned long long));
    if (e != hipSuccess) return drop_copies(ctx, order, e);
  }
  trim_scratch(ctx, order);
  order.nonfinite[0] = int64_t(words[0]);
  order.nonfinite[1] = int64_t(words[1]);
  return hipSuccess;
}

}  // namespace vgicp
