// Grouping a cloud's points by cells and bricks of 4 x 4 x 4 cells, on gfx950.
//
// Points are counted into an open-addressed table of 64 counters per brick, so
// nothing of the cloud's size is sorted; only the bricks are ordered, by
// counting, for each, the ones before it.  Bound by the latency of dependent
// launches, atomics and gathers, not by the bytes (for a scan of 20,000 points
// 4 MB of counters are cleared and about 2 MB moved), so the steps are few and
// each keeps many loads in flight:
//   clear    the counters and slots of the table;
//   insert   per point: its brick's slot, its arrival number in its cell;
//   compact  per 512 slots: a list of the occupied ones, and where each
//            cell's points start in a list of points;
//   scatter  per point: its index into its cell's part of the list.
// The points of a cell arrive in any order; who reads the list puts them back
// in point order.
#pragma once

#include "vgicp_internal.hpp"

namespace vgicp {

// The largest grouped cloud.  (Voxels of 2^20 street points: 160 us grouped and
// 680 sorted at 0.5 m, 227 and 500 at 0.25 m; the totals below hold 2^21 - 1.)
constexpr int64_t kGroupMaxPoints = int64_t(1) << 20;
constexpr uint32_t kGroupMaxSlots = 1u << 15;  // 8 MB of counters
constexpr uint32_t kGroupProbes = 64;          // slots a point tries
constexpr uint32_t kLightMax = 64;             // points of a cell a wave orders
// Error bit: a brick found no slot or a cell has too many points, so the cloud
// has to be sorted.  Whatever follows in the chain then does nothing.
constexpr uint32_t kErrFull = 4u;
constexpr uint32_t kNoCell = 0xffffffffu;

// Totals of the listed bricks in one word: points in the low 21 bits, cells in
// the next 21, bricks above.
constexpr uint32_t kCellsShift = 21, kBricksShift = 42;
constexpr uint32_t kTotalsMask = (1u << 21) - 1u;
static_assert(kGroupMaxPoints <= int64_t(kTotalsMask), "totals in 21 bits");

struct GroupHeader {
  uint64_t totals;
  uint32_t n_heavy;    // cells of more than kLightMax points,
  uint32_t max_count;  // points of the fullest of them (0 without one),
  uint32_t heavy_at;   // and how many of them are listed
  uint32_t err;
  uint32_t done;  // blocks of the last kernel that have read the workspace
};

struct Group {
  GroupHeader *hdr;
  uint64_t *keys;   // [slots] brick key or kEmptyKey
  uint32_t *count;  // [slots][64] points per cell
  uint32_t *rel;    // [slots][64] first point of a cell in its brick's list
  uint32_t *first;  // [slots] first point of a brick in the list
  uint64_t *bkey, *bmask;  // [bricks] in any order: key, occupied cells,
  uint32_t *bslot, *bpts;  // slot and points
  uint32_t *code, *arrival;  // [n] slot * 64 + cell of the point
  uint32_t *list;            // [n] points, cell after cell
  uint32_t log2slots;
};

// Twice as many slots as there can be bricks for a small cloud; a larger one
// has eight or more points to a brick (a street of 20,000 returns has about
// 1,000 bricks of 2 m and 2,500 of 1 m), and the counters cost 256 bytes a
// slot to clear.
inline uint32_t group_log2slots(uint32_t n) {
  const uint32_t want = std::min(2 * n, std::max(8192u, n / 2));
  uint32_t l = 10;
  while ((1u << l) < kGroupMaxSlots && (1u << l) < want) ++l;
  return l;
}

// The next piece of a workspace: `count` values at base + at.
template <typename T>
inline void carve_piece(char *base, size_t &at, T **p, size_t count) {
  *p = reinterpret_cast<T *>(base + at);
  at += (count * sizeof(T) + 255) & ~size_t(255);
}

// Lays a group for n points out at base + at (base NULL: only sizes it).
inline void carve_group(char *base, size_t &at, size_t n, Group *g) {
  g->log2slots = group_log2slots(uint32_t(n));
  const size_t slots = size_t(1) << g->log2slots;
  carve_piece(base, at, &g->hdr, 1);
  carve_piece(base, at, &g->keys, slots);
  carve_piece(base, at, &g->count, slots * 64);
  carve_piece(base, at, &g->rel, slots * 64);
  carve_piece(base, at, &g->first, slots);
  carve_piece(base, at, &g->bkey, slots);
  carve_piece(base, at, &g->bmask, slots);
  carve_piece(base, at, &g->bslot, slots);
  carve_piece(base, at, &g->bpts, slots);
  carve_piece(base, at, &g->code, n);
  carve_piece(base, at, &g->arrival, n);
  carve_piece(base, at, &g->list, n);
}

// Sum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
  int x = int(v);
#define VGICP_ADD(CTRL, MASK) x += __builtin_amdgcn_update_dpp(0, x, CTRL, MASK, 0xf, false);
  VGICP_ADD(0xb1, 0xf) VGICP_ADD(0x4e, 0xf) VGICP_ADD(0x141, 0xf) VGICP_ADD(0x140, 0xf)
  VGICP_ADD(0x142, 0xa) VGICP_ADD(0x143, 0xc)
#undef VGICP_ADD
  return uint32_t(__builtin_amdgcn_readlane(x, 63));
}

// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  const uint32_t lane = threadIdx.x & 63;
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(v, d);
    if (lane >= d) v += o;
  }
  return v;
}

// Blocks of 256 threads over 16 slots each.
__device__ __forceinline__ void group_clear(const Group &g, uint32_t block) {
  const uint32_t i = block * 256 + threadIdx.x, slots = 1u << g.log2slots;  // 16 bytes each
  if (i < slots * 16) reinterpret_cast<uint4 *>(g.count)[i] = make_uint4(0, 0, 0, 0);
  if (i < slots) g.keys[i] = kEmptyKey;
  if (i == 0) *g.hdr = GroupHeader{0, 0, 0, 0, 0, 0};
}

// Point i of n.  key(i, brick, cell) sets the point's brick key and its cell in
// the brick and returns the error bits of a point that is refused; a cell takes
// `most` points.
// Consecutive points of a scan often fall in one cell (the near rings put
// hundreds there), so a wave's runs of equal keys look their brick up once and
// take their arrival numbers with one atomic (320,000 points: 60 us with an
// atomic each, 28 us by runs).
template <typename Key>
__device__ __forceinline__ void group_point(const Group &g, uint32_t i, uint32_t n, uint32_t most,
                                            Key key) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t brick = 0;
  uint32_t cell = 0;
  uint32_t bad = i < n ? key(i, brick, cell) : 0u;
  const bool valid = i < n && !bad;
  // whole waves shuffle
  const uint64_t pbrick = __shfl_up((unsigned long long)brick, 1);
  const uint32_t pcell = __shfl_up(valid ? cell : kNoCell, 1);
  const bool joins = lane > 0 && valid && pbrick == brick && pcell == cell;
  const uint64_t heads = __ballot(!joins);
  const uint32_t head = 63u - uint32_t(__clzll(heads & (~0ull >> (63 - lane))));
  uint32_t code = kNoCell, arrival = 0;
  if (valid && !joins) {
    const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
    const uint32_t run = later ? uint32_t(__ffsll((unsigned long long)later)) : 64u - lane;
    const uint32_t smask = (1u << g.log2slots) - 1u;
    uint32_t h = uint32_t((brick * 0x9E3779B97F4A7C15ull) >> (64 - g.log2slots));
    bad = kErrFull;
    for (uint32_t p = 0; p < kGroupProbes; ++p) {
      // a slot's key never changes once set, and a stale empty one only sends
      // the point to the exchange, so a cached one serves (2 us of 320,000
      // points' 35)
      uint64_t at = __hip_atomic_load(&g.keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (at == kEmptyKey) {
        at = atomicCAS(reinterpret_cast<unsigned long long *>(&g.keys[h]),
                       (unsigned long long)kEmptyKey, (unsigned long long)brick);
        if (at == kEmptyKey) at = brick;
      }
      if (at == brick) {
        bad = 0;
        break;
      }
      h = (h + 1) & smask;
    }
    if (!bad) {
      code = (h << 6) | cell;
      arrival = atomicAdd(&g.count[code], run);
      if (arrival + run > most) bad = kErrFull;
    }
  }
  const uint64_t refused = __ballot(bad != 0);
  if (refused) {
    uint32_t bits = 0;
#pragma unroll
    for (uint32_t b = 1; b <= kErrFull; b <<= 1) bits |= __ballot((bad & b) != 0) ? b : 0u;
    if (lane == uint32_t(__ffsll((unsigned long long)refused)) - 1u) atomicOr(&g.hdr->err, bits);
  }
  code = __shfl(code, int(head));
  arrival = __shfl(arrival, int(head)) + (lane - head);
  if (i < n) {
    g.code[i] = code;
    g.arrival[i] = arrival;
  }
}

// Whether a kernel of the chain goes on; the insert's waves may set it meanwhile.
__device__ __forceinline__ bool group_full(const Group &g) {
  const uint32_t err = __hip_atomic_load(&g.hdr->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_amdgcn_readfirstlane(err) & kErrFull;
}

// The points of one wave of insert_grid's blocks of 256 threads.
// Of a large cloud a wave takes several groups of 64 points one after the
// other, so that those of a cloud that has to be sorted stop once one has found
// out.  (All at once, an insert ran to its end before anything could be known of
// it: 105 us for 320,000 points in 60,600 bricks, now 86, and 349 for 2^20 in
// 127,900, now 112.)  Fewer waves are enough to keep the atomics busy: at 320,000
// points a voxelization takes 83 us in 4 groups, 89 in 8 and 93 in one, at 2^20
// 161 in 8 and in 4, 178 in one.  Up to 2^17 points one group each leaves no CU
// without waves.
__host__ __device__ inline uint32_t insert_runs(uint32_t n) {
  return n <= (1u << 17) ? 1u : n <= (1u << 19) ? 4u : 8u;
}
__host__ __device__ inline uint32_t insert_grid(uint32_t n) {
  const uint32_t points = 256 * insert_runs(n);
  return (n + points - 1) / points;
}

template <typename Key>
__device__ __forceinline__ void group_insert(const Group &g, uint32_t block, uint32_t n,
                                             uint32_t most, Key key) {
  const uint32_t runs = insert_runs(n);
  const uint32_t first = (block * 256 + (threadIdx.x & ~63u)) * runs + (threadIdx.x & 63u);
  for (uint32_t r = 0; r < runs; ++r) {
    if (r > 0 && group_full(g)) return;
    group_point(g, first + r * 64, n, most, key);
  }
}

// One block of 16 waves per kCompactSlots slots; each wave takes four bricks at
// once.  The blocks place their bricks and points with one atomic each, few
// enough (at most 64) that its serial updates do not show: with a block per 64
// slots they took 10 us more.
constexpr uint32_t kCompactSlots = 512;
constexpr uint32_t kCompactThreads = 1024;
constexpr uint32_t kCompactWaves = kCompactThreads / 64;
constexpr uint32_t kSlotWaves = kCompactSlots / 64;
static_assert(kSlotWaves <= kCompactWaves, "a thread per slot");

__device__ __forceinline__ void group_compact(const Group &g, uint32_t block) {
  __shared__ uint32_t occupied[kCompactSlots], points[kCompactSlots], slot_n[kSlotWaves],
      point_n[kSlotWaves], cell_n, heavy_n, most_n;
  __shared__ uint64_t masks[kCompactSlots];
  __shared__ uint64_t at;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t slot = block * kCompactSlots + tid;
  const uint32_t err = g.hdr->err;
  const bool used = tid < kCompactSlots && g.keys[slot] != kEmptyKey;
  if (err & kErrFull) return;  // no brick is listed then
  const uint64_t m = __ballot(used);
  if (lane == 0 && wave < kSlotWaves) slot_n[wave] = uint32_t(__popcll(m));
  if (tid == 0) cell_n = heavy_n = most_n = 0;
  __syncthreads();
  uint32_t nb = 0, pos = uint32_t(__popcll(m & ((1ull << lane) - 1ull)));
#pragma unroll
  for (uint32_t w = 0; w < kSlotWaves; ++w) {
    if (w < wave) pos += slot_n[w];
    nb += slot_n[w];
  }
  if (nb == 0) return;
  if (used) occupied[pos] = slot;
  __syncthreads();
  uint32_t cells = 0, heavy = 0, most = 0;
  for (uint32_t b0 = wave * 4; b0 < nb; b0 += kCompactWaves * 4) {
    uint32_t c[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) c[q] = g.count[(occupied[min(b0 + q, nb - 1)] << 6) | lane];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      if (b0 + q >= nb) break;
      const uint32_t incl = wave_scan(c[q]);
      const uint64_t mask = __ballot(c[q] > 0);
      if (c[q] > 0) g.rel[(occupied[b0 + q] << 6) | lane] = incl - c[q];
      if (lane == 63) {
        points[b0 + q] = incl;
        masks[b0 + q] = mask;
      }
      cells += uint32_t(__popcll(mask));
      heavy += uint32_t(__popcll(__ballot(c[q] > kLightMax)));
      most = max(most, c[q]);
    }
  }
  if (heavy > 0) atomicMax(&most_n, most);
  if (lane == 0) {
    atomicAdd(&cell_n, cells);
    atomicAdd(&heavy_n, heavy);
  }
  __syncthreads();
  const uint32_t p = tid < nb ? points[tid] : 0u;
  const uint32_t incl = wave_scan(p);
  if (lane == 63 && wave < kSlotWaves) point_n[wave] = incl;
  __syncthreads();
  if (tid == 0) {
    uint64_t pts = 0;
    for (uint32_t w = 0; w < kSlotWaves; ++w) pts += point_n[w];
    at = atomicAdd(reinterpret_cast<unsigned long long *>(&g.hdr->totals),
                   (unsigned long long)((uint64_t(nb) << kBricksShift) |
                                        (uint64_t(cell_n) << kCellsShift) | pts));
    if (heavy_n > 0) {
      atomicAdd(&g.hdr->n_heavy, heavy_n);
      atomicMax(&g.hdr->max_count, most_n);
    }
  }
  __syncthreads();
  if (tid < nb) {
    uint32_t before = incl - p;
    for (uint32_t w = 0; w < wave; ++w) before += point_n[w];
    const uint32_t id = uint32_t(at >> kBricksShift) + tid, sl = occupied[tid];
    g.bkey[id] = g.keys[sl];
    g.bmask[id] = masks[tid];
    g.bslot[id] = sl;
    g.bpts[id] = p;
    g.first[sl] = (uint32_t(at) & kTotalsMask) + before;
  }
}

// Point i of n, after compact.
__device__ __forceinline__ void group_scatter(const Group &g, uint32_t i, uint32_t n) {
  if (i >= n) return;
  const uint32_t err = g.hdr->err, code = g.code[i];  // the code is not set if full
  if (!(err & kErrFull) && code != kNoCell) g.list[g.first[code >> 6] + g.rel[code] + g.arrival[i]] = i;
}

}  // namespace vgicp
