// The walk of a call of few query tiles in one launch (paper Sec. 2, Alg. 1).
//
// Pools of different subtrees never meet, so a workgroup takes one subtree
// for one query tile from the first tested level down to the last pools by
// itself: its frontier stays in LDS, the levels are a loop, and only the
// surviving last-level pools go to memory (the bucketed frontier that the leaf
// test reads).  The level-by-level kernels pay their launch, their 130 KB
// query tile and a chain of dependent loads on every level, 40 us each however
// few the entries; here a level is one round of row loads and a barrier.
#include <math.h>

#include <algorithm>

#include "gt_internal.h"
#include "gt_device.h"
#include "gt_mma.h"
#include "gt_numerics.h"

namespace gt {

namespace {

constexpr int kSubtreeThreads = 512;
constexpr int kSubtreeLevels = 11;        // most levels below a subtree's root pool
constexpr int kSubtreeLds = 160 * 1024;
constexpr int kSteps = 32;                // 64-byte row steps in flight per lane
constexpr int kWindowLds = 128 * 1024;    // query bytes held at once where a tile does not fit

// LDS: the query rows, then the lists of (pool, mask) entries.  A list of level
// l holds at most 2^(l - top) entries; consecutive levels alternate between
// two lists, the larger sized for level depth - 2 (the last level's entries
// leave the workgroup).
__host__ __device__ inline int list_entries(int depth, int top, int which) {
  const int m = depth - 2 - top - which;  // which: 0 the larger, 1 the smaller
  return m < 0 ? 1 : 1 << m;
}
__host__ __device__ inline int subtree_lds(int qbytes, int qrows, int depth, int top) {
  return qrows * (qbytes + 16) + (list_entries(depth, top, 0) + list_entries(depth, top, 1)) * 12 + 64;
}

// Copies nbytes (a multiple of 16) of each of the tile's query rows, from
// column byte `from`, to LDS rows of stride rs.
__device__ __forceinline__ void stage_queries(unsigned char* lds, const unsigned char* src,
                                              int rowbytes, int from, int nbytes, int rs,
                                              int qrows) {
  const int vpr = nbytes / 16, nvec = qrows * vpr;
  for (int v0 = 0; v0 < nvec; v0 += 8 * kSubtreeThreads) {
    uint4 buf[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int v = v0 + k * kSubtreeThreads + (int)threadIdx.x, vv = v < nvec ? v : nvec - 1;
      buf[k] = *reinterpret_cast<const uint4*>(src + (size_t)(vv / vpr) * rowbytes + from + (vv % vpr) * 16);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int v = v0 + k * kSubtreeThreads + (int)threadIdx.x;
      if (v < nvec) *reinterpret_cast<uint4*>(lds + (v / vpr) * rs + (v % vpr) * 16) = buf[k];
    }
  }
}

// Products of one 16-row group with the staged query columns: nsteps 64-byte
// steps from `row` against `brow`.  The matrix-core operand of lane 16 g + i is
// row i, 16-byte chunk g; loads in that order touch four lines with each four
// lanes.  kQuads: four lanes take 64 contiguous bytes of a row (lanes 4 R ..
// 4 R + 3: row R), and the operand comes from lane 4 i + g (bp).  Kernel with /
// without (us): float8 of 300,007 x 777, 257 queries 124 / 134; float32 of
// 100,003 x 300, 65 queries 55 / 60.  Not where the passing between lanes costs
// more: one block of queries (float32, 524,288 x 500, 1 query 40 / 33), or
// bfloat16 (4 blocks 88 / 86).
template <int FMT, int NQB>
constexpr bool kQuads = FMT != GT_POOL_BF16 && NQB >= 2;

template <int FMT, int NQB>
__device__ __forceinline__ void group_products(const unsigned char* row, const unsigned char* brow,
                                               int rs, int nsteps, int bp, f32x4 (&acc)[NQB]) {
  for (int s0 = 0; s0 < nsteps; s0 += kSteps) {
    uint4 x[kSteps];
#pragma unroll
    for (int c = 0; c < kSteps; c += 4)
      if (s0 + c < nsteps) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int st = s0 + c + u < nsteps ? s0 + c + u : nsteps - 1;
          x[c + u] = ld_global16(row + 64 * st);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < kSteps; ++c)
      if (s0 + c < nsteps) {
        uint4 v = x[c];
        if constexpr (kQuads<FMT, NQB>) {
          v.x = (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)v.x);
          v.y = (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)v.y);
          v.z = (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)v.z);
          v.w = (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)v.w);
        }
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
          mma16x16<FMT>(v, ld_lds16(brow + qb * 16 * rs + 64 * (s0 + c)), acc[qb]);
      }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A wave takes 16 pool rows at a time (16 pools of the first level, then both
// children of 8 entries), 32 64-byte steps of them in flight.
// Scores, thresholds and decisions are those of the level kernels' direct
// test (the sums run over the same products in another order, which the
// thresholds' slack covers).
// WIN: the tile's query rows do not fit beside the lists and pass through LDS
// in windows; the waves then step through the windows together, two groups
// each, so that a window serves up to 16 groups.
template <int FMT, int NQB, bool WIN>
__global__ __launch_bounds__(kSubtreeThreads, 1) void k_walk_subtree(SubtreeArgs a) {
  using F = WalkFmt<FMT>;
  constexpr int TQ = F::TQ, NW = kSubtreeThreads / 64, G = WIN ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ uint32_t cnt[GT_MAX_LEVELS], prs[GT_MAX_LEVELS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, g4 = lane >> 4;
  // the tiles of a subtree run on one XCD, which then shares its rows in L2
  const int i = blockIdx.x / kXcds;
  const int t = i % a.nt;
  const int64_t sub = (int64_t)(i / a.nt) * kXcds + blockIdx.x % kXcds;
  const int D = a.depth;
  if ((sub << (D - a.top)) >= a.n_epoch) return;  // no row below it
  const uint64_t tmask = a.tile_mask[t];
  if (tmask == 0ull) return;

  const int rowbytes = a.dp * F::ESZ;
  const int qbytes = WIN ? a.window : rowbytes;  // query columns held at once
  const int rs = qbytes + 16;                    // LDS row stride (bank spread)
  const int cap0 = list_entries(D, a.top, 0);
  uint64_t* const mask0 = reinterpret_cast<uint64_t*>(lds + a.qrows * rs);
  uint64_t* const mask1 = mask0 + cap0;
  uint32_t* const node0 = reinterpret_cast<uint32_t*>(mask1 + list_entries(D, a.top, 1));
  uint32_t* const node1 = node0 + cap0;
  if (tid < GT_MAX_LEVELS) cnt[tid] = prs[tid] = 0u;
  const unsigned char* qsrc =
      reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)t * TQ * rowbytes;
  if (!WIN) stage_queries(lds, qsrc, rowbytes, 0, rowbytes, rs, a.qrows);
  float th0[NQB];
  int qe[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    th0[qb] = a.thr[t * TQ + 16 * qb + c16];
    qe[qb] = FMT == GT_POOL_FP8E4M3 ? a.qexp[t * TQ + 16 * qb + c16] : 0;
  }
  const uint32_t slot = (uint32_t)(sub >> (a.top - a.nb)) * (uint32_t)a.nt + (uint32_t)t;
  const unsigned char* brow = lds + c16 * rs + 16 * g4;
  const int bp = 4 * (4 * c16 + g4);

  for (int l = a.first; l < D; ++l) {
    __syncthreads();  // the query rows, and the entries of the level above
    const bool head = l == a.first;
    const int par = (D - 2 - (l - 1)) & 1, out = (D - 2 - l) & 1;
    const uint64_t* in_mask = par ? mask1 : mask0;
    const uint32_t* in_node = par ? node1 : node0;
    uint64_t* om = out ? mask1 : mask0;
    uint32_t* on = out ? node1 : node0;
    const uint32_t root = (uint32_t)(sub << (l - a.top));  // the subtree's first pool here
    const int shift = D - l;
    uint32_t n;  // rows to test
    if (head) {
      const int64_t pop = ((a.n_epoch - 1) >> shift) + 1 - (int64_t)root;
      n = (uint32_t)min((int64_t)1 << (l - a.top), pop);
    } else {
      n = 2u * cnt[l - 1];
    }
    float th[NQB];
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
      th[qb] = FMT == GT_POOL_FP8E4M3 ? ldexpf(th0[qb] * kFp8ThrFactor, -(qe[qb] + a.lexp[l])) : th0[qb];
    const unsigned char* level = reinterpret_cast<const unsigned char*>(a.pools) +
                                 (size_t)((int64_t(1) << l) - 1) * rowbytes + 16 * (kQuads<FMT, NQB> ? lane & 3 : g4);
    uint32_t pairs = 0;
    // (every wave takes part in every round of a windowed tile)
    for (uint32_t g0 = WIN ? 0u : (uint32_t)wave; 16u * g0 < n; g0 += G * NW) {
      uint32_t node[G];
      uint64_t pm[G];
      const unsigned char* row[G];  // of the row this lane loads
      f32x4 acc[G][NQB];
      bool any[G];  // the wave has this group
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const uint32_t gf = 16u * (g0 + (WIN ? (uint32_t)(wave + k * NW) : 0u));
        any[k] = gf < n;
        const uint32_t r = gf + (uint32_t)c16, rr = r < n ? r : any[k] ? gf : 0u;
        if (head) {
          node[k] = root + rr;
          pm[k] = r < n ? tmask : 0ull;
        } else {
          node[k] = 2u * in_node[rr >> 1] + (rr & 1u);
          pm[k] = r < n && ((int64_t)node[k] << shift) < a.n_epoch ? in_mask[rr >> 1] : 0ull;
        }
        const uint32_t rn = kQuads<FMT, NQB> ? (uint32_t)__shfl((int)node[k], lane >> 2, 64) : node[k];
        row[k] = level + (size_t)rn * rowbytes;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
          for (int x = 0; x < 4; ++x) acc[k][qb][x] = 0.0f;
      }
      if constexpr (WIN) {
        for (int from = 0; from < rowbytes; from += qbytes) {
          const int nb = min(qbytes, rowbytes - from);
          __syncthreads();  // every wave is done with the previous window
          stage_queries(lds, qsrc, rowbytes, from, nb, rs, a.qrows);
          __syncthreads();
#pragma unroll
          for (int k = 0; k < G; ++k)
            if (any[k])
              group_products<FMT, NQB>(row[k] + from, brow, rs, nb / 64, bp, acc[k]);
        }
      } else {
        group_products<FMT, NQB>(row[0], brow, rs, rowbytes / 64, bp, acc[0]);
      }
#pragma unroll
      for (int k = 0; k < G; ++k) {
        // register x of lane j: row 4 (j / 16) + x, query 16 qb + j % 16; lane
        // r < 16 ends with row r's mask
        uint64_t mine = 0ull;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          uint64_t part = 0ull;
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            const uint64_t bal = __ballot(acc[k][qb][x] >= th[qb]);
            part |= ((bal >> (16 * ((lane & 15) >> 2))) & 0xffffull) << (16 * qb);
          }
          if ((lane & 3) == x) mine = part;
        }
        mine = lane < 16 ? (mine & pm[k]) : 0ull;
        if (lane < 16) pairs += (uint32_t)__popcll(pm[k]);
        const uint64_t bal = __ballot(mine != 0ull);
        if (bal == 0ull) continue;
        const uint32_t rank = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        uint32_t base = 0;
        if (l < D - 1) {
          if (lane == 0) base = atomicAdd(&cnt[l], (uint32_t)__popcll(bal));
          base = __shfl(base, 0, 64);
          if (mine) {
            on[base + rank] = node[k];
            om[base + rank] = mine;
          }
        } else {
          if (lane == 0)
            base = atomicAdd(&a.lvl_count[(size_t)l * kMaxSlots + slot], (uint32_t)__popcll(bal));
          base = __shfl(base, 0, 64);
          if (mine) {
            if (base + rank < a.bcap) {
              const size_t o = (size_t)slot * a.bcap + base + rank;
              a.out_node[o] = node[k];
              a.out_mask[o] = mine;
            } else {
              atomicOr(a.over, 1u);
            }
          }
        }
      }
    }
    for (int o = 8; o >= 1; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0 && pairs) atomicAdd(&prs[l], pairs);
  }
  __syncthreads();
  if (tid < D && tid >= a.first) {
    if (tid < D - 1 && cnt[tid]) atomicAdd(&a.lvl_count[(size_t)tid * kMaxSlots + slot], cnt[tid]);
    if (prs[tid]) stat_add(a.stat + tid, GT_MAX_LEVELS, blockIdx.x, prs[tid]);
  }
}

template <int FMT, int NQB, bool WIN>
hipError_t launch_subtree(const SubtreeArgs& a, hipStream_t s) {
  const int bytes = subtree_lds(WIN ? a.window : a.dp * WalkFmt<FMT>::ESZ, a.qrows, a.depth, a.top);
  const int64_t subs = ((a.n_epoch - 1) >> (a.depth - a.top)) + 1;
  const int64_t grid = kXcds * ((subs + kXcds - 1) / kXcds) * a.nt;
  const void* fn = reinterpret_cast<const void*>(k_walk_subtree<FMT, NQB, WIN>);
  if (hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)) return e;
  hipLaunchKernelGGL((k_walk_subtree<FMT, NQB, WIN>), dim3((unsigned)grid), dim3(kSubtreeThreads),
                     (size_t)bytes, s, a);
  return hipGetLastError();
}

template <int FMT>
hipError_t launch_subtree_fmt(const SubtreeArgs& a, hipStream_t s) {
  const bool win = a.window > 0;
  if (a.qrows == 16) return win ? launch_subtree<FMT, 1, true>(a, s) : launch_subtree<FMT, 1, false>(a, s);
  if (a.qrows == 32) return win ? launch_subtree<FMT, 2, true>(a, s) : launch_subtree<FMT, 2, false>(a, s);
  if constexpr (WalkFmt<FMT>::TQ == 64) {
    if (a.qrows == 64) return win ? launch_subtree<FMT, 4, true>(a, s) : launch_subtree<FMT, 4, false>(a, s);
  }
  return hipErrorInvalidValue;
}

int esz_of(int fmt) { return fmt == GT_POOL_F32 ? 4 : fmt == GT_POOL_BF16 ? 2 : 1; }

bool subtree_fits(int qbytes, int qrows, int depth, int top) {
  return depth - 1 - top <= kSubtreeLevels && subtree_lds(qbytes, qrows, depth, top) + 512 <= kSubtreeLds;
}

}  // namespace

// About one workgroup per CU over all tiles (2^8 subtrees for one tile), and
// more, smaller subtrees where the frontier lists would not fit beside the
// query rows.  Query rows that do not fit with the largest lists are windowed.
bool subtree_shape(int fmt, int dp, int nt, int qrows, int depth, int first, int& top, int& window) {
  if (first > depth - 1 || depth > 31) return false;
  int lg = 0;
  while ((1 << lg) < nt) ++lg;
  const int rowbytes = dp * esz_of(fmt);
  window = qrows * (rowbytes + 16) + 12 * 1024 <= kSubtreeLds ? 0 : kWindowLds / qrows;
  for (top = std::max(std::min(std::max(8 - lg, 0), first), depth - 1 - kSubtreeLevels); top <= depth - 1; ++top)
    if (subtree_fits(window > 0 ? window : rowbytes, qrows, depth, top)) return true;
  return false;
}

hipError_t launch_walk_subtree(int fmt, const SubtreeArgs& a, hipStream_t s) {
  if (a.n_epoch < 1 || a.nt < 1 || a.nt > kMaxTiles || a.dp < 128 || a.dp % 128 != 0 || a.nb < 0 ||
      a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots || a.top < a.nb ||
      a.first < a.top || a.first > a.depth - 1 || a.depth > 31 || a.window < 0 || a.window % 128 != 0 ||
      a.n_epoch > (int64_t(1) << a.depth) ||
      !subtree_fits(a.window > 0 ? a.window : a.dp * esz_of(fmt), a.qrows, a.depth, a.top))
    return hipErrorInvalidValue;
  switch (fmt) {
    case GT_POOL_BF16: return launch_subtree_fmt<GT_POOL_BF16>(a, s);
    case GT_POOL_FP8E4M3: return launch_subtree_fmt<GT_POOL_FP8E4M3>(a, s);
    case GT_POOL_F32: return launch_subtree_fmt<GT_POOL_F32>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gt
