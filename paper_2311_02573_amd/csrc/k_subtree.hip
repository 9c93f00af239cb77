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
#include <type_traits>

#include "gt_internal.h"
#include "gt_device.h"
#include "gt_mma.h"
#include "gt_numerics.h"

namespace gt {

namespace {

constexpr int kSubtreeThreads = 512;
constexpr int kSubtreeLevels = 11;        // most levels below a subtree's root pool
constexpr int kSubtreeLds = 160 * 1024;
constexpr int kWaves = kSubtreeThreads / 64;
constexpr int kWindowChunks = 8 * kWaves; // of a window, where a tile's rows do not fit


// LDS: the query rows, then the lists of (pool, mask) entries.  A list of level
// l holds at most 2^(l - top) entries; consecutive levels alternate between
// two lists, the larger sized for level depth - 2 (the last level's entries
// leave the workgroup).
__host__ __device__ inline int list_entries(int depth, int top, int which) {
  const int m = depth - 2 - top - which;  // which: 0 the larger, 1 the smaller
  return m < 0 ? 1 : 1 << m;
}
__host__ __device__ inline int subtree_lds(int query_lds, int depth, int top) {
  return query_lds + (list_entries(depth, top, 0) + list_entries(depth, top, 1)) * 12 + 64;
}
// The query rows, padded by 16 bytes each (bank spread), or two windows of them.
__host__ __device__ inline int query_lds_of(int rowbytes, int qrows, int window) {
  return window > 0 ? 2 * qrows * (window + 16) : qrows * (rowbytes + 16);
}

// The columns of one window of the query rows, from byte `from`, in two parts: 8
// chunks a wave to registers, and from there to LDS.  (Not direct loads: with
// one in flight the compiler lets no LDS read go before all of a wave's loads.)
template <int NQB>
struct WindowCopy {
  static constexpr int M = kWindowChunks / kWaves, CPR = kWindowChunks / (16 * NQB);  // chunks of a wave, row
  uint4 v[M];
  __device__ __forceinline__ void load(const unsigned char* src, int rowbytes, int from, int wave, int lane) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int row = (wave * M + m) / CPR, c = (wave * M + m) % CPR * kStageChunk;
      const int byte = from + c + 16 * lane;
      v[m] = ld_global16(src + (size_t)row * rowbytes + (byte < rowbytes ? byte : 0));
    }
  }
  __device__ __forceinline__ void store(unsigned char* buf, int wave, int lane) const {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int row = (wave * M + m) / CPR, c = (wave * M + m) % CPR * kStageChunk;
      *reinterpret_cast<uint4*>(buf + row * (CPR * kStageChunk + 16) + c + 16 * lane) = v[m];
    }
  }
};

// Products of one 16-row group with the staged query columns: nsteps 64-byte
// steps from `row` against `brow`.  The matrix-core operand of lane 16 g + i is
// row i, 16-byte chunk g; loads in that order touch four lines with each four
// lanes.  kQuads: four lanes take 64 contiguous bytes of a row (lanes 4 R ..
// 4 R + 3: row R), and the operand comes from lane 4 i + g (bp).  Kernel with /
// without (us): float8 of 300,007 x 777, 257 queries 97 / 106; float32 of
// 100,003 x 300, 65 queries 51 / 55.  Not where the passing between lanes costs
// as much: one block of queries (bfloat16, 2^20 x 1000, 23 / 22), windows
// (float8, 65,536 x 3000, 64 / 54), bfloat16 (2^19 x 256, 512 queries 180 / 172,
// though 2^20 x 1000, 128 queries 130 / 136).
template <int FMT, int NQB, bool WIN>
constexpr bool kQuads = FMT != GT_POOL_BF16 && NQB >= 2 && !WIN;

__device__ __forceinline__ uint4 by_quads(const uint4& x, int bp) {
  return make_uint4((uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)x.x),
                    (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)x.y),
                    (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)x.z),
                    (uint32_t)__builtin_amdgcn_ds_bpermute(bp, (int)x.w));
}

// The first `left` of C steps of G groups against the staged columns at `b`.
// The operands of a unit (a step, or the two of a float8 product) are read
// while the one before it is multiplied: its own reads take longer than its
// products.  Walk with / without (us): bfloat16 2^19 x 256, 512 queries 168 /
// 208; 2^20 x 1000, 64 queries 77 / 85; float8 300,007 x 777, 257 queries 112 /
// 126, and 96 with 128 columns to a product.
template <int FMT, int NQB, bool WIN, int G, int C>
__device__ __forceinline__ void step_products(const uint4 (&x)[G][C], const unsigned char* b, int rs,
                                              int left, int bp, f32x4 (&acc)[G][NQB]) {
  constexpr int S = FMT == GT_POOL_FP8E4M3 ? 2 : 1;  // steps of a unit
  constexpr int U = FMT == GT_POOL_FP8E4M3 ? 2 : 4;  // steps of 128 columns: rows hold whole ones
  uint4 p[2][G][S], q[2][NQB][S];
  auto read = [&](int c, int o) {
#pragma unroll
    for (int u = 0; u < S; ++u) {
#pragma unroll
      for (int k = 0; k < G; ++k) p[o][k][u] = kQuads<FMT, NQB, WIN> ? by_quads(x[k][c + u], bp) : x[k][c + u];
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) q[o][qb][u] = ld_lds16(b + qb * 16 * rs + 64 * (c + u));
    }
  };
  if (left > 0) read(0, 0);
#pragma unroll
  for (int c = 0; c < C; c += S)
    if (c / U * U < left) {
      const int o = c / S & 1;
      if (c % U + S < U || (c + S < C && c + S < left)) read(c + S, o ^ 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int k = 0; k < G; ++k) {
          if constexpr (S == 2)
            mma_f8_16x16x128(p[o][k][0], p[o][k][1], q[o][qb][0], q[o][qb][1], acc[k][qb]);
          else
            mma16x16<FMT>(p[o][k][0], q[o][qb][0], acc[k][qb]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
}

// C steps of a row from step s0 (the last one again past the row's end).
template <int C>
__device__ __forceinline__ void load_steps(uint4 (&x)[C], const unsigned char* row, int s0, int nsteps) {
#pragma unroll
  for (int c = 0; c < C; c += 4)
    if (c == 0 || s0 + c < nsteps) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int st = s0 + c + u < nsteps ? s0 + c + u : nsteps - 1;
        x[c + u] = ld_global16(row + 64 * st);
      }
    }
}

// Products of G 16-row groups of each wave where the query columns pass
// through LDS in windows (wg: windows multiplied so far; on entry `copy` holds
// the first).  The loads of a block of C steps are issued before the products
// of the one before it, across windows too, and the next window is on its way
// while one is multiplied: without either, a level of 2048 bfloat16 columns
// took 21 us, 12 of them for copying 256 KB.  Walk of 2^17 x 2048, 256 queries:
// 82 us, 152 before.  (Blocks are what the registers hold of bfloat16 and float32
// rows: a larger one spills, 98 us.  Float8, whose operands are read two steps at
// a time, spills 7 to 29 registers at these sizes.)
template <int FMT, int NQB, int G>
__device__ __forceinline__ void windowed_products(const unsigned char* const (&row)[G], bool any,
                                                  unsigned char* lds, const unsigned char* qsrc,
                                                  int brow, int rowbytes, int bp, int wave, int lane,
                                                  uint32_t& wg, WindowCopy<NQB>& copy,
                                                  f32x4 (&acc)[G][NQB]) {
  constexpr int W = WindowCopy<NQB>::CPR * kStageChunk, RS = W + 16, BUF = 16 * NQB * RS;
  constexpr int C = G == 2 ? 4 : NQB == 4 ? 8 : 16;  // steps of a block and group (what the registers hold)
  constexpr int NB = W / (64 * C);     // blocks of a window
  const int nsteps = rowbytes / 64, nblk = (nsteps + C - 1) / C;
  uint4 x0[G][C], x1[G][C];
  auto load = [&](uint4 (&x)[G][C], int i) {
#pragma unroll
    for (int k = 0; k < G; ++k) load_steps<C>(x[k], row[k], i * C, nsteps);
  };
  auto block = [&](const uint4 (&cu)[G][C], uint4 (&nx)[G][C], int i) {
    if (i % NB == 0) {
      copy.store(lds + wg % 2u * BUF, wave, lane);  // (all are done with the window before the last)
      __syncthreads();
      const int next = (i / NB + 1) * W;
      copy.load(qsrc, rowbytes, next < rowbytes ? next : 0, wave, lane);
      ++wg;
    }
    if (!any) return;
    if (i + 1 < nblk) load(nx, i + 1);
    __builtin_amdgcn_sched_barrier(0);
    step_products<FMT, NQB, true, G, C>(cu, lds + (wg - 1u) % 2u * BUF + brow + i % NB * (64 * C), RS,
                                  nsteps - i * C, bp, acc);
  };
  if (any) load(x0, 0);
  for (int i = 0; i < nblk; i += 2) {
    block(x0, x1, i);
    if (i + 1 < nblk) block(x1, x0, i + 1);
  }
}

// A wave takes 16 pool rows at a time (16 pools of the first level, then both
// children of 8 entries).
// Scores, thresholds and decisions are those of the level kernels' direct
// test (the sums run over the same products in another order, which the
// thresholds' slack covers).
// WIN: the tile's query rows do not fit beside the lists and pass through LDS
// in windows; the waves then step through the windows together, with two
// groups each where there are more than 8.
template <int FMT, int NQB, bool WIN>
__global__ __launch_bounds__(kSubtreeThreads, 1) void k_walk_subtree(SubtreeArgs a) {
  using F = WalkFmt<FMT>;
  constexpr int TQ = F::TQ, NW = kWaves;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ uint32_t cnt[GT_MAX_LEVELS], prs[GT_MAX_LEVELS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  const int rs = (WIN ? a.window : rowbytes) + 16;  // LDS row stride (bank spread)
  const int cap0 = list_entries(D, a.top, 0);
  uint64_t* const mask0 = reinterpret_cast<uint64_t*>(lds + query_lds_of(rowbytes, 16 * NQB, WIN ? a.window : 0));
  uint64_t* const mask1 = mask0 + cap0;
  uint32_t* const node0 = reinterpret_cast<uint32_t*>(mask1 + list_entries(D, a.top, 1));
  uint32_t* const node1 = node0 + cap0;
  if (tid < GT_MAX_LEVELS) cnt[tid] = prs[tid] = 0u;
  const unsigned char* qsrc =
      reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)t * TQ * rowbytes;
  WindowCopy<NQB> copy;
  if constexpr (WIN)
    copy.load(qsrc, rowbytes, 0, wave, lane);
  else
    stage_rows<16 * NQB, kWaves>(lds, qsrc, rowbytes, wave, lane);
  uint32_t windows = 0;  // multiplied so far
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

  wait_loads();

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
                                 (size_t)((int64_t(1) << l) - 1) * rowbytes + 16 * (kQuads<FMT, NQB, WIN> ? lane & 3 : g4);
    uint32_t pairs = 0;
    const int nsteps = rowbytes / 64;

    struct Group {
      uint32_t node;             // of row c16, and its live queries
      uint64_t pm;
      const unsigned char* row;  // this lane loads
    };
    // The 16 rows from row gf (gf >= n: any row, no queries).
    auto group = [&](uint32_t gf) {
      Group g;
      const uint32_t r = gf + (uint32_t)c16, rr = r < n ? r : gf < n ? gf : 0u;
      if (head) {
        g.node = root + rr;
        g.pm = r < n ? tmask : 0ull;
      } else {
        g.node = 2u * in_node[rr >> 1] + (rr & 1u);
        g.pm = r < n && ((int64_t)g.node << shift) < a.n_epoch ? in_mask[rr >> 1] : 0ull;
      }
      const uint32_t rn = kQuads<FMT, NQB, WIN> ? (uint32_t)__shfl((int)g.node, lane >> 2, 64) : g.node;
      g.row = level + (size_t)rn * rowbytes;
      return g;
    };
    auto clear = [&](f32x4 (&acc)[NQB]) {
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[qb][x] = 0.0f;
    };
    // The group's surviving entries, to the next list or the frontier.
    auto emit = [&](const Group& g, const f32x4 (&acc)[NQB]) {
      // register x of lane j: row 4 (j / 16) + x, query 16 qb + j % 16; lane
      // r < 16 ends with row r's mask
      uint64_t mine = 0ull;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        uint64_t part = 0ull;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const uint64_t bal = __ballot(acc[qb][x] >= th[qb]);
          part |= ((bal >> (16 * ((lane & 15) >> 2))) & 0xffffull) << (16 * qb);
        }
        if ((lane & 3) == x) mine = part;
      }
      mine = lane < 16 ? (mine & g.pm) : 0ull;
      if (a.bitmap && lane < 16 && g.pm) {
        const uint64_t row = ((uint64_t)1 << l) - 1 + g.node;
        atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
      }
      if (lane < 16) pairs += (uint32_t)__popcll(g.pm);
      const uint64_t bal = __ballot(mine != 0ull);
      if (bal == 0ull) return;
      const uint32_t rank = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      uint32_t base = 0;
      if (l < D - 1) {
        if (lane == 0) base = atomicAdd(&cnt[l], (uint32_t)__popcll(bal));
        base = __shfl(base, 0, 64);
        if (mine) {
          on[base + rank] = g.node;
          om[base + rank] = mine;
        }
      } else {
        if (lane == 0)
          base = atomicAdd(&a.lvl_count[(size_t)l * kMaxSlots + slot], (uint32_t)__popcll(bal));
        base = __shfl(base, 0, 64);
        if (mine) {
          if (base + rank < a.bcap) {
            const size_t o = (size_t)slot * a.bcap + base + rank;
            a.out_node[o] = g.node;
            a.out_mask[o] = mine;
          } else {
            atomicOr(a.over, 1u);
          }
        }
      }
    };

    if constexpr (WIN) {
      // every wave takes part in every round, with one or two groups
      const int b0 = c16 * rs + 16 * g4;
      auto round = [&](uint32_t g0, auto ng) {
        constexpr int G = decltype(ng)::value;
        Group g[G];
        const unsigned char* row[G];
        f32x4 acc[G][NQB];
#pragma unroll
        for (int k = 0; k < G; ++k) {
          g[k] = group(16u * (g0 + (uint32_t)(wave + k * NW)));
          row[k] = g[k].row;
          clear(acc[k]);
        }
        windowed_products<FMT, NQB, G>(row, 16u * (g0 + (uint32_t)wave) < n, lds, qsrc, b0, rowbytes, bp,
                                       wave, lane, windows, copy, acc);
#pragma unroll
        for (int k = 0; k < G; ++k) emit(g[k], acc[k]);
      };
      for (uint32_t g0 = 0; 16u * g0 < n; g0 += 2 * NW) {
        if (16u * (g0 + (uint32_t)NW) < n)
          round(g0, std::integral_constant<int, 2>());
        else
          round(g0, std::integral_constant<int, 1>());
      }
    } else {
      constexpr int C = FMT == GT_POOL_FP8E4M3 ? 16 : 32;  // steps in flight
      for (uint32_t gw = (uint32_t)wave; 16u * gw < n; gw += NW) {
        const Group g = group(16u * gw);
        f32x4 acc[1][NQB];
        clear(acc[0]);
        for (int s0 = 0; s0 < nsteps; s0 += C) {
          uint4 x[1][C];
          load_steps<C>(x[0], g.row, s0, nsteps);
          __builtin_amdgcn_sched_barrier(0);
          step_products<FMT, NQB, false, 1, C>(x, brow + 64 * s0, rs, nsteps - s0, bp, acc);
        }
        emit(g, acc[0]);
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
  const int bytes = subtree_lds(query_lds_of(a.dp * WalkFmt<FMT>::ESZ, a.qrows, WIN ? a.window : 0), a.depth, a.top);
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

bool subtree_fits(int query_lds, int depth, int top) {
  return depth - 1 - top <= kSubtreeLevels && subtree_lds(query_lds, depth, top) + 512 <= kSubtreeLds;
}

}  // namespace

// As many subtrees as give every CU of an XCD at most one workgroup over all
// tiles (each holds a CU's registers; 2^8 for one tile of a full tree), but
// one for every XCD, and
// more, smaller ones where the frontier lists would not fit beside the query
// rows.  Query rows that do not fit with the largest lists are windowed.
bool subtree_shape(int fmt, int dp, int nt, int qrows, int depth, int first, int64_t n_epoch, int n_cu,
                   int& top, int& window) {
  if (first > depth - 1 || depth > 31 || n_epoch < 1) return false;
  auto per_xcd = [&](int t) { return ((((n_epoch - 1) >> (depth - t)) + kXcds) / kXcds) * nt; };
  int most = 0;
  while (most < depth - 1 && per_xcd(most + 1) <= std::max(n_cu / kXcds, nt)) ++most;
  const int rowbytes = dp * esz_of(fmt);
  window = qrows * (rowbytes + 16) + 12 * 1024 <= kSubtreeLds ? 0 : kWindowChunks / qrows * kStageChunk;
  for (top = std::max(std::min(most, first), depth - 1 - kSubtreeLevels); top <= depth - 1; ++top)
    if (subtree_fits(query_lds_of(rowbytes, qrows, window), depth, top)) return true;
  return false;
}

hipError_t launch_walk_subtree(int fmt, const SubtreeArgs& a, hipStream_t s) {
  if (a.n_epoch < 1 || a.nt < 1 || a.nt > kMaxTiles || a.dp < 128 || a.dp % 128 != 0 || a.nb < 0 ||
      a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots || a.top < a.nb ||
      a.first < a.top || a.first > a.depth - 1 || a.depth > 31 || a.qrows < 16 ||
      (a.window != 0 && a.window != kWindowChunks / a.qrows * kStageChunk) ||
      a.n_epoch > (int64_t(1) << a.depth) ||
      !subtree_fits(query_lds_of(a.dp * esz_of(fmt), a.qrows, a.window), a.depth, a.top))
    return hipErrorInvalidValue;
  switch (fmt) {
    case GT_POOL_BF16: return launch_subtree_fmt<GT_POOL_BF16>(a, s);
    case GT_POOL_FP8E4M3: return launch_subtree_fmt<GT_POOL_FP8E4M3>(a, s);
    case GT_POOL_F32: return launch_subtree_fmt<GT_POOL_F32>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gt
