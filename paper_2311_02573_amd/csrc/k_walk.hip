// The level-wise binary-splitting walk (paper Sec. 2, Alg. 1; one level per
// round as in the pruning analysis of Sec. 4), the exact leaf test, the
// float64 recheck and the result compaction.
//
// Frontier representation.  Queries are grouped in tiles of TQ (64 for bf16 /
// float8 pools, 32 for float32 pools).  The frontier of a tile at level l is a
// list of entries (pool j, mask): pool j of level l survived for the queries
// whose bits are set.  One level step reads both children of every entry (two
// adjacent rows), scores them against all TQ queries of the tile with matrix
// cores, and keeps child c for query b iff the parent's bit b is set and the
// score reaches the query's lowered threshold tau'_b.  Children with a
// non-empty mask are appended to the tile's next frontier.
#include <math.h>

#include "gt_internal.h"
#include "gt_device.h"
#include "gt_mma.h"
#include "gt_numerics.h"

namespace gt {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

// One 16-byte slice of a row (per lane) against the same slice of a query:
// bf16: one 32x32x16 step; float8: two 32x32x16 steps; float32: four 32x32x2
// steps.  Lanes 0-31 and 32-63 carry different slices, and the A (pool) and B
// (query) operands of a lane always hold the same dimensions, so the sum over
// all slices is the full dot product whatever order the hardware uses inside.
template <int FMT>
__device__ __forceinline__ void mma16(const uint4& a, const uint4& b, f32x16& acc);

template <>
__device__ __forceinline__ void mma16<GT_POOL_BF16>(const uint4& a, const uint4& b, f32x16& acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma16<GT_POOL_FP8E4M3>(const uint4& a, const uint4& b,
                                                       f32x16& acc) {
  const long a0 = (long)(((unsigned long)a.y << 32) | a.x);
  const long a1 = (long)(((unsigned long)a.w << 32) | a.z);
  const long b0 = (long)(((unsigned long)b.y << 32) | b.x);
  const long b1 = (long)(((unsigned long)b.w << 32) | b.z);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a0, b0, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a1, b1, acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma16<GT_POOL_F32>(const uint4& a, const uint4& b, f32x16& acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// Exclusive prefix pre[0..n] of the entry counts of bucket slots
// slot0 .. slot0 + n - 1 (n <= 1024), computed by wave 0.  Dense input: every
// pool of the bucket (1 << shift of them) for the tile's queries.
__device__ __forceinline__ void slot_prefix(uint32_t* pre, int n, int slot0, int nt, int dense,
                                            int shift, const uint64_t* tile_mask,
                                            const uint32_t* counts, uint32_t cap) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const int per_lane = (n + 63) / 64;
    const int s0 = lane * per_lane;
    uint32_t loc[16];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int sl = s0 + i;
      uint32_t c = 0;
      if (i < per_lane && sl < n) {
        const int gs = slot0 + sl;
        c = dense ? (tile_mask[gs % nt] ? (1u << shift) : 0u) : min(counts[gs], cap);
      }
      loc[i] = sum;
      sum += c;
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    const uint32_t excl = incl - sum;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int sl = s0 + i;
      if (i < per_lane && sl < n) pre[sl] = excl + loc[i];
    }
    if (lane == 63) pre[n] = incl;
  }
  __syncthreads();
}

// The f8f6f4 form of 32x32 products: 32 bytes per lane as in mma_f8_16x16x128.
__device__ __forceinline__ void mma_f8_32x32x64(const uint4& a0, const uint4& a1, const uint4& b0,
                                                const uint4& b1, f32x16& acc) {
  acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(pack32(a0, a1), pack32(b0, b1), acc, 0, 0,
                                                       0, 0, 0, 0);
}

// Index i with pre[i] <= g < pre[i + 1] (pre ascending, n + 1 values).
__device__ __forceinline__ int find_slot(const uint32_t* pre, int n, uint32_t g) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= g) lo = mid; else hi = mid;
  }
  return lo;
}

// Entries [lo, hi) of a bucket's n that part m of c takes: whole groups (a part
// that ends inside one costs a wave step for each side of it), dealt by
// buckets in rotation so that the parts' totals stay even.  Level kernel on
// 2^20 x 1000 float32 pools, 256 queries, nine levels: 845 us, 1050 with equal
// shares; even at 1024 queries, and worse for the smaller groups of k_walk_sub
// (256 queries 173 / 160), which keeps equal shares.
__device__ __forceinline__ void bucket_share(uint32_t n, int m, int c, int bucket, uint32_t group,
                                             uint32_t& lo, uint32_t& hi) {
  const uint32_t g = (n + group - 1) / group, rot = (uint32_t)(bucket % c);
  auto cut = [&](int k) {
    return k <= 0 ? 0u : k >= c ? g : (uint32_t)(((uint64_t)g * (uint32_t)k + rot) / (uint32_t)c);
  };
  lo = min(n, cut(m) * group);
  hi = min(n, cut(m + 1) * group);
}

constexpr int kPipe = 8;  // 64-byte steps of a lane's two rows fetched ahead

// One level step of the sparse walk.  Workgroup -> XCD x = blockIdx % 8 (the
// hardware deals workgroups to XCDs round robin), which owns an even
// contiguous range of the buckets that hold rows (with ranges of all buckets,
// a tree filled to 57% left three XCDs idle: the leaf of 257 queries, n =
// 300,007 of 2^19, took 143 us, now 96).  Within an XCD the workgroups split the query tiles; when
// there are fewer tiles than workgroups, the c workgroups of a tile each take
// part m of every bucket.  Every workgroup goes through its buckets in
// order, so at any moment the XCD's workgroups read the same subtrees for
// different tiles and the repeated pool rows are found in L2.
template <int FMT, int NSTEPS>
__global__ __launch_bounds__(kWalkThreads, 1) void k_walk_level(WalkLevelArgs a) {
  using F = WalkFmt<FMT>;
  constexpr int TQ = F::TQ;
  constexpr int NQB = TQ / 16;  // 16-query column blocks
  __shared__ __attribute__((aligned(16))) unsigned char qlds[TQ * (F::MAXDP * F::ESZ + 16)];
  static_assert(kMaxBucketsPerXcd <= 64, "one bucket per lane of wave 0");
  __shared__ uint32_t gpre[kMaxBucketsPerXcd + 1];
  __shared__ uint32_t glo[kMaxBucketsPerXcd], ghi[kMaxBucketsPerXcd];
  // Thresholds of the tile.  Read from LDS in the loop: a value loaded from
  // global memory before the loop would make the compiler wait for every
  // load in flight at its first use in each iteration.
  __shared__ float thr_lds[TQ];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nwaves = blockDim.x >> 6;
  const int rowbytes = a.dp * F::ESZ;
  const int rs = rowbytes + 16;           // LDS row stride (bank spread)
  // 64-byte steps per row; a compile-time count (the common padded widths)
  // unrolls the stage loop completely
  const int nsteps = NSTEPS > 0 ? NSTEPS : rowbytes / 64;
  const int c16 = lane & 15, g4 = lane >> 4;

  const int xs = a.nbu < kXcds ? a.nbu : kXcds;
  const int x = blockIdx.x % kXcds;
  const int b0 = x * a.nbu / xs, R = (x + 1) * a.nbu / xs - b0;  // this XCD's buckets
  const int W = gridDim.x / kXcds, j = blockIdx.x / kXcds;
  if (x >= xs) return;
  int t0, tstep, m, c;
  if (a.nt <= W) {
    t0 = j % a.nt;
    tstep = a.nt;
    m = j / a.nt;
    c = (W - 1 - t0) / a.nt + 1;
  } else {
    t0 = j;
    tstep = W;
    m = 0;
    c = 1;
  }
  const int bshift = a.level - a.nb;  // node -> bucket
  unsigned long long pairs = 0;

  for (int t = t0; t < a.nt; t += tstep) {
    const uint64_t tmask = a.tile_mask[t];
    __syncthreads();  // LDS of the previous tile no longer read
    if (wave == 0) {  // groups of this workgroup's share of each bucket (R <= 16)
      uint32_t ng = 0, lo = 0, hi = 0;
      if (lane < R && tmask) {
        const uint32_t n = a.dense ? (1u << bshift)
                                   : min(a.in_count[(size_t)(b0 + lane) * a.nt + t], (uint32_t)a.bcap);
        bucket_share(n, m, c, b0 + lane, kGroupEntries, lo, hi);
        ng = (hi - lo + kGroupEntries - 1) / kGroupEntries;
      }
      uint32_t incl = ng;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane < R) {
        gpre[lane] = incl - ng;
        glo[lane] = lo;
        ghi[lane] = hi;
      }
      if (lane == 63) gpre[R] = incl;
    }
    __syncthreads();
    const uint32_t gtot = gpre[R];
    if (gtot == 0) continue;
    stage_rows<TQ, kWalkThreads / 64>(
        qlds, reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)t * TQ * rowbytes, rowbytes,
        __builtin_amdgcn_readfirstlane(wave), lane);
    if (tid < TQ) {
      const int qi = t * TQ + tid;
      float th = a.thr[qi];
      if (FMT == GT_POOL_FP8E4M3) th = ldexpf(th * kFp8ThrFactor, -(a.qexp[qi] + a.lexp));
      thr_lds[tid] = th;
    }
    wait_loads();
    __syncthreads();

    // entries of group gg held by this lane: rows c16 (entry c16 / 2) and
    // 16 + c16 (entry 8 + c16 / 2) of the group's 32 child rows
    auto fetch = [&](uint32_t gg, uint32_t& p0, uint64_t& pm0, uint32_t& p1, uint64_t& pm1,
                     uint32_t& slot) {
      const int r = find_slot(gpre, R, gg);
      const uint32_t e0 = glo[r] + (gg - gpre[r]) * kGroupEntries + (c16 >> 1);
      const uint32_t e1 = e0 + 8;
      const uint32_t hi = ghi[r];
      const uint32_t bk = (uint32_t)(b0 + r);
      slot = bk * (uint32_t)a.nt + (uint32_t)t;
      // Loads are issued in both input modes and for padding lanes (at the
      // group's first entry, always valid) so that no branch separates them
      // from their use; dense input (every pool of the bucket) ignores them.
      const uint32_t ef = e0 - (c16 >> 1);
      const uint32_t i0 = e0 < hi ? e0 : ef, i1 = e1 < hi ? e1 : ef;
      const size_t at0 = input_entry(a.dense, slot, a.bcap, i0), at1 = input_entry(a.dense, slot, a.bcap, i1);
      const uint32_t ld0 = a.in_node[at0], ld1 = a.in_node[at1];
      const uint64_t lm0 = a.in_mask[at0], lm1 = a.in_mask[at1];
      const uint32_t first = bk << bshift;
      p0 = a.dense ? first + i0 : ld0;
      p1 = a.dense ? first + i1 : ld1;
      pm0 = e0 < hi ? (a.dense ? tmask : lm0) : 0ull;
      pm1 = e1 < hi ? (a.dense ? tmask : lm1) : 0ull;
    };
    // Rows this lane loads.  A load instruction gives each 4 consecutive
    // lanes 64 contiguous bytes of one row (lanes 4R .. 4R+3: row R of the
    // block, entry R / 2, child R % 2), so each lane quad touches one cache
    // line; the matrix-core layout (row = lane % 16) would give every quad
    // four rows.  p0 / p1 are the entries of this lane's output rows
    // (c16 / 2 and 8 + c16 / 2); lane 2e holds entry e.
    auto rows_of = [&](uint32_t p0, uint32_t p1, const unsigned char*& r0,
                       const unsigned char*& r1) {
      const int src = 2 * (lane >> 3);
      const uint32_t q0 = (uint32_t)__shfl((int)p0, src, 64);
      const uint32_t q1 = (uint32_t)__shfl((int)p1, src, 64);
      const uint32_t ch = (uint32_t)((lane >> 2) & 1);
      const unsigned char* base = reinterpret_cast<const unsigned char*>(a.child_rows) + 16 * (lane & 3);
      r0 = base + (size_t)(2u * q0 + ch) * rowbytes;
      r1 = base + (size_t)(2u * q1 + ch) * rowbytes;
    };
    // Loaded slice -> matrix-core operand: lane 16 g + i takes row i, 16-byte
    // chunk g of the step, which the load left in lane 4 i + g.
    const int bp_addr = 4 * (4 * c16 + g4);
    auto to_mfma = [&](const uint4& v) {
      uint4 r;
      r.x = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.x);
      r.y = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.y);
      r.z = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.z);
      r.w = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.w);
      return r;
    };
    // The steps of consecutive groups form one pipeline: while a stage is
    // multiplied, the next one (possibly the first stage of the wave's next
    // group) is in flight.  Loads are unconditional (steps past a row re-read
    // its last step) so the number in flight is static and the compiler waits
    // only for the stage it is about to use.
    const int slast = nsteps - 1;
    uint4 bA0[kPipe], bA1[kPipe], bB0[kPipe], bB1[kPipe];
    uint32_t np0 = 0, np1 = 0, nslot = 0;
    uint64_t npm0 = 0ull, npm1 = 0ull;
    if ((uint32_t)wave < gtot) {
      fetch(wave, np0, npm0, np1, npm1, nslot);
      const unsigned char *r0, *r1;
      rows_of(np0, np1, r0, r1);
#pragma unroll
      for (int u = 0; u < kPipe; ++u) {
        const int st = u < slast ? u : slast;
        bA0[u] = ld_global16(r0 + 64 * st);
        bA1[u] = ld_global16(r1 + 64 * st);
      }
    }
    bool pend = false;
    uint32_t pend_child = 0, pend_slot = 0;
    uint64_t pend_mask = 0ull, pend_bal = 0ull;

    for (uint32_t gg = wave; gg < gtot; gg += nwaves) {
      const uint32_t p0 = np0, p1 = np1, slot = nslot;
      const uint64_t pm0 = npm0, pm1 = npm1;
      const uint32_t child0 = 2u * p0 + (uint32_t)(lane & 1);
      const uint32_t child1 = 2u * p1 + (uint32_t)(lane & 1);
      const unsigned char *arow0, *arow1;
      rows_of(p0, p1, arow0, arow1);
      const unsigned char* brow = qlds + c16 * rs + 16 * g4;
      const bool has_next = gg + nwaves < gtot;
      // the next group's entries (this group's again when there is none)
      fetch(has_next ? gg + nwaves : gg, np0, npm0, np1, npm1, nslot);
      // reserve output slots for the previous group; the reply is awaited
      // only after this group's matrix work
      if (a.bitmap && lane < 16) {
        if (pm0) {
          const uint64_t row = (uint64_t)a.bit_base + child0;
          atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
        }
        if (pm1) {
          const uint64_t row = (uint64_t)a.bit_base + child1;
          atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
        }
      }
      uint32_t pend_base = 0;
      if (pend && lane == 0) pend_base = atomicAdd(&a.out_count[pend_slot], (uint32_t)__popcll(pend_bal));

      f32x4 acc[2][NQB];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[rb][qb][i] = 0.0f;

      auto step = [&](const uint4& l0, const uint4& l1, int s) {
        const uint4 x0 = to_mfma(l0), x1 = to_mfma(l1);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const uint4 bq = ld_lds16(brow + qb * 16 * rs + 64 * s);
          mma16x16<FMT>(x0, bq, acc[0][qb]);
          mma16x16<FMT>(x1, bq, acc[1][qb]);
        }
      };
      // float8: steps s and s + 1 in one 16x16x128 product
      auto step2 = [&](const uint4& l0a, const uint4& l1a, const uint4& l0b, const uint4& l1b,
                       int s) {
        const uint4 x0a = to_mfma(l0a), x1a = to_mfma(l1a);
        const uint4 x0b = to_mfma(l0b), x1b = to_mfma(l1b);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const uint4 bqa = ld_lds16(brow + qb * 16 * rs + 64 * s);
          const uint4 bqb = ld_lds16(brow + qb * 16 * rs + 64 * (s + 1));
          mma_f8_16x16x128(x0a, x0b, bqa, bqb, acc[0][qb]);
          mma_f8_16x16x128(x1a, x1b, bqa, bqb, acc[1][qb]);
        }
      };
#pragma unroll
      for (int s0 = 0; s0 < nsteps; s0 += 2 * kPipe) {
#pragma unroll
        for (int u = 0; u < kPipe; ++u) {
          const int st = s0 + kPipe + u < slast ? s0 + kPipe + u : slast;
          bB0[u] = ld_global16(arow0 + 64 * st);
          bB1[u] = ld_global16(arow1 + 64 * st);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FMT == GT_POOL_FP8E4M3) {
          // (a float8 row has an even number of 64-byte steps)
#pragma unroll
          for (int u = 0; u < kPipe; u += 2)
            if (s0 + u < nsteps) step2(bA0[u], bA1[u], bA0[u + 1], bA1[u + 1], s0 + u);
        } else {
#pragma unroll
          for (int u = 0; u < kPipe; ++u)
            if (s0 + u < nsteps) step(bA0[u], bA1[u], s0 + u);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
          // next stage of this group, or the first stage of the next group
          const bool same = s0 + 2 * kPipe < nsteps;
          if (!same && pend) {
            // Survivors of the previous group go out here, before the next
            // group's loads are issued: waiting for the slot reservation then
            // only waits for loads that the next stage needs anyway.
            pend_base = __shfl(pend_base, 0, 64);
            if (lane < 32 && pend_mask) {
              const uint32_t pos = pend_base + (uint32_t)__popcll(pend_bal & ((1ull << lane) - 1ull));
              if (pos < a.bcap) {
                const size_t o = (size_t)pend_slot * a.bcap + pos;
                a.out_node[o] = pend_child;
                a.out_mask[o] = pend_mask;
              } else {
                atomicOr(a.over, 1u);
              }
            }
            pend = false;
          }
          const unsigned char *r0 = arow0, *r1 = arow1;
          if (!same) rows_of(np0, np1, r0, r1);
          const int sf = same ? s0 + 2 * kPipe : 0;
#pragma unroll
          for (int u = 0; u < kPipe; ++u) {
            const int st = sf + u < slast ? sf + u : slast;
            bA0[u] = ld_global16(r0 + 64 * st);
            bA1[u] = ld_global16(r1 + 64 * st);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FMT == GT_POOL_FP8E4M3) {
#pragma unroll
          for (int u = 0; u < kPipe; u += 2)
            if (s0 + kPipe + u < nsteps)
              step2(bB0[u], bB1[u], bB0[u + 1], bB1[u + 1], s0 + kPipe + u);
        } else {
#pragma unroll
          for (int u = 0; u < kPipe; ++u)
            if (s0 + kPipe + u < nsteps) step(bB0[u], bB1[u], s0 + kPipe + u);
        }
        __builtin_amdgcn_sched_barrier(0);
      }

      // Child row r (lane r < 32): block r / 16, register r % 4, lane group
      // (r % 16) / 4; column block qb supplies query bits 16 qb .. 16 qb + 15.
      const int gsel = 16 * ((lane & 15) >> 2);
      uint64_t mine = 0ull;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint64_t part = 0ull;
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            const uint64_t bal = __ballot(acc[rb][qb][i] >= thr_lds[16 * qb + c16]);
            part |= ((bal >> gsel) & 0xffffull) << (16 * qb);
          }
          if ((lane >> 4) == rb && (lane & 3) == i) mine = part;
        }
      const uint64_t pm_own = lane < 16 ? pm0 : pm1;
      mine = lane < 32 ? (mine & pm_own) : 0ull;
      if (lane < 32) pairs += (unsigned long long)__popcll(pm_own);
      pend_bal = __ballot(mine != 0ull);
      pend = pend_bal != 0ull;
      pend_child = lane < 16 ? child0 : child1;
      pend_mask = mine;
      pend_slot = slot;
    }
    if (pend) {
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&a.out_count[pend_slot], (uint32_t)__popcll(pend_bal));
      base = __shfl(base, 0, 64);
      if (lane < 32 && pend_mask) {
        const uint32_t pos = base + (uint32_t)__popcll(pend_bal & ((1ull << lane) - 1ull));
        if (pos < a.bcap) {
          const size_t o = (size_t)pend_slot * a.bcap + pos;
          a.out_node[o] = pend_child;
          a.out_mask[o] = pend_mask;
        } else {
          atomicOr(a.over, 1u);
        }
      }
    }
  }
  if (a.stat_pairs) {
    for (int o = 32; o >= 1; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0 && pairs)
      stat_add(a.stat_pairs, GT_MAX_LEVELS, blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), pairs);
  }
}

// Level step for rows wider than the LDS query tile (padded width above
// WalkFmt::MAXDP: the whole tile no longer fits in LDS).  Same buckets, XCD
// split, groups and decisions as k_walk_level, but the tile's query rows pass
// through LDS in windows of kWideWindow bytes: the workgroup's waves work in
// rounds of one group each, and within a round every wave multiplies its
// group's 32 child rows window by window, all waves stepping through the
// windows together (one barrier pair per window).  Each window's 64-byte
// steps are loaded eight at a time.  Scores are the same sums over the same
// dimensions (in another order), so the decisions keep their slack.  Windows go
// to LDS by direct loads: 400,000 x 1200 of any sign, 1024 queries, three
// levels 923 us, 1196 through registers; 995 with 1 KB windows copied while
// another is multiplied (the subtree walk's way, whose waves have fewer rows).
constexpr int kWideWindow = 2048;  // bytes of every query row per LDS window

template <int FMT>
__global__ __launch_bounds__(kWalkThreads, 1) void k_walk_wide(WalkLevelArgs a) {
  using F = WalkFmt<FMT>;
  constexpr int TQ = F::TQ;
  constexpr int NQB = TQ / 16;
  constexpr int RS = kWideWindow + 16;  // LDS row stride (bank spread)
  __shared__ __attribute__((aligned(16))) unsigned char qlds[TQ * RS];
  __shared__ uint32_t gpre[kMaxBucketsPerXcd + 1];
  __shared__ uint32_t glo[kMaxBucketsPerXcd], ghi[kMaxBucketsPerXcd];
  __shared__ float thr_lds[TQ];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nwaves = blockDim.x >> 6;
  const int rowbytes = a.dp * F::ESZ;
  const int nwin = (rowbytes + kWideWindow - 1) / kWideWindow;
  const int c16 = lane & 15, g4 = lane >> 4;

  const int xs = a.nbu < kXcds ? a.nbu : kXcds;
  const int x = blockIdx.x % kXcds;
  const int b0 = x * a.nbu / xs, R = (x + 1) * a.nbu / xs - b0;  // this XCD's buckets
  const int W = gridDim.x / kXcds, j = blockIdx.x / kXcds;
  if (x >= xs) return;
  int t0, tstep, m, c;
  if (a.nt <= W) {
    t0 = j % a.nt;
    tstep = a.nt;
    m = j / a.nt;
    c = (W - 1 - t0) / a.nt + 1;
  } else {
    t0 = j;
    tstep = W;
    m = 0;
    c = 1;
  }
  const int bshift = a.level - a.nb;
  unsigned long long pairs = 0;

  for (int t = t0; t < a.nt; t += tstep) {
    const uint64_t tmask = a.tile_mask[t];
    __syncthreads();
    if (wave == 0) {
      uint32_t ng = 0, lo = 0, hi = 0;
      if (lane < R && tmask) {
        const uint32_t n = a.dense ? (1u << bshift)
                                   : min(a.in_count[(size_t)(b0 + lane) * a.nt + t], (uint32_t)a.bcap);
        bucket_share(n, m, c, b0 + lane, kGroupEntries, lo, hi);
        ng = (hi - lo + kGroupEntries - 1) / kGroupEntries;
      }
      uint32_t incl = ng;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane < R) {
        gpre[lane] = incl - ng;
        glo[lane] = lo;
        ghi[lane] = hi;
      }
      if (lane == 63) gpre[R] = incl;
    }
    if (tid < TQ) {
      const int qi = t * TQ + tid;
      float th = a.thr[qi];
      if (FMT == GT_POOL_FP8E4M3) th = ldexpf(th * kFp8ThrFactor, -(a.qexp[qi] + a.lexp));
      thr_lds[tid] = th;
    }
    __syncthreads();
    const uint32_t gtot = gpre[R];
    if (gtot == 0) continue;
    const unsigned char* qsrc = reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)t * TQ * rowbytes;

    for (uint32_t base = 0; base < gtot; base += (uint32_t)nwaves) {
      const uint32_t gg = base + (uint32_t)wave;
      const bool valid = gg < gtot;  // uniform per wave
      // group gg's entries held by this lane (rows c16 and 16 + c16 of the
      // group's 32 child rows), as in k_walk_level; a wave without a group
      // this round takes the last group with empty masks
      const uint32_t ge = valid ? gg : gtot - 1;
      const int r = find_slot(gpre, R, ge);
      const uint32_t e0 = glo[r] + (ge - gpre[r]) * kGroupEntries + (c16 >> 1);
      const uint32_t e1 = e0 + 8;
      const uint32_t ehi = ghi[r];
      const uint32_t bk = (uint32_t)(b0 + r);
      const uint32_t slot = bk * (uint32_t)a.nt + (uint32_t)t;
      const uint32_t ef = e0 - (c16 >> 1);
      const uint32_t i0 = e0 < ehi ? e0 : ef, i1 = e1 < ehi ? e1 : ef;
      const size_t at0 = input_entry(a.dense, slot, a.bcap, i0), at1 = input_entry(a.dense, slot, a.bcap, i1);
      const uint32_t first = bk << bshift;
      const uint32_t p0 = a.dense ? first + i0 : a.in_node[at0];
      const uint32_t p1 = a.dense ? first + i1 : a.in_node[at1];
      const uint64_t pm0 = (valid && e0 < ehi) ? (a.dense ? tmask : a.in_mask[at0]) : 0ull;
      const uint64_t pm1 = (valid && e1 < ehi) ? (a.dense ? tmask : a.in_mask[at1]) : 0ull;
      // rows this lane loads: lanes 4R'..4R'+3 take 64 contiguous bytes of
      // row R' (entry R' / 2, child R' % 2) of each block
      const int src = 2 * (lane >> 3);
      const uint32_t q0 = (uint32_t)__shfl((int)p0, src, 64);
      const uint32_t q1 = (uint32_t)__shfl((int)p1, src, 64);
      const uint32_t ch = (uint32_t)((lane >> 2) & 1);
      const unsigned char* rbase = reinterpret_cast<const unsigned char*>(a.child_rows) + 16 * (lane & 3);
      const unsigned char* arow0 = rbase + (size_t)(2u * q0 + ch) * rowbytes;
      const unsigned char* arow1 = rbase + (size_t)(2u * q1 + ch) * rowbytes;
      const int bp_addr = 4 * (4 * c16 + g4);
      auto to_mfma = [&](const uint4& v) {
        uint4 o;
        o.x = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.x);
        o.y = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.y);
        o.z = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.z);
        o.w = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.w);
        return o;
      };
      f32x4 acc[2][NQB];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[rb][qb][i] = 0.0f;

      for (int wi = 0; wi < nwin; ++wi) {
        const int wofs = wi * kWideWindow;
        const int wbytes = rowbytes - wofs < kWideWindow ? rowbytes - wofs : kWideWindow;
        __syncthreads();  // every wave is done with the previous window
        stage_columns<TQ, kWalkThreads / 64>(qlds, RS, qsrc + wofs, rowbytes, wbytes,
                                             __builtin_amdgcn_readfirstlane(wave), lane);
        wait_loads();
        __syncthreads();
        if (valid) {
          const int wsteps = wbytes / 64;
          const unsigned char* brow = qlds + c16 * RS + 16 * g4;
          for (int s0 = 0; s0 < wsteps; s0 += 8) {
            uint4 l0[8], l1[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              const int st = s0 + u < wsteps ? s0 + u : wsteps - 1;
              l0[u] = ld_global16(arow0 + wofs + 64 * st);
              l1[u] = ld_global16(arow1 + wofs + 64 * st);
            }
            if constexpr (FMT == GT_POOL_FP8E4M3) {
              // steps s and s + 1 in one 16x16x128 product (an even count per window)
#pragma unroll
              for (int u = 0; u < 8; u += 2) {
                if (s0 + u < wsteps) {
                  const uint4 x0a = to_mfma(l0[u]), x1a = to_mfma(l1[u]);
                  const uint4 x0b = to_mfma(l0[u + 1]), x1b = to_mfma(l1[u + 1]);
#pragma unroll
                  for (int qb = 0; qb < NQB; ++qb) {
                    const uint4 bqa = ld_lds16(brow + qb * 16 * RS + 64 * (s0 + u));
                    const uint4 bqb = ld_lds16(brow + qb * 16 * RS + 64 * (s0 + u + 1));
                    mma_f8_16x16x128(x0a, x0b, bqa, bqb, acc[0][qb]);
                    mma_f8_16x16x128(x1a, x1b, bqa, bqb, acc[1][qb]);
                  }
                }
              }
            } else {
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                if (s0 + u < wsteps) {
                  const uint4 x0 = to_mfma(l0[u]), x1 = to_mfma(l1[u]);
#pragma unroll
                  for (int qb = 0; qb < NQB; ++qb) {
                    const uint4 bq = ld_lds16(brow + qb * 16 * RS + 64 * (s0 + u));
                    mma16x16<FMT>(x0, bq, acc[0][qb]);
                    mma16x16<FMT>(x1, bq, acc[1][qb]);
                  }
                }
              }
            }
          }
        }
      }
      if (!valid) continue;
      if (a.bitmap && lane < 16) {
        const uint32_t child0 = 2u * p0 + (uint32_t)(lane & 1), child1 = 2u * p1 + (uint32_t)(lane & 1);
        if (pm0) {
          const uint64_t row = (uint64_t)a.bit_base + child0;
          atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
        }
        if (pm1) {
          const uint64_t row = (uint64_t)a.bit_base + child1;
          atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
        }
      }
      // survival bits as in k_walk_level: lane r < 32 ends with child row r's mask
      const int gsel = 16 * ((lane & 15) >> 2);
      uint64_t mine = 0ull;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint64_t part = 0ull;
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            const uint64_t bal = __ballot(acc[rb][qb][i] >= thr_lds[16 * qb + c16]);
            part |= ((bal >> gsel) & 0xffffull) << (16 * qb);
          }
          if ((lane >> 4) == rb && (lane & 3) == i) mine = part;
        }
      const uint64_t pm_own = lane < 16 ? pm0 : pm1;
      mine = lane < 32 ? (mine & pm_own) : 0ull;
      if (lane < 32) pairs += (unsigned long long)__popcll(pm_own);
      const uint64_t bal = __ballot(mine != 0ull);
      if (bal == 0ull) continue;
      uint32_t obase = 0;
      if (lane == 0) obase = atomicAdd(&a.out_count[slot], (uint32_t)__popcll(bal));
      obase = __shfl(obase, 0, 64);
      if (mine) {
        const uint32_t pos = obase + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        if (pos < a.bcap) {
          const size_t o = (size_t)slot * a.bcap + pos;
          a.out_node[o] = 2u * (lane < 16 ? p0 : p1) + (uint32_t)(lane & 1);
          a.out_mask[o] = mine;
        } else {
          atomicOr(a.over, 1u);
        }
      }
    }
  }
  if (a.stat_pairs) {
    for (int o = 32; o >= 1; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0 && pairs)
      stat_add(a.stat_pairs, GT_MAX_LEVELS, blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), pairs);
  }
}

// Level step with subtraction (bfloat16 pools; paper Sec. 2 and Alg. 1 derive
// the score of one half of a pool from the pool's score and the other half's).
// Every entry carries a score record: upper bounds of its pool's real score
// for all 64 queries of the tile, as bfloat16, query q at 4 (q % 16) + q / 16
// (so that a lane's four values of a pool are eight contiguous bytes).  A
// wave takes 32 entries and reads only their right children (one row each):
// the right child's score s is computed with the matrix cores and tested as
// in k_walk_level; the left child's real score is at most
//   U = diff_upper(sp, score_lower(s, a_b))
// (sp the entry's record, a_b the query's absolute term), and the left child
// is kept for query b iff U >= tau'_b.  Where the right child holds rows at
// or beyond the call's epoch (which later inserts may have grown), U is just
// sp: a part of a pool never scores above the pool.  Every kept child gets a
// complete record (score_upper(s) for the right child, U for the left, each
// rounded up to bfloat16), so the values of queries that are not live are
// bounds too.  Halves the pool rows read per level.
constexpr int kSubGroup = 32;  // entries per wave step
constexpr int kSubPipe = 4;   // 64-byte steps of a lane's two rows fetched ahead
constexpr int kSubThreads = kWalkThreads;  // threads per workgroup

template <int NSTEPS, int PIPE>
__global__ __launch_bounds__(kSubThreads, 1) void k_walk_sub(WalkLevelArgs a) {
  constexpr int FMT = GT_POOL_BF16;
  using F = WalkFmt<FMT>;
  constexpr int TQ = F::TQ;
  constexpr int NQB = TQ / 16;
  static_assert(TQ == 64, "records hold 64 queries");
  static_assert(PIPE == 4, "a row has whole groups of 128 columns, four steps");
  __shared__ __attribute__((aligned(16))) unsigned char qlds[TQ * (F::MAXDP * F::ESZ + 16)];
  __shared__ uint32_t gpre[kMaxBucketsPerXcd + 1];
  __shared__ uint32_t glo[kMaxBucketsPerXcd], ghi[kMaxBucketsPerXcd];
  __shared__ float thr_lds[TQ], sabs_lds[TQ];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nwaves = blockDim.x >> 6;
  const int rowbytes = a.dp * F::ESZ;
  const int rs = rowbytes + 16;
  const int nsteps = NSTEPS > 0 ? NSTEPS : rowbytes / 64;
  const int c16 = lane & 15, g4 = lane >> 4;
  const int e32 = lane & 31;  // the entry this lane fetches (lanes 32-63 repeat 0-31)

  const int xs = a.nbu < kXcds ? a.nbu : kXcds;
  const int x = blockIdx.x % kXcds;
  const int b0 = x * a.nbu / xs, R = (x + 1) * a.nbu / xs - b0;  // this XCD's buckets
  const int W = gridDim.x / kXcds, j = blockIdx.x / kXcds;
  if (x >= xs) return;
  int t0, tstep, m, c;
  if (a.nt <= W) {
    t0 = j % a.nt;
    tstep = a.nt;
    m = j / a.nt;
    c = (W - 1 - t0) / a.nt + 1;
  } else {
    t0 = j;
    tstep = W;
    m = 0;
    c = 1;
  }
  // right child 2p+1 of a level-l pool p covers leaves [(2p+1) 2^s, (2p+2) 2^s)
  const int lshift = a.depth - a.level - 1;
  // subtraction is used where the right child lies wholly below the epoch:
  // then the parent and both children hold only rows the call sees, none of
  // which an insert changes
  auto sub_ok = [&](uint32_t ep) {
    return ((uint64_t)(2u * ep + 2u) << lshift) <= (uint64_t)a.n_epoch;
  };
  // upper bound of the left child's score from the pool's bound sp and the
  // right child's computed score sr (a right score that overflowed gives no
  // lower bound)
  auto left_ub = [&](float sp, float sr, float sa, bool sub) {
    if (!sub || !(sr < INFINITY)) return sp;
    return diff_upper(sp, score_lower(sr, sa));
  };
  const float aup = score_abs_up(a.dp);
  unsigned long long pairs = 0;

  for (int t = t0; t < a.nt; t += tstep) {
    const uint64_t tmask = a.tile_mask[t];
    __syncthreads();
    if (wave == 0) {
      uint32_t ng = 0, lo = 0, hi = 0;
      if (lane < R && tmask) {
        const uint32_t n = min(a.in_count[(size_t)(b0 + lane) * a.nt + t], (uint32_t)a.bcap);
        lo = (uint32_t)(((uint64_t)n * m) / c);
        hi = (uint32_t)(((uint64_t)n * (m + 1)) / c);
        ng = (hi - lo + kSubGroup - 1) / kSubGroup;
      }
      uint32_t incl = ng;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane < R) {
        gpre[lane] = incl - ng;
        glo[lane] = lo;
        ghi[lane] = hi;
      }
      if (lane == 63) gpre[R] = incl;
    }
    __syncthreads();
    const uint32_t gtot = gpre[R];
    if (gtot == 0) continue;
    stage_rows<TQ, kSubThreads / 64>(
        qlds, reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)t * TQ * rowbytes, rowbytes,
        __builtin_amdgcn_readfirstlane(wave), lane);
    if (tid < TQ) {
      thr_lds[tid] = a.thr[t * TQ + tid];
      sabs_lds[tid] = a.sabs[t * TQ + tid];
    }
    wait_loads();
    __syncthreads();

    // entry e32 of group gg: its pool, mask and position (padding lanes take
    // the group's first entry with an empty mask, so every load is valid)
    auto fetch = [&](uint32_t gg, uint32_t& p, uint64_t& pm, uint32_t& pos, uint32_t& slot) {
      const int r = find_slot(gpre, R, gg);
      const uint32_t ef = glo[r] + (gg - gpre[r]) * kSubGroup;
      const uint32_t e = ef + (uint32_t)e32;
      const uint32_t hi = ghi[r];
      slot = (uint32_t)(b0 + r) * (uint32_t)a.nt + (uint32_t)t;
      const uint32_t ie = e < hi ? e : ef;
      pos = (uint32_t)((size_t)slot * a.bcap + ie);
      p = a.in_node[pos];
      const uint64_t lm = a.in_mask[pos];
      pm = e < hi ? lm : 0ull;
    };
    // The right-child rows this lane loads: lanes 4R' .. 4R'+3 take 64
    // contiguous bytes of entry R' (block 0) and entry 16 + R' (block 1).
    auto rows_of = [&](uint32_t p, const unsigned char*& r0, const unsigned char*& r1) {
      const uint32_t q0 = (uint32_t)__shfl((int)p, lane >> 2, 64);
      const uint32_t q1 = (uint32_t)__shfl((int)p, 16 + (lane >> 2), 64);
      const unsigned char* base = reinterpret_cast<const unsigned char*>(a.child_rows) + 16 * (lane & 3);
      r0 = base + (size_t)(2u * q0 + 1u) * rowbytes;
      r1 = base + (size_t)(2u * q1 + 1u) * rowbytes;
    };
    const int bp_addr = 4 * (4 * c16 + g4);
    auto to_mfma = [&](const uint4& v) {
      uint4 r;
      r.x = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.x);
      r.y = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.y);
      r.z = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.z);
      r.w = (uint32_t)__builtin_amdgcn_ds_bpermute(bp_addr, (int)v.w);
      return r;
    };
    const int slast = nsteps - 1;
    uint4 bA0[PIPE], bA1[PIPE], bB0[PIPE], bB1[PIPE];
    uint32_t np = 0, npos = 0, nslot = 0;
    uint64_t npm = 0ull;
    if ((uint32_t)wave < gtot) {
      fetch(wave, np, npm, npos, nslot);
      const unsigned char *r0, *r1;
      rows_of(np, r0, r1);
#pragma unroll
      for (int u = 0; u < PIPE; ++u) {
        const int st = u < slast ? u : slast;
        bA0[u] = ld_global16(r0 + 64 * st);
        bA1[u] = ld_global16(r1 + 64 * st);
      }
    }

    for (uint32_t gg = wave; gg < gtot; gg += nwaves) {
      const uint32_t p = np, pos = npos, slot = nslot;
      const uint64_t pm = npm;
      const unsigned char *arow0, *arow1;
      rows_of(p, arow0, arow1);
      const unsigned char* brow = qlds + c16 * rs + 16 * g4;
      // the pools' score records, read while the rows are multiplied: for
      // entry 16 rb + 4 (l / 16) + i the bounds of queries c, 16 + c, 32 + c,
      // 48 + c (c = l % 16), eight contiguous bytes
      uint2 prec[2][4];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t eps = (uint32_t)__shfl((int)pos, 16 * rb + 4 * g4 + i, 64);
          prec[rb][i] = *reinterpret_cast<const uint2*>(a.in_rec + (size_t)eps * TQ + 4 * c16);
        }
      const bool has_next = gg + nwaves < gtot;
      fetch(has_next ? gg + nwaves : gg, np, npm, npos, nslot);
      if (a.bitmap && lane < 32 && pm) {
        const uint64_t row = (uint64_t)a.bit_base + 2u * p + 1u;
        atomicOr(&a.bitmap[row >> 5], 1u << (row & 31));
      }

      f32x4 acc[2][NQB];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[rb][qb][i] = 0.0f;
      auto step = [&](const uint4& l0, const uint4& l1, int s) {
        const uint4 x0 = to_mfma(l0), x1 = to_mfma(l1);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          const uint4 bq = ld_lds16(brow + qb * 16 * rs + 64 * s);
          mma16x16<FMT>(x0, bq, acc[0][qb]);
          mma16x16<FMT>(x1, bq, acc[1][qb]);
        }
      };
#pragma unroll
      for (int s0 = 0; s0 < nsteps; s0 += 2 * PIPE) {
#pragma unroll
        for (int u = 0; u < PIPE; ++u) {
          const int st = s0 + PIPE + u < slast ? s0 + PIPE + u : slast;
          bB0[u] = ld_global16(arow0 + 64 * st);
          bB1[u] = ld_global16(arow1 + 64 * st);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < PIPE; ++u) step(bA0[u], bA1[u], s0 + u);
        __builtin_amdgcn_sched_barrier(0);
        {
          const bool same = s0 + 2 * PIPE < nsteps;
          const unsigned char *r0 = arow0, *r1 = arow1;
          if (!same) rows_of(np, r0, r1);
          const int sf = same ? s0 + 2 * PIPE : 0;
#pragma unroll
          for (int u = 0; u < PIPE; ++u) {
            const int st = sf + u < slast ? sf + u : slast;
            bA0[u] = ld_global16(r0 + 64 * st);
            bA1[u] = ld_global16(r1 + 64 * st);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s0 + PIPE < nsteps) {
#pragma unroll
          for (int u = 0; u < PIPE; ++u) step(bB0[u], bB1[u], s0 + PIPE + u);
        }
        __builtin_amdgcn_sched_barrier(0);
      }

      // Element (rb, qb, i) of lane l: entry 16 rb + 4 (l / 16) + i of the
      // group, query 16 qb + l % 16.  Decisions are gathered per entry by
      // ballots (lane j < 32 ends with entry j's masks, as in k_walk_level);
      // then every kept child gets its complete record.
      auto rec_of = [&](int rb, int i, int qb) {
        const uint32_t w = qb < 2 ? prec[rb][i].x : prec[rb][i].y;
        return bf16_to_f32((uint16_t)((qb & 1) ? (w >> 16) : (w & 0xFFFFu)));
      };
      const int gsel = 16 * ((lane & 15) >> 2);
      uint64_t mine_r = 0ull, mine_l = 0ull;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int er = 16 * rb + 4 * g4 + i;
          const uint64_t em = __shfl(pm, er, 64);
          const bool sub = sub_ok((uint32_t)__shfl((int)p, er, 64));
          uint64_t part_r = 0ull, part_l = 0ull;
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            const int q = 16 * qb + c16;
            const bool live = (em >> q) & 1ull;
            const float sr = acc[rb][qb][i];
            const float th = thr_lds[q];
            const uint64_t br = __ballot(live && sr >= th);
            const uint64_t bl = __ballot(live && left_ub(rec_of(rb, i, qb), sr, sabs_lds[q], sub) >= th);
            part_r |= ((br >> gsel) & 0xffffull) << (16 * qb);
            part_l |= ((bl >> gsel) & 0xffffull) << (16 * qb);
          }
          if ((lane >> 4) == rb && (lane & 3) == i) {
            mine_r = part_r;
            mine_l = part_l;
          }
        }
      // outputs: lane j < 32 the right child of entry j, lane 32 + j its left
      // (the shuffle runs in every lane: a lane that is switched off gives
      // no data to the others)
      const uint64_t left_m = __shfl(mine_l, e32, 64);
      const uint64_t out_m = lane < 32 ? mine_r : left_m;
      if (lane < 32) pairs += 2ull * (unsigned long long)__popcll(pm);
      const uint64_t bal = __ballot(out_m != 0ull);
      if (bal == 0ull) continue;
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&a.out_count[slot], (uint32_t)__popcll(bal));
      base = __shfl(base, 0, 64);
      const uint32_t opos = base + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      if (out_m) {
        if (opos < a.bcap) {
          const size_t o = (size_t)slot * a.bcap + opos;
          a.out_node[o] = 2u * p + (lane < 32 ? 1u : 0u);
          a.out_mask[o] = out_m;
        } else {
          atomicOr(a.over, 1u);
        }
      }
      if (!a.out_rec) continue;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int er = 16 * rb + 4 * g4 + i;
          const bool sub = sub_ok((uint32_t)__shfl((int)p, er, 64));
          const bool keep_r = ((bal >> er) & 1ull) != 0ull;
          const bool keep_l = ((bal >> (32 + er)) & 1ull) != 0ull;
          const uint32_t or_ = (uint32_t)__shfl((int)opos, er, 64);
          const uint32_t ol_ = (uint32_t)__shfl((int)opos, 32 + er, 64);
          uint32_t vr[NQB], vl[NQB];
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            const int q = 16 * qb + c16;
            const float sr = acc[rb][qb][i];
            vr[qb] = bf16_ceil_hi(score_upper(sr, aup));
            vl[qb] = bf16_ceil_hi(left_ub(rec_of(rb, i, qb), sr, sabs_lds[q], sub));
          }
          if (keep_r && or_ < a.bcap)
            *reinterpret_cast<uint2*>(a.out_rec + ((size_t)slot * a.bcap + or_) * TQ + 4 * c16) =
                make_uint2((vr[0] >> 16) | vr[1], (vr[2] >> 16) | vr[3]);
          if (keep_l && ol_ < a.bcap)
            *reinterpret_cast<uint2*>(a.out_rec + ((size_t)slot * a.bcap + ol_) * TQ + 4 * c16) =
                make_uint2((vl[0] >> 16) | vl[1], (vl[2] >> 16) | vl[3]);
        }
    }
  }
  if (a.stat_pairs) {
    for (int o = 32; o >= 1; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0 && pairs)
      stat_add(a.stat_pairs, GT_MAX_LEVELS, blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), pairs);
  }
}

// Dense level step: every pool of a level against every query, as a matrix
// product with a masked epilogue.  Used where almost every (pool, query tile)
// pair is live (the first tested level): each pool row is read once per
// 256-query column block instead of once per tile.  A workgroup (4 waves, one
// per SIMD) computes 256 pools x 256 queries (4 tiles); wave w owns pools
// 128 (w / 2) .. +127 and tiles 2 (w % 2), 2 (w % 2) + 1: 4 x 4 blocks of
// 32x32 matrix-core tiles whose accumulators fill the wave's accumulation
// registers, so that every 16-byte operand read from LDS feeds four matrix
// products.  K advances 128 bytes per row per stage.  A stage is loaded
// straight from global memory into LDS (no staging registers) one stage
// ahead, into the other of two buffers; within a stage the operands of the
// next K step are read from LDS while the current step's matrix products
// run, and the next stage's first step is read across the stage's barrier.
// Child j of level L survives for query b iff its parent's bit b is set and
// its score reaches tau'_b.  Output: per-(pool, tile) masks for a following
// dense level, or the bucketed sparse frontier for the walk that follows.
//
// LDS layout of a stage: two regions (pool rows, query rows) of 256 rows x
// 128 bytes, each in 32 blocks of 8 rows; row R of a region is row R / 32 of
// block R % 32, and the blocks are 1040 bytes apart.  The 16-byte skew per
// block puts the same chunk of 8 (or 16) consecutive rows on distinct banks,
// so operand reads are conflict-free, and every read of a wave is one base
// register plus an immediate offset.  One direct-to-LDS load instruction
// fills one block (its 64 lanes write 1 KB contiguously).
constexpr int kDM = 256, kDN = 256, kDK = 128;  // pools, queries, K bytes per stage
constexpr int kDBlk = 8 * kDK + 16;             // block pitch
constexpr int kDRegion = 32 * kDBlk;
constexpr int kDStage = 2 * kDRegion;           // 2 x 32.5 KB
constexpr int kDThreads = 256;
constexpr int kDTiles = kDN / 64;  // query tiles per workgroup

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// A thread's 16 direct-to-LDS loads of a stage: instructions j = w + 4 m of
// wave w (j < 32: pool block j, else query block j - 32).  Lane l of an
// instruction writes byte 16 l of its block, i.e. chunk l % 8 of block row
// l / 8, which is region row 32 (l / 8) + block.  Sources are 32-bit offsets
// from the workgroup's first pool row and first query row.  Rows past the
// last pool re-read the last pool; query rows past the last tile re-read the
// last query row (their columns are never tested).
struct DenseLoads {
  const unsigned char* pool;   // first pool row of the workgroup
  const unsigned char* query;  // first query row of the workgroup
  uint32_t off[16];
};
__device__ __forceinline__ void dense_sources(DenseLoads& L, int rowbytes, int64_t row0,
                                              int64_t rows, int q0, int qrows, int wave,
                                              int lane) {
  const int plim = (int)min(rows - row0, (int64_t)kDM), qlim = min(qrows - q0, kDN);
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int j = wave + 4 * m;                 // instruction of the stage
    const int R = 32 * (lane >> 3) + (j & 31);  // region row
    const int lim = j < 32 ? plim : qlim;
    const int rr = R < lim ? R : lim - 1;
    L.off[m] = (uint32_t)rr * (uint32_t)rowbytes + 16u * (uint32_t)(lane & 7);
  }
}
// (instruction m of wave w fills block w + 4 m of the pool region for m < 8,
// block w + 4 m - 32 of the query region after; the destination is the
// wave's offset plus a constant.  The empty asm keeps that offset from being
// treated as loop-invariant: otherwise all 32 destinations are precomputed
// and held in scalar registers through the loop.)
__device__ __forceinline__ void dense_issue(const DenseLoads& L, unsigned char* buf, int s,
                                            uint32_t wave_off) {
  asm volatile("" : "+s"(wave_off));
  const unsigned char* ps = L.pool + s * kDK;
  const unsigned char* qs = L.query + s * kDK;
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const uint32_t c = m < 8 ? 4 * m * kDBlk : kDRegion + (4 * m - 32) * kDBlk;
    __builtin_amdgcn_global_load_lds((const void*)((m < 8 ? ps : qs) + L.off[m]),
                                     (lds_void_ptr)(buf + wave_off + c), 16, 0, 0);
  }
}

// Thresholds of tile t for the two 32-query halves a lane's accumulator
// columns belong to (query t * 64 + 32 j + r).
template <int FMT>
__device__ __forceinline__ void dense_thresholds(const DenseLevelArgs& a, int t, int r, float (&thr)[2]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int qi = t * 64 + 32 * j + r;
    float th = a.thr[qi];
    if (FMT == GT_POOL_FP8E4M3) th = ldexpf(th * kFp8ThrFactor, -(a.qexp[qi] + a.lexp));
    thr[j] = th;
  }
}

// Survival mask of one 32-pool block against tile t: c0 and c1 are the
// 32x32 accumulators of the tile's query halves.  Lane l holds query column
// l % 32 of rows 8 (x / 4) + 4 (l / 32) + x % 4 (register x), so the ballot
// of register x over a query half holds, in its low 32 bits, row
// 8 (x / 4) + x % 4 and, in its high 32 bits, the row 4 below; each half is
// selected into that row's lane.  Lane r < 32 ends with row r's
// 64-query mask (other lanes: 0).
__device__ __forceinline__ uint64_t dense_block_mask(const f32x16& c0, const f32x16& c1,
                                                     const float (&thr)[2], int lane) {
  uint32_t mlo = 0u, mhi = 0u;  // queries 0-31 and 32-63
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const uint64_t b0 = __ballot(c0[x] >= thr[0]);
    const uint64_t b1 = __ballot(c1[x] >= thr[1]);
    const int rr = 8 * (x >> 2) + (x & 3);
    if (lane == rr) {
      mlo = (uint32_t)b0;
      mhi = (uint32_t)b1;
    }
    if (lane == rr + 4) {
      mlo = (uint32_t)(b0 >> 32);
      mhi = (uint32_t)(b1 >> 32);
    }
    // (the empty asm makes each register's ballots be used at once: left to
    // itself the compiler gathers all 32 wave-wide results first, and they
    // overflow the scalar registers)
    asm volatile("" : "+v"(mlo), "+v"(mhi));
  }
  return ((uint64_t)mhi << 32) | mlo;
}

// Score records of the kept pools (subtraction step): upper bounds of each
// pool's real score for all 64 queries of the tile, query q at
// 4 (q % 16) + q / 16 of the pool's 128-byte record.  A block's bounds are
// first written to LDS in record order (32 rows x 128 bytes), then the kept
// rows are copied out with 16-byte accesses.  Lane l holds queries l % 32
// (c0) and 32 + l % 32 (c1) of rows 8 (x / 4) + 4 (l / 32) + x % 4
// (register x): two 16-bit writes per register at fixed offsets from the
// lane's base.
__device__ __forceinline__ void dense_stage_records(unsigned char* blk, float aup,
                                                    const f32x16& c0, const f32x16& c1,
                                                    int lane) {
  const int q = lane & 15, hi16 = (lane >> 4) & 1;
  unsigned char* base = blk + (lane >> 5) * 4 * 128 + 8 * q + 2 * hi16;
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int rr = 8 * (x >> 2) + (x & 3);
    const uint32_t v0 = bf16_ceil_hi(score_upper(c0[x], aup));
    const uint32_t v1 = bf16_ceil_hi(score_upper(c1[x], aup));
    *reinterpret_cast<uint16_t*>(base + rr * 128) = (uint16_t)(v0 >> 16);
    *reinterpret_cast<uint16_t*>(base + rr * 128 + 4) = (uint16_t)(v1 >> 16);
  }
}
// Copies the records of the kept rows of a staged block: oe, lane r < 32, is
// the output entry of row r (-1: not kept).  Lane l moves chunk l % 8 of rows
// l / 8 + 8 k.
__device__ __forceinline__ void dense_copy_records(uint16_t* out_rec, const unsigned char* blk,
                                                   int64_t oe, int lane) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int row = (lane >> 3) + 8 * k;
    const int64_t o = __shfl(oe, row, 64);
    const uint4 v = *reinterpret_cast<const uint4*>(blk + row * 128 + 16 * (lane & 7));
    if (o >= 0) *reinterpret_cast<uint4*>(out_rec + (size_t)o * 64 + 8 * (lane & 7)) = v;
  }
}

// Operands of one K step of a wave: bf16, 16 elements (one 32x32x16
// product per block pair); float8, 64 elements (one 32x32x64 product).
// Lanes 0-31 and 32-63 carry different K ranges, the same in A and B.
template <int FMT>
struct DenseOps {
  static constexpr int NC = FMT == GT_POOL_FP8E4M3 ? 2 : 1;  // 16-byte chunks per lane
  uint4 a[4][NC], b[4][NC];
};
// Lane (r, half) reads, for block i of its pool rows (region row
// 128 wr + 32 i + r: block r, block row 4 wr + i) and K step st, chunks
// NC (2 st + half) + h: base + 128 i + 16 (2 NC st + h), with
// base = 1040 r + 512 wr + 16 NC half (queries alike with wq, in the second
// region).
template <int FMT>
__device__ __forceinline__ void dense_read(const unsigned char* buf, int st, uint32_t abase,
                                           uint32_t bbase, DenseOps<FMT>& o) {
  constexpr int NC = DenseOps<FMT>::NC;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int h = 0; h < NC; ++h)
      o.a[i][h] = *reinterpret_cast<const uint4*>(buf + abase + kDK * i + 16 * (2 * NC * st + h));
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int h = 0; h < NC; ++h)
      o.b[j][h] = *reinterpret_cast<const uint4*>(buf + bbase + kDK * j + 16 * (2 * NC * st + h));
}
template <int FMT, int I0, int I1>
__device__ __forceinline__ void dense_mma(const DenseOps<FMT>& o, f32x16 (&acc)[4][4]) {
#pragma unroll
  for (int i = I0; i < I1; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (FMT == GT_POOL_FP8E4M3)
        mma_f8_32x32x64(o.a[i][0], o.a[i][1], o.b[j][0], o.b[j][1], acc[i][j]);
      else
        mma16<FMT>(o.a[i][0], o.b[j][0], acc[i][j]);
    }
}

template <int FMT>
__global__ __launch_bounds__(kDThreads, 1) void k_dense_level(DenseLevelArgs a) {
  using F = WalkFmt<FMT>;
  static_assert(F::TQ == 64, "dense steps use 64-query tiles");
  // K steps per stage: bf16 steps of 32 bytes, float8 steps of 64 bytes
  constexpr int NS = FMT == GT_POOL_FP8E4M3 ? 2 : 4;
  // (two separate arrays: a read of one is then known not to depend on the
  // loads in flight into the other)
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[kDStage];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[kDStage];
  // output reservations of the workgroup: entries per (tile, bucket) of its
  // 256 pools (at most 8 buckets once a bucket holds 32 pools or more), and
  // the slots' bases
  __shared__ uint32_t wg_cnt[kDTiles][8], wg_base[kDTiles][8];
  const int64_t rows = a.rows;  // pools holding a row below the call's epoch
  const int64_t RB = (rows + kDM - 1) / kDM;
  const int QB = (a.nt + kDTiles - 1) / kDTiles;
  const int64_t total = RB * QB;
  // XCD-aware order: the workgroups of one XCD take consecutive tiles, i.e.
  // all query blocks of a pool block, which then passes through one L2
  const int64_t per_xcd = (total + 7) / 8;
  const int64_t wid = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (wid >= total) return;
  const int qb = (int)(wid % QB);
  const int64_t row0 = (wid / QB) * kDM;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wq = wave & 1;
  const int r = lane & 31, half = lane >> 5;
  const int rowbytes = a.dp * F::ESZ;
  const int nst = rowbytes / kDK;

  const uint32_t wave_off = (uint32_t)(wave * kDBlk);
  DenseLoads L;
  L.pool = reinterpret_cast<const unsigned char*>(a.child_rows) + (size_t)row0 * rowbytes;
  L.query = reinterpret_cast<const unsigned char*>(a.qtile) + (size_t)qb * kDN * rowbytes;
  dense_sources(L, rowbytes, row0, rows, qb * kDN, a.nt * 64, wave, lane);
  constexpr int NC = DenseOps<FMT>::NC;
  const uint32_t abase = (uint32_t)(kDBlk * r + 4 * kDK * wr + 16 * NC * half);
  const uint32_t bbase = (uint32_t)(kDRegion + kDBlk * r + 4 * kDK * wq + 16 * NC * half);

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.0f;

  // Stage s sits in buffer s % 2.  Stage s + 1 is loaded while stage s is
  // multiplied.  At the last K step of stage s a barrier, after this wave's
  // reads of stage s and its loads of stage s + 1 are complete, tells that
  // every wave is done with stage s (its buffer then takes stage s + 2) and
  // that stage s + 1 has landed; the first step of stage s + 1 is read while
  // the last step of stage s is multiplied.  The scheduling barriers keep
  // each step's LDS reads ahead of the matrix work that hides them.
  // (operands alternate between two register sets by the parity of the K
  // step, which is static: a stage has an even number of steps.  The loop
  // runs an even number of stages and holds no data-dependent branch around
  // the reads, so that both sets keep their registers: for an odd number of
  // K stages, position 0 is a stage of zeros and position p holds K stage
  // p - 1.  A step issues its first row of products before the next step's
  // reads: with direct-to-LDS loads in flight the compiler waits for all LDS
  // reads before a step's products, and by then they have had the other
  // twelve products' time.)
  DenseOps<FMT> ops[2];
  const int odd = nst & 1, npos = nst + odd;
  L.pool -= odd * kDK;
  L.query -= odd * kDK;
  // One position from buffer cb; with `next`, its last step crosses the
  // barrier into position p + 1 in buffer nb and, if `issue`, loads position
  // p + 2 into cb.
  auto stage = [&](unsigned char* cb, unsigned char* nb, int p, bool next, bool issue) {
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const DenseOps<FMT>& cu = ops[st & 1];
      DenseOps<FMT>& nx = ops[(st + 1) & 1];
      dense_mma<FMT, 0, 1>(cu, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (st + 1 < NS) {
        dense_read<FMT>(cb, st + 1, abase, bbase, nx);
      } else if (next) {
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
        __syncthreads();
        if (issue) dense_issue(L, cb, p + 2, wave_off);
        dense_read<FMT>(nb, 0, abase, bbase, nx);
      }
      __builtin_amdgcn_sched_barrier(0);
      dense_mma<FMT, 1, 4>(cu, acc);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (tid < kDTiles * 8) (&wg_cnt[0][0])[tid] = 0u;
  if (odd) {
    for (int i = tid; i < kDStage / 16; i += kDThreads)
      *reinterpret_cast<uint4*>(lds0 + 16 * i) = make_uint4(0u, 0u, 0u, 0u);
  } else {
    dense_issue(L, lds0, 0, wave_off);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __syncthreads();
  dense_issue(L, lds1, 1, wave_off);
  dense_read<FMT>(lds0, 0, abase, bbase, ops[0]);
  int p = 0;
  for (; p + 3 < npos; p += 2) {  // positions p + 2 and p + 3 exist
    stage(lds0, lds1, p, true, true);
    stage(lds1, lds0, p + 1, true, true);
  }
  stage(lds0, lds1, p, true, false);
  stage(lds1, lds0, p + 1, false, false);

  // Output: the wave's 8 blocks (tile tt, pool block i).  Child j survives
  // for query b iff its parent's bit b is set and its score reaches tau'_b.
  // All blocks' masks first; the workgroup's frontier reservations are then
  // gathered in LDS and made with one atomic per (bucket, tile) slot (the
  // slot counters share a few cache lines, and one atomic per block and wave
  // queues on them); then the writes: per-(pool, tile) masks for a following
  // dense level, or the bucketed sparse frontier (and, for the subtraction
  // step, the kept pools' score records).
  float thr[2][2];
  uint64_t pm[2][4];  // parent masks (lane r < 32: pool row r of the block)
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const int t = qb * kDTiles + 2 * wq + tt;
    thr[tt][0] = thr[tt][1] = 0.0f;
    if (t < a.nt) dense_thresholds<FMT>(a, t, r, thr[tt]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = row0 + wr * 128 + i * 32 + r;
      pm[tt][i] = 0ull;
      if (t < a.nt && lane < 32 && row < rows)
        pm[tt][i] = a.parent ? a.parent[(row >> 1) * a.nt + t] : a.tile_mask[t];
    }
  }
  const int bshift = a.level - a.nb;  // node -> bucket of the sparse output
  unsigned long long pairs = 0;
  uint64_t mine[2][4];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = row0 + wr * 128 + i * 32 + r;
      mine[tt][i] = dense_block_mask(acc[i][2 * tt], acc[i][2 * tt + 1], thr[tt], lane) & pm[tt][i];
      pairs += (unsigned long long)__popcll(pm[tt][i]);
      if (a.bitmap && pm[tt][i])
        atomicOr(&a.bitmap[(a.bit_base + row) >> 5], 1u << ((a.bit_base + row) & 31));
    }
  if (a.out_dense) {
    // non-empty masks per tile, one atomic per tile and workgroup
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = qb * kDTiles + 2 * wq + tt;
        const int64_t row = row0 + wr * 128 + i * 32 + r;
        if (t < a.nt && lane < 32 && row < rows) a.out_dense[row * a.nt + t] = mine[tt][i];
        const uint64_t eb = __ballot(mine[tt][i] != 0ull);
        if (lane == 0 && eb) atomicAdd(&wg_cnt[2 * wq + tt][0], (uint32_t)__popcll(eb));
      }
    __syncthreads();
    if (tid < kDTiles && qb * kDTiles + tid < a.nt && wg_cnt[tid][0])
      atomicAdd(&a.out_count[qb * kDTiles + tid], wg_cnt[tid][0]);
  } else {
    // one reservation per (bucket, tile) slot of the workgroup when a
    // bucket holds 32 pools or more, else one per row
    const bool grouped = bshift >= 5;
    int64_t oe[2][4];    // output entry of this lane's row (-1: none)
    uint32_t off[2][4];  // the block's first entry within the workgroup's slot
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = qb * kDTiles + 2 * wq + tt;
        const int64_t rb0 = row0 + wr * 128 + i * 32;
        const uint64_t eb = __ballot(mine[tt][i] != 0ull);
        oe[tt][i] = -1;
        off[tt][i] = 0u;
        if (grouped) {
          const int bi = (int)((rb0 >> bshift) - (row0 >> bshift));
          if (lane == 0 && eb) off[tt][i] = atomicAdd(&wg_cnt[2 * wq + tt][bi], (uint32_t)__popcll(eb));
        } else if (mine[tt][i]) {
          off[tt][i] = atomicAdd(&a.out_count[(uint32_t)((rb0 + r) >> bshift) * (uint32_t)a.nt + t], 1u);
        }
      }
    if (grouped) {
      __syncthreads();
      if (tid < kDTiles * 8) {
        const int tw = tid >> 3, bi = tid & 7, t = qb * kDTiles + tw;
        const uint32_t c = wg_cnt[tw][bi];
        if (c && t < a.nt)
          wg_base[tw][bi] =
              atomicAdd(&a.out_count[(uint32_t)((row0 >> bshift) + bi) * (uint32_t)a.nt + t], c);
      }
      __syncthreads();
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = qb * kDTiles + 2 * wq + tt;
        const int64_t rb0 = row0 + wr * 128 + i * 32, row = rb0 + r;
        const uint64_t eb = __ballot(mine[tt][i] != 0ull);
        if (!eb) continue;
        const uint32_t slot = (uint32_t)(row >> bshift) * (uint32_t)a.nt + t;
        uint32_t pos = off[tt][i];
        if (grouped) {
          const int bi = (int)((rb0 >> bshift) - (row0 >> bshift));
          pos = wg_base[2 * wq + tt][bi] + (uint32_t)__builtin_amdgcn_readfirstlane(off[tt][i]) +
                (uint32_t)__popcll(eb & ((1ull << lane) - 1ull));
        }
        if (mine[tt][i]) {
          if (pos < a.bcap) {
            const int64_t o = (int64_t)slot * a.bcap + pos;
            oe[tt][i] = o;
            a.out_node[o] = (uint32_t)row;
            a.out_mask[o] = mine[tt][i];
          } else {
            atomicOr(a.over, 1u);
          }
        }
      }
    if (FMT == GT_POOL_BF16 && a.out_rec) {
      // (the stage buffers are free once every wave is past its last reads;
      // each wave stages its 8 blocks in 32 KB of its own)
      __syncthreads();
      unsigned char* region = (wave < 2 ? lds0 : lds1) + (wave & 1) * 32768;
      const float aup = score_abs_up(a.dp);
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dense_stage_records(region + (tt * 4 + i) * 4096, aup, acc[i][2 * tt],
                              acc[i][2 * tt + 1], lane);
      __syncthreads();
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dense_copy_records(a.out_rec, region + (tt * 4 + i) * 4096, oe[tt][i], lane);
    }
  }
  if (a.stat_pairs) {
    for (int o = 32; o >= 1; o >>= 1) pairs += __shfl_xor(pairs, o, 64);
    if (lane == 0 && pairs)
      stat_add(a.stat_pairs, GT_MAX_LEVELS, blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), pairs);
  }
}

// Exact leaf test: entries (pool p at level depth-1, mask) -> vectors 2p and
// 2p+1 for every query of the mask.  A wave takes two entries at a time and,
// per step, one mask bit of each: 2 entries x 2 vectors = four dot products of
// six rows (an entry has 1.0 to 1.6 live queries here, so two bits per step
// left half of the products unused).  The steps form one pipeline: a slice of
// the next step's rows is requested as soon as the present one's is used up, so
// that row loads are in flight through the reduction and the classification;
// the next entries and their norms are requested two and one pairs ahead.  Row
// addresses are scalar bases with a 32-bit lane offset, which leaves registers
// for three waves per SIMD (four for narrow rows).  Bound by the memory beyond
// L2: 1024 queries on 2^20 x 1000 (0.27 M entries, 12 KB each) 0.39 ms with
// eight products per unpipelined step, now 0.33 + 0.01 for the sort; on
// 2^20 x 512 of any sign (0.66 M entries) 0.49 ms, now 0.34 + 0.01; 4096
// queries (1.3 M entries) 1.88 ms, now 1.35 + 0.04.
struct LeafEntry {
  int t;
  uint32_t p;
  uint64_t m;
  float inv0, inv1;  // inverse norms of vectors 2p and 2p+1 (0: beyond the epoch or zero)
};

// SORTED: slots are the XCD's buckets, entries sorted by pool.
template <bool SORTED>
__device__ __forceinline__ LeafEntry leaf_entry(const LeafArgs& a, const uint32_t* epre, int nsl,
                                                int slot0, uint32_t idx, uint32_t etot,
                                                int& cursor) {
  LeafEntry x;
  x.t = 0;
  x.p = 0;
  x.m = 0ull;
  x.inv0 = x.inv1 = 0.0f;
  if (idx >= etot) return x;
  // a wave's indices only grow: few, large sorted slots are walked by a cursor,
  // the many small ones of the unsorted sweep searched
  if constexpr (SORTED) {
    while ((uint32_t)__builtin_amdgcn_readfirstlane((int)epre[cursor + 1]) <= idx) ++cursor;
  } else {
    cursor = __builtin_amdgcn_readfirstlane(find_slot(epre, nsl, idx));
  }
  const int sl = cursor;
  const uint32_t e = idx - epre[sl];
  const int gs = slot0 + sl;
  if constexpr (SORTED) {
    const size_t o = (size_t)gs * a.nt * a.bcap + e;
    x.t = gs;
    x.p = a.sort_node[o];
    x.m = a.sort_mask[o];
    return x;
  }
  x.t = gs % a.nt;
  if (a.dense) {
    x.p = ((uint32_t)(gs / a.nt) << (a.level - a.nb)) + e;
    x.m = a.tile_mask[x.t];
  } else {
    x.p = a.in_node[(size_t)gs * a.bcap + e];
    x.m = a.in_mask[(size_t)gs * a.bcap + e];
  }
  return x;
}
// Pool and tile of a requested entry (SORTED: t is its bucket and p the sorted
// value until here, which takes no registers while the request is on its way).
template <bool SORTED>
__device__ __forceinline__ uint32_t entry_pool(const LeafArgs& a, const LeafEntry& x) {
  return SORTED ? ((uint32_t)x.t << (a.level - a.nb)) + (x.p >> a.tile_bits) : x.p;
}

// Entries of a bucket sorted by pool (a counting sort in LDS, one workgroup per
// bucket; pools share a bin where a bucket has more than kSortBins).  Unsorted,
// a leaf pair is read again for every tile that kept it, far apart in time:
// 4096 queries on 2^20 x 1000 fetched 13.4 GB for 3.3 GB of distinct rows.
// Sorted, the tiles' entries of a pool are neighbours, mostly of the same wave.
// Bound by the latency of its reads and LDS adds: 8 us for 0.27 M entries of
// 16 tiles, 42 us for 1.3 M of 64.
constexpr int kSortBins = 4096;
__global__ __launch_bounds__(1024) void k_leaf_sort(LeafArgs a, uint32_t* out_node,
                                                    uint64_t* out_mask, uint32_t* out_count) {
  __shared__ uint32_t bin[kSortBins];
  __shared__ uint32_t wsum[16];
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int bits = a.level - a.nb;  // pools per bucket (log2)
  const int shift = bits > 12 ? bits - 12 : 0;
  const uint32_t first = (uint32_t)b << bits;
  static_assert(kSortBins == 1 << 12, "bins of the top 12 bits");
  for (int i = t; i < kSortBins; i += 1024) bin[i] = 0u;
  __syncthreads();
  // 16 waves, one tile's slot at a time
  for (int tl = w; tl < a.nt; tl += 16) {
    const size_t gs = (size_t)b * a.nt + tl;
    const uint32_t n = min(a.in_count[gs], (uint32_t)a.bcap);
    const uint32_t* node = a.in_node + gs * a.bcap;
    for (uint32_t i = lane; i < n; i += 256) {  // four loads in flight
      uint32_t v[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) v[k] = node[i + 64 * k < n ? i + 64 * k : i];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k)
        if (i + 64 * k < n) atomicAdd(&bin[(v[k] - first) >> shift], 1u);
    }
  }
  __syncthreads();
  // exclusive prefix over the bins, four per thread
  uint32_t c[4], sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = sum;
    sum += bin[4 * t + k];
  }
  uint32_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t before = incl - sum;
  for (int k = 0; k < w; ++k) before += wsum[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) bin[4 * t + k] = before + c[k];
  if (t == 1023) out_count[b] = before + sum;
  __syncthreads();
  const size_t base = (size_t)b * a.nt * a.bcap;
  for (int tl = w; tl < a.nt; tl += 16) {
    const size_t gs = (size_t)b * a.nt + tl;
    const uint32_t n = min(a.in_count[gs], (uint32_t)a.bcap);
    const uint32_t* node = a.in_node + gs * a.bcap;
    const uint64_t* mask = a.in_mask + gs * a.bcap;
    for (uint32_t i = lane; i < n; i += 256) {
      uint32_t v[4];
      uint64_t m[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t j = i + 64 * k < n ? i + 64 * k : i;
        v[k] = node[j];
        m[k] = mask[j];
      }
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k)
        if (i + 64 * k < n) {
          const uint32_t rel = v[k] - first;
          const uint32_t pos = atomicAdd(&bin[rel >> shift], 1u);
          out_node[base + pos] = (rel << a.tile_bits) | (uint32_t)tl;
          out_mask[base + pos] = m[k];
        }
    }
  }
}

// Inverse norms of an entry's two vectors, fetched one round before its use
// (the entry itself is fetched two rounds before).
template <bool SORTED>
__device__ __forceinline__ void leaf_norms(const LeafArgs& a, LeafEntry& x) {
  const int64_t i0 = 2 * (int64_t)entry_pool<SORTED>(a, x);
  x.inv0 = i0 < a.n_epoch ? a.invn_f[i0] : 0.0f;
  x.inv1 = i0 + 1 < a.n_epoch ? a.invn_f[i0 + 1] : 0.0f;
}

// The entry's values (the same in every lane) in scalar registers, so that its
// rows are read at scalar bases and take no vector registers for addresses.
template <bool SORTED>
__device__ __forceinline__ LeafEntry leaf_uniform(const LeafArgs& a, const LeafEntry& v) {
  auto u = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
  LeafEntry x;
  x.t = (int)u(SORTED ? v.p & ((1u << a.tile_bits) - 1u) : (uint32_t)v.t);
  x.p = u(entry_pool<SORTED>(a, v));
  x.m = ((uint64_t)u((uint32_t)(v.m >> 32)) << 32) | u((uint32_t)v.m);
  x.inv0 = __uint_as_float(u(__float_as_uint(v.inv0)));
  x.inv1 = __uint_as_float(u(__float_as_uint(v.inv1)));
  return x;
}
struct LeafStep {
  uint32_t q0, q1, p0, p1;
  float i00, i01, i10, i11;  // inverse norms of the entries' vectors (0: not tested)
  float invq;                // of the lane's query
  double rho;
};

// Workgroup -> XCD x = blockIdx % 8, which owns an even contiguous range of
// the buckets that hold rows (slots are bucket-major, so theirs are contiguous
// too); the XCD's
// workgroups sweep its entries in slot order, so the tiles' copies of a leaf
// pair are tested close together in time and share the XCD's L2.
// NV: 16-byte slices per lane and 1024-column chunk that can be non-zero, 4
// in general, 2 for rows of at most 512 columns and 1 for at most 256 (whose
// other slices would only reload the row's last slice; 2^20 x 256, 1024
// queries: 324 us, 379 with two).  Each dot product is summed in the
// same order either way: a slice past dp is zero and adds nothing to
// chunk_sum4.
template <int NV, bool SORTED>
__global__ __launch_bounds__(256) void k_leaf(LeafArgs a) {
  __shared__ uint32_t epre[kMaxSlotsPerXcd + 1];
  __shared__ Hit hstage[4][kHitStage];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xs = a.nbu < kXcds ? a.nbu : kXcds;
  const int x = blockIdx.x % kXcds;
  if (x >= xs) return;
  const int b0 = x * a.nbu / xs;
  const int R = (x + 1) * a.nbu / xs - b0;
  const int nsl = SORTED ? R : R * a.nt;
  const int slot0 = SORTED ? b0 : b0 * a.nt;
  if constexpr (SORTED)
    slot_prefix(epre, nsl, slot0, a.nt, 0, 0, a.tile_mask, a.sort_count, 0xFFFFFFFFu);
  else
    slot_prefix(epre, nsl, slot0, a.nt, a.dense, a.level - a.nb, a.tile_mask, a.in_count,
                (uint32_t)a.bcap);
  const uint32_t etot = (uint32_t)__builtin_amdgcn_readfirstlane((int)epre[nsl]);
  const uint32_t nw = blockDim.x >> 6;
  const uint32_t wgs = gridDim.x / kXcds;
  const uint32_t stride = 2u * wgs * nw;
  Hit* buf = hstage[w];
  int cnt = 0;
  unsigned long long npairs = 0;
  const int vs = lane >> 5, vl = (lane >> 4) & 1;  // value owned after the reduction
  const int nchunks = (a.dp + 1023) / 1024;

  // The wave's entries: en (uniform, in scalar registers) is worked on, nx has
  // its norms requested, nn itself is requested.
  uint32_t idx = 2u * ((blockIdx.x / kXcds) * nw + (uint32_t)w);  // of nx
  int cursor = 0;
  LeafEntry nx0 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx, etot, cursor);
  LeafEntry nx1 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx + 1, etot, cursor);
  leaf_norms<SORTED>(a, nx0);
  leaf_norms<SORTED>(a, nx1);
  LeafEntry nn0 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx + stride, etot, cursor);
  LeafEntry nn1 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx + stride + 1, etot, cursor);
  LeafEntry e0, e1;
  e0.t = e1.t = 0;
  e0.p = e1.p = 0u;
  e0.m = e1.m = 0ull;
  e0.inv0 = e0.inv1 = e1.inv0 = e1.inv1 = 0.0f;

  // A step tests one query against both vectors of each of two entries.
  LeafStep cur, nxt;
  auto start = [&](LeafEntry& e) {
    if (a.bitmap && lane == 0 && e.m) {
      const int64_t i = a.bit_base + 2 * (int64_t)e.p;
      if (e.inv0 != 0.0f) atomicOr(&a.bitmap[i >> 5], 1u << (i & 31));
      if (e.inv1 != 0.0f) atomicOr(&a.bitmap[(i + 1) >> 5], 1u << ((i + 1) & 31));
    }
    // a zero vector has no cosine and is never a member
    if (e.inv0 == 0.0f && e.inv1 == 0.0f) e.m = 0ull;
  };
  // (an entry whose bits are done: valid rows, sums dropped)
  auto take = [&](LeafEntry& e, uint32_t& q, uint32_t& p, float& i0, float& i1) {
    const bool live = e.m != 0ull;
    q = live ? (uint32_t)(e.t * a.tq + (__ffsll((unsigned long long)e.m) - 1)) : 0u;
    p = e.p;
    i0 = live ? e.inv0 : 0.0f;
    i1 = live ? e.inv1 : 0.0f;
    e.m &= e.m - 1ull;
  };
  auto next_step = [&](LeafStep& st) {
    while (!(e0.m | e1.m)) {
      if (idx >= etot) return false;
      e0 = leaf_uniform<SORTED>(a, nx0);
      e1 = leaf_uniform<SORTED>(a, nx1);
      nx0 = nn0;
      nx1 = nn1;
      leaf_norms<SORTED>(a, nx0);
      leaf_norms<SORTED>(a, nx1);
      idx += stride;
      nn0 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx + stride, etot, cursor);
      nn1 = leaf_entry<SORTED>(a, epre, nsl, slot0, idx + stride + 1, etot, cursor);
      start(e0);
      start(e1);
    }
    take(e0, st.q0, st.p0, st.i00, st.i01);
    take(e1, st.q1, st.p1, st.i10, st.i11);
    const uint32_t qg = vs ? st.q1 : st.q0;
    st.invq = a.invn_q[qg];
    st.rho = a.rho[qg];
    return true;
  };
  // Slice v of chunk c of the step's six rows.
  float4 qx[NV][2], fx[NV][2][2];
  auto load_slice = [&](const LeafStep& st, int c, int v) {
    bool ok;
    // (a 32-bit byte offset from a scalar base: no address registers)
    const uint32_t off = 16u * (uint32_t)slice_index(c, v, lane, a.dp, ok);
    auto ld = [&](const float* row) {
      return *reinterpret_cast<const float4*>(reinterpret_cast<const unsigned char*>(row) + off);
    };
    const float* f0 = a.leaves + 2 * (size_t)st.p0 * a.dp;
    const float* f1 = a.leaves + 2 * (size_t)st.p1 * a.dp;
    qx[v][0] = ld(a.qf + (size_t)st.q0 * a.dp);
    fx[v][0][0] = ld(f0);
    fx[v][0][1] = ld(f0 + a.dp);
    qx[v][1] = ld(a.qf + (size_t)st.q1 * a.dp);
    fx[v][1][0] = ld(f1);
    fx[v][1][1] = ld(f1 + a.dp);
  };
  float acc[4];
  int c = 0;
  bool go = next_step(cur);
  if (go) {
#pragma unroll
    for (int v = 0; v < NV; ++v) load_slice(cur, 0, v);
  }
  while (go) {
    // what follows: the next chunk of the same rows, or the next step; its
    // slices are requested as this one's are used up (at the end of the
    // wave's work the last rows again)
    const bool last = c + 1 == nchunks;
    bool more = true;
    int nc = c + 1;
    if (last) {
      more = next_step(nxt);
      nc = more ? 0 : c;
    }
    if (!last || !more) nxt = cur;
    float sv[4][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (v >= NV) {
#pragma unroll
        for (int vi = 0; vi < 4; ++vi) sv[vi][v] = 0.0f;
        continue;
      }
      bool ok;
      (void)slice_index(c, v, lane, a.dp, ok);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int l = 0; l < 2; ++l) {
          // computed for every slice (a redirected slice holds valid data),
          // then selected: no branch per slice
          const float dv = slice_dot4(qx[v][s2], fx[v][s2][l]);
          sv[2 * s2 + l][v] = ok ? dv : 0.0f;
        }
      __builtin_amdgcn_sched_barrier(0);
      load_slice(nxt, nc, v);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int vi = 0; vi < 4; ++vi) {
      const float part = chunk_sum4(sv[vi][0], sv[vi][1], sv[vi][2], sv[vi][3]);
      acc[vi] = c == 0 ? part : __fadd_rn(acc[vi], part);
    }
    if (last) {
      if (cur.i00 == 0.0f) acc[0] = 0.0f;
      if (cur.i01 == 0.0f) acc[1] = 0.0f;
      if (cur.i10 == 0.0f) acc[2] = 0.0f;
      if (cur.i11 == 0.0f) acc[3] = 0.0f;
      const float dot = wave_reduce4(acc, lane);
      // lane 16 v classifies value v = (entry vs, vector vl)
      const float invf = vs ? (vl ? cur.i11 : cur.i10) : (vl ? cur.i01 : cur.i00);
      Hit h;
      uint32_t flag = 0;
      if ((lane & 15) == 0 && invf != 0.0f) {
        const float cs = __fmul_rn(__fmul_rn(dot, cur.invq), invf);
        flag = classify(cs, cur.rho);
        h.q = vs ? cur.q1 : cur.q0;
        h.id = 2u * (vs ? cur.p1 : cur.p0) + (uint32_t)vl;
        h.sim = cs;
        h.flag = flag;
        ++npairs;
      }
      stage_hits(buf, cnt, flag != 0u, h, a.qcount, a.ctr, a.hits, a.hit_cap, a.band_idx, lane);
    }
    cur = nxt;
    c = nc;
    go = more;
  }
  flush_hits(buf, cnt, a.qcount, a.ctr, a.hits, a.hit_cap, a.band_idx, lane, w);
  for (int o = 32; o >= 1; o >>= 1) npairs += __shfl_xor(npairs, o, 64);
  if (lane == 0 && npairs) stat_add(a.stat_pairs, kLeafStride, blockIdx.x * nw + w, npairs);
}

// Candidates within 1e-5 of rho are re-decided with the canonical float64
// cosine, bit-identical to the oracle: the dot product and the query's squared
// norm run sequentially over k, one wave per candidate; the rows' squared norms
// are the canonical ones of ingest.  The time is the chain of one row, so the
// wave forms the products q_k f_k and q_k^2 of 1024 columns first (exact in
// float64, so adding them is the same as a fused multiply-add), into LDS, and
// lane 0 adds up the ones while lane 1 adds up the others (the launch at d =
// 1000 with few candidates: 10 us; with the sums passed from lane to lane 13;
// with operands read and converted in the chain 22).
// Workgroups from kRecheckGroups on sum the frontier entries of one level
// each over its slots' counters (the automatic dense level and a server's
// memory estimates read them); the last one looks for queries that the
// preparation marked as not allowed.
constexpr int kRecheckGroups = 64;
__device__ __forceinline__ void level_entries(const uint32_t* __restrict__ counts, int l,
                                              DevCounters* ctr) {
  __shared__ unsigned long long part[4];
  const int t = threadIdx.x;
  const uint4* c4 = reinterpret_cast<const uint4*>(counts + (size_t)l * kMaxSlots);
  unsigned long long sum = 0;
#pragma unroll
  for (int k = 0; k < kMaxSlots / 4 / 256; ++k) {
    const uint4 v = c4[t + 256 * k];
    sum += (unsigned long long)v.x + v.y + v.z + v.w;
  }
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((t & 63) == 0) part[t >> 6] = sum;
  __syncthreads();
  if (t == 0) ctr->entries[l] = part[0] + part[1] + part[2] + part[3];
}

__global__ __launch_bounds__(256) void k_recheck(Hit* hits, const uint32_t* band_idx,
                                                 const unsigned long long* nband,
                                                 unsigned long long cap,
                                                 const float* __restrict__ qf,
                                                 const float* __restrict__ leaves, int d, int dp,
                                                 const double* __restrict__ ff,
                                                 const double* __restrict__ rho, QCount qcount,
                                                 const uint32_t* lvl_count, int first,
                                                 const int* __restrict__ qexp, int nq,
                                                 DevCounters* ctr) {
  if (blockIdx.x == gridDim.x - 1) {
    bool bad = false;
    for (int i = threadIdx.x; i < nq; i += blockDim.x) bad = bad || qexp[i] == kBadQuery;
    if (bad) atomicOr(&ctr->err, 1u);
    return;
  }
  if (blockIdx.x >= kRecheckGroups) {
    level_entries(lvl_count, first + (int)blockIdx.x - kRecheckGroups, ctr);
    return;
  }
  __shared__ __attribute__((aligned(16))) double prod[4][2][1024];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long n = *nband < cap ? *nband : cap;
  const unsigned long long nw = blockDim.x >> 6;
  const double2* mine = reinterpret_cast<const double2*>(prod[w][lane & 1]);
  for (unsigned long long b = blockIdx.x * nw + w; b < n; b += kRecheckGroups * nw) {
    const uint32_t hi = band_idx[b];
    Hit x = hits[hi];
    const float* q = qf + (size_t)x.q * dp;
    const float* f = leaves + (size_t)x.id * dp;
    double acc = 0.0;
    for (int c = 0; c < d; c += 1024) {
      const int cols = min(1024, dp - c);  // (a multiple of 128; zero past d: acc + 0 = acc)
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 4 * lane + 256 * j;
        if (k < cols) {
          const float4 u = *reinterpret_cast<const float4*>(q + c + k);
          const float4 v = *reinterpret_cast<const float4*>(f + c + k);
          double2* p = reinterpret_cast<double2*>(&prod[w][0][k]);
          double2* r = reinterpret_cast<double2*>(&prod[w][1][k]);
          p[0] = make_double2(__dmul_rn((double)u.x, (double)v.x), __dmul_rn((double)u.y, (double)v.y));
          p[1] = make_double2(__dmul_rn((double)u.z, (double)v.z), __dmul_rn((double)u.w, (double)v.w));
          r[0] = make_double2(__dmul_rn((double)u.x, (double)u.x), __dmul_rn((double)u.y, (double)u.y));
          r[1] = make_double2(__dmul_rn((double)u.z, (double)u.z), __dmul_rn((double)u.w, (double)u.w));
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // 16 columns at a time, the next 16 read while these are added (every
      // lane does it: no branch around the reads)
      double2 v[8], nx[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = mine[j];
      for (int k = 8; k <= cols / 2; k += 8) {
        const int kn = k < cols / 2 ? k : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) nx[j] = mine[kn + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = __dadd_rn(__dadd_rn(acc, v[j].x), v[j].y);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = nx[j];
      }
    }
    const double s = __shfl(acc, 0, 64), sq = __shfl(acc, 1, 64);
    if (lane == 0) {
      const double cs = __ddiv_rn(s, __dmul_rn(__dsqrt_rn(sq), __dsqrt_rn(ff[x.id])));
      atomicAdd(&ctr->rechecked, 1ull);
      if (cs >= rho[x.q]) {
        x.flag = HIT_ACCEPT | accept_slot(qcount, x.q, ctr);
        x.sim = (float)cs;
      } else {
        x.flag = HIT_REJECT;
      }
      hits[hi] = x;
    }
  }
}

// True where every candidate was kept and the results fit the output; the
// placement and the sort are enqueued before the host has seen the counts and
// do nothing otherwise.
__device__ __forceinline__ bool results_fit(const DevCounters* ctr, unsigned long long total,
                                            unsigned long long hit_cap, unsigned long long lim) {
  return ctr->nhits <= hit_cap && total <= lim && ctr->slot_over == 0u && ctr->err == 0u;
}

// Exclusive scan of the per-query counts by a workgroup of 1024: thread t gets
// the offset of its first query (per consecutive queries each); returns the
// total.
__device__ __forceinline__ int64_t scan_counts(QCount qcount, int nq, int per, int64_t& first) {
  __shared__ int64_t wsum[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int lo = min(nq, t * per), hi = min(nq, lo + per);
  int64_t s = 0;
  for (int i = lo; i < hi; ++i) s += qcount.p[(size_t)i << qcount.shift];
  int64_t incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int64_t before = 0, total = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (k < w) before += wsum[k];
    total += wsum[k];
  }
  first = before + incl - s;
  return total;
}

// Offsets and statistics of a call (one workgroup of 1024), and the host's copy
// of the counters: a store to pinned memory instead of a copy of its own.
// Offsets go to the caller's array too unless the call has to be repeated or
// refused.
__device__ __forceinline__ void write_call(const PlaceArgs& a, int per, int64_t first,
                                           int64_t total) {
  const int t = threadIdx.x;
  const DevCounters* c = a.ctr;
  int64_t* out = c->nhits <= a.hit_cap && c->slot_over == 0u && c->err == 0u && c->fr_over == 0u
                     ? a.offs_out : nullptr;
  int64_t run = first;
  for (int i = min(a.nq, t * per); i < min(a.nq, t * per + per); ++i) {
    a.offs[i] = run;
    if (out) out[i] = run;
    run += a.qcount.p[(size_t)i << a.qcount.shift];
  }
  if (t <= GT_MAX_LEVELS) {  // thread l: tests of level l; the last: leaf tests
    const unsigned long long* p =
        t < GT_MAX_LEVELS ? a.stat + t : a.stat + (size_t)kStatStripes * GT_MAX_LEVELS;
    const int stride = t < GT_MAX_LEVELS ? GT_MAX_LEVELS : kLeafStride;
    unsigned long long sum = 0;
#pragma unroll 16
    for (int k = 0; k < kStatStripes; ++k) sum += p[(size_t)k * stride];
    if (t < GT_MAX_LEVELS) a.ctr->pairs[t] = sum; else a.ctr->leaf_pairs = sum;
  }
  if (t == 1023) {
    a.offs[a.nq] = total;
    if (out) out[a.nq] = total;
    a.ctr->total = (unsigned long long)total;
  }
  __syncthreads();
  if (a.host_ctr) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.ctr);
    uint32_t* dst = reinterpret_cast<uint32_t*>(a.host_ctr);
    for (int i = t; i < (int)(sizeof(DevCounters) / 4); i += 1024) dst[i] = src[i];
  }
}

// Accepted pairs to their query's segment: slot = offset of the query + the
// pair's slot among the query's results.  Up to kPlaceQueries queries every
// workgroup scans the counts for itself (the offsets in LDS; the first one
// writes them out), which saves a launch; above, k_scan_offsets ran before.
// Four pairs a thread in flight on every CU: 1.0 M pairs of 4096 queries 41 us,
// 54 with one on half of them.
constexpr int kPlaceQueries = 4096;
__global__ __launch_bounds__(1024) void k_scan_offsets(PlaceArgs a) {
  const int per = (a.nq + 1023) / 1024;
  int64_t first;
  const int64_t total = scan_counts(a.qcount, a.nq, per, first);
  write_call(a, per, first, total);
}

template <bool SCAN>
__global__ __launch_bounds__(1024) void k_place(PlaceArgs a) {
  __shared__ int64_t loffs[SCAN ? kPlaceQueries : 1];
  int64_t total;
  if constexpr (SCAN) {
    const int per = (a.nq + 1023) / 1024, t = threadIdx.x;
    int64_t first;
    total = scan_counts(a.qcount, a.nq, per, first);
    int64_t run = first;
    for (int i = min(a.nq, t * per); i < min(a.nq, t * per + per); ++i) {
      loffs[i] = run;
      run += a.qcount.p[(size_t)i << a.qcount.shift];
    }
    if (blockIdx.x == 0) write_call(a, per, first, total);
    __syncthreads();
  } else {
    total = (int64_t)a.ctr->total;
  }
  if (!results_fit(a.ctr, (unsigned long long)total, a.hit_cap, a.lim)) return;
  const unsigned long long n = a.ctr->nhits;
  const unsigned long long step = gridDim.x * 1024ull;
  for (unsigned long long h = blockIdx.x * 1024ull + threadIdx.x; h < n; h += 4 * step) {
    Hit x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = a.hits[h + k * step < n ? h + k * step : h];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (h + k * step >= n || hit_kind(x[k].flag) != HIT_ACCEPT) continue;
      const int64_t pos = (SCAN ? loffs[x[k].q] : a.offs[x[k].q]) + (int64_t)hit_slot(x[k].flag);
      a.out_id[pos] = x[k].id;
      a.out_sim[pos] = x[k].sim;
    }
  }
}

// Sort each query's results by id (ids of one query are distinct), by their
// bin: the top 12 bits of the id (id >> shift, shift chosen by the host so that
// every id below the call's epoch has a bin below 4096; the top 8 for a few
// results, whose bins cost more than they).  A bin's results are counted, the
// counts scanned, and a result's place is its bin's start plus the number of
// smaller ids in its bin, read in LDS.  Up to 4096 results a workgroup holds
// them in registers; above, it passes over them once per window of about 2048
// places, and up to kSegSplit workgroups share a segment's windows.  Bins
// wider than half a window (more than 2^22 rows) and segments whose passes
// would cost more than a radix sort take stable 4-bit LSD passes by one
// workgroup.  256 threads, 256 bins and radix passes above 4096 before / now
// (us): 64 queries of 5,100 results on average 285 / 35, 512 of them 700 / 100,
// 512 of 2,080 161 / 52, 51 of 2,000 and more 21 / 8, 4096 of 250 18 / 18.
constexpr int kSegThreads = 512, kSegBins = 4096, kSegKeys = 4096, kSegFew = 512;
constexpr int kSegWindow = kSegKeys / 2;  // results of a window: a key and a value each
constexpr int kSegSplit = 16;
constexpr int64_t kSegWindowed = 1 << 18;
__global__ __launch_bounds__(kSegThreads) void k_sort_segments(
    const int64_t* offs, uint32_t* id, float* sim, uint32_t* tmp_id, float* tmp_sim, int64_t* ids_out,
    float* sims_out, const DevCounters* ctr, unsigned long long hit_cap, unsigned long long lim,
    int shift) {
  constexpr int T = kSegThreads, W = T / 64, B = kSegBins / T, kSegPerThread = kSegKeys / T;
  __shared__ uint32_t bin[kSegBins + 1];
  __shared__ uint32_t key[kSegKeys];
  __shared__ uint32_t cur[kSegBins];
  __shared__ uint32_t wsum[W];
  if (!results_fit(ctr, ctr->total, hit_cap, lim)) return;
  const int q = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t lo = offs[q], n = offs[q + 1] - lo;
  const bool radix = n > kSegKeys && (n > kSegWindowed || (2 << shift) > kSegWindow);
  if (n <= 0 || (blockIdx.y > 0 && (n <= kSegKeys || radix))) return;
  if (n <= kSegFew) {
    const int ni = (int)n;
    if (t < 256) bin[t] = 0u;
    uint32_t k[kSegFew / T], g[kSegFew / T], r[kSegFew / T];
    float v[kSegFew / T];
#pragma unroll
    for (int e = 0; e < kSegFew / T; ++e) {
      const int i = t + T * e < ni ? t + T * e : 0;
      k[e] = id[lo + i];
      v[e] = sim[lo + i];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kSegFew / T; ++e)
      if (t + T * e < ni) {
        g[e] = min(k[e] >> (shift + 4), 255u);
        r[e] = atomicAdd(&bin[g[e]], 1u);
      }
    __syncthreads();
    if (w == 0) {  // exclusive prefix of the 256 bins, four per lane
      uint32_t c[4], sum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        c[j] = bin[4 * t + j];
        sum += c[j];
      }
      uint32_t incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(incl, o, 64);
        if (t >= o) incl += x;
      }
      uint32_t run = incl - sum;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bin[4 * t + j] = run;
        run += c[j];
      }
      if (t == 63) bin[256] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kSegFew / T; ++e)
      if (t + T * e < ni) key[bin[g[e]] + r[e]] = k[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kSegFew / T; ++e)
      if (t + T * e < ni) {
        const uint32_t b0 = bin[g[e]], b1 = bin[g[e] + 1];
        uint32_t pos = b0;
        for (uint32_t j = b0; j < b1; ++j) pos += key[j] < k[e];
        ids_out[lo + pos] = (int64_t)k[e];
        sims_out[lo + pos] = v[e];
      }
    return;
  }
  // the bins' counts to their starts, in place
  auto scan_bins = [&]() {
    uint32_t c[B], sum = 0;
#pragma unroll
    for (int j = 0; j < B; ++j) {
      c[j] = bin[t * B + j];
      sum += c[j];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
#pragma unroll
    for (int k = 0; k < W; ++k)
      if (k < w) run += wsum[k];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      bin[t * B + j] = run;
      run += c[j];
    }
    if (t == 0) bin[kSegBins] = (uint32_t)n;
    __syncthreads();
  };
  if (n <= kSegKeys) {
    const int ni = (int)n;
    for (int i = t; i < kSegBins; i += T) bin[i] = 0u;
    uint32_t k[kSegPerThread], g[kSegPerThread], r[kSegPerThread];
    float v[kSegPerThread];
#pragma unroll
    for (int e = 0; e < kSegPerThread; ++e) {
      const int i = t + T * e < ni ? t + T * e : 0;
      if (T * e < ni) {
        k[e] = id[lo + i];
        v[e] = sim[lo + i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kSegPerThread; ++e)
      if (t + T * e < ni) {
        g[e] = min(k[e] >> shift, (uint32_t)kSegBins - 1u);
        r[e] = atomicAdd(&bin[g[e]], 1u);
      }
    __syncthreads();
    scan_bins();
#pragma unroll
    for (int e = 0; e < kSegPerThread; ++e)
      if (t + T * e < ni) key[bin[g[e]] + r[e]] = k[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kSegPerThread; ++e)
      if (t + T * e < ni) {
        const uint32_t b0 = bin[g[e]], b1 = bin[g[e] + 1];
        uint32_t pos = b0;
        for (uint32_t j = b0; j < b1; ++j) pos += key[j] < k[e];
        ids_out[lo + pos] = (int64_t)k[e];
        sims_out[lo + pos] = v[e];
      }
    return;
  }
  if (!radix) {
    const uint32_t* src = id + lo;
    for (int i = t; i < kSegBins; i += T) bin[i] = cur[i] = 0u;
    __syncthreads();
    for (int64_t i0 = 0; i0 < n; i0 += 8 * T) {
      uint32_t k[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t i = i0 + T * e + t;
        k[e] = src[i < n ? i : n - 1];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (i0 + T * e + t < n) atomicAdd(&bin[min(k[e] >> shift, (uint32_t)kSegBins - 1u)], 1u);
    }
    __syncthreads();
    scan_bins();
    // window: the bins that start in [first, first + step); a bin has at most
    // 2^shift ids, so at most kSegWindow results
    const uint32_t step = (uint32_t)(kSegWindow - (1 << shift));
    for (uint32_t first = blockIdx.y * step; first < n; first += gridDim.y * step) {
      // (bins of one window follow each other: it holds places base .. end - 1)
      if (t == 0) wsum[0] = 0xFFFFFFFFu, wsum[1] = 0u;
      __syncthreads();
      for (int i = t; i < kSegBins; i += T) {
        const uint32_t b0 = bin[i], b1 = bin[i + 1];
        if (b0 < b1 && b0 - first < step) {
          atomicMin(&wsum[0], b0);
          atomicMax(&wsum[1], b1);
        }
      }
      __syncthreads();
      const uint32_t base = wsum[0], end = wsum[1];
      for (int64_t i0 = 0; i0 < n; i0 += 8 * T) {
        uint32_t k[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int64_t i = i0 + T * e + t;
          k[e] = src[i < n ? i : n - 1];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int64_t i = i0 + T * e + t;
          const uint32_t g = min(k[e] >> shift, (uint32_t)kSegBins - 1u);
          if (i < n && bin[g] - first < step) {
            const uint32_t at = bin[g] - base + atomicAdd(&cur[g], 1u);
            key[at] = k[e];
            key[kSegWindow + at] = __float_as_uint(sim[lo + i]);
          }
        }
      }
      __syncthreads();
      for (uint32_t i = t; base + i < end; i += T) {
        const uint32_t k = key[i], g = min(k >> shift, (uint32_t)kSegBins - 1u);
        const uint32_t b0 = bin[g], b1 = bin[g + 1];
        uint32_t pos = b0;
        for (uint32_t j = b0; j < b1; ++j) pos += key[j - base] < k;
        ids_out[lo + pos] = (int64_t)k;
        sims_out[lo + pos] = __uint_as_float(key[kSegWindow + i]);
      }
      __syncthreads();
    }
    return;
  }
  // (256 threads: hist of (digit, thread) in key, its sums in cur)
  uint32_t *hist = key, *tot = cur;
  uint32_t *si = id + lo, *di = tmp_id + lo;
  float *sv = sim + lo, *dv = tmp_sim + lo;
  const bool on = t < 256;
  const int64_t chunk = (n + 255) / 256;
  const int64_t a0 = on ? min(n, t * chunk) : 0, a1 = on ? min(n, a0 + chunk) : 0;
  for (int pass = 0; pass < 8; ++pass) {
    const int sh = 4 * pass;
    uint32_t h[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) h[b] = 0;
    for (int64_t i = a0; i < a1; ++i) h[(si[i] >> sh) & 15u]++;
    if (on) {
#pragma unroll
      for (int b = 0; b < 16; ++b) hist[b * 256 + t] = h[b];
    }
    __syncthreads();
    // exclusive scan over hist in (digit, thread) order: thread t owns 16 slots
    if (on) {
      uint32_t s = 0;
      for (int k = 0; k < 16; ++k) s += hist[t * 16 + k];
      tot[t] = s;
    }
    __syncthreads();
    if (t == 0) {
      uint32_t run = 0;
      for (int k = 0; k < 256; ++k) {
        const uint32_t v = tot[k];
        tot[k] = run;
        run += v;
      }
    }
    __syncthreads();
    if (on) {
      uint32_t run = tot[t];
      for (int k = 0; k < 16; ++k) {
        const uint32_t v = hist[t * 16 + k];
        hist[t * 16 + k] = run;
        run += v;
      }
    }
    __syncthreads();
    if (on) {
#pragma unroll
      for (int b = 0; b < 16; ++b) h[b] = hist[b * 256 + t];
    }
    for (int64_t i = a0; i < a1; ++i) {
      const uint32_t k = si[i];
      const uint32_t pos = h[(k >> sh) & 15u]++;
      di[pos] = k;
      dv[pos] = sv[i];
    }
    __syncthreads();
    uint32_t* ti = si; si = di; di = ti;
    float* tv = sv; sv = dv; dv = tv;
  }
  for (int64_t i = t; i < n; i += T) {
    ids_out[lo + i] = (int64_t)si[i];
    sims_out[lo + i] = sv[i];
  }
}

int grid_for(int64_t work, int block) {
  int64_t g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (int)g;
}

}  // namespace

template <int FMT, int NFAST>
hipError_t launch_walk_fmt(const WalkLevelArgs& a, int grid, hipStream_t s) {
  const int nsteps = a.dp * WalkFmt<FMT>::ESZ / 64;
  if (nsteps == NFAST)
    hipLaunchKernelGGL((k_walk_level<FMT, NFAST>), dim3(grid), dim3(kWalkThreads), 0, s, a);
  else
    hipLaunchKernelGGL((k_walk_level<FMT, 0>), dim3(grid), dim3(kWalkThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_walk_level(int fmt, const WalkLevelArgs& a, int grid, hipStream_t s) {
  // whole workgroups per XCD; bucket and slot limits of the kernels
  grid = kXcds * ((grid + kXcds - 1) / kXcds);
  if (a.nb < 0 || a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots ||
      a.level < a.nb || a.nt < 1 || a.nt > kMaxTiles || a.dp < 128 || a.dp % 128 != 0 ||
      a.dp > kMaxWalkWidth || a.nbu < 1 || a.nbu > (1 << a.nb))
    return hipErrorInvalidValue;
  // rows wider than the LDS query tile: windows of the tile through LDS
  if (a.dp > maxdp_walk(fmt)) {
    switch (fmt) {
      case GT_POOL_BF16:
        hipLaunchKernelGGL(k_walk_wide<GT_POOL_BF16>, dim3(grid), dim3(kWalkThreads), 0, s, a);
        break;
      case GT_POOL_FP8E4M3:
        hipLaunchKernelGGL(k_walk_wide<GT_POOL_FP8E4M3>, dim3(grid), dim3(kWalkThreads), 0, s, a);
        break;
      case GT_POOL_F32:
        hipLaunchKernelGGL(k_walk_wide<GT_POOL_F32>, dim3(grid), dim3(kWalkThreads), 0, s, a);
        break;
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // fast paths: padded width 1024
  switch (fmt) {
    case GT_POOL_BF16: return launch_walk_fmt<GT_POOL_BF16, 32>(a, grid, s);
    case GT_POOL_FP8E4M3: return launch_walk_fmt<GT_POOL_FP8E4M3, 16>(a, grid, s);
    case GT_POOL_F32: return launch_walk_fmt<GT_POOL_F32, 64>(a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_walk_sub(const WalkLevelArgs& a, int grid, hipStream_t s) {
  grid = kXcds * ((grid + kXcds - 1) / kXcds);
  if (a.dp > kMaxDpBf16 || a.dp < 128 || a.dp % 128 != 0 ||
      a.nb < 0 || a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots ||
      a.level < a.nb || a.nt < 1 || a.nt > kMaxTiles || a.nbu < 1 || a.nbu > (1 << a.nb) ||
      a.dense || !a.in_rec || !a.sabs ||
      a.level + 1 >= a.depth || a.depth > 32)
    return hipErrorInvalidValue;
  if (a.dp * 2 / 64 == 32)
    hipLaunchKernelGGL((k_walk_sub<32, kSubPipe>), dim3(grid), dim3(kSubThreads), 0, s, a);
  else
    hipLaunchKernelGGL((k_walk_sub<0, kSubPipe>), dim3(grid), dim3(kSubThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_dense_level(int fmt, const DenseLevelArgs& a, hipStream_t s) {
  if (!a.out_dense &&
      (a.nb < 0 || a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots || a.level < a.nb))
    return hipErrorInvalidValue;
  if (a.rows < 1 || a.rows > (int64_t(1) << a.level)) return hipErrorInvalidValue;
  if ((a.dp * (fmt == GT_POOL_FP8E4M3 ? 1 : 2)) % kDK != 0) return hipErrorInvalidValue;
  const int64_t rows = a.rows;
  const int64_t total = ((rows + kDM - 1) / kDM) * ((a.nt + kDTiles - 1) / kDTiles);
  const int64_t grid = 8 * ((total + 7) / 8);
  switch (fmt) {
    case GT_POOL_BF16:
      hipLaunchKernelGGL(k_dense_level<GT_POOL_BF16>, dim3((unsigned)grid), dim3(kDThreads), 0, s, a);
      break;
    case GT_POOL_FP8E4M3:
      hipLaunchKernelGGL(k_dense_level<GT_POOL_FP8E4M3>, dim3((unsigned)grid), dim3(kDThreads), 0, s, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_leaf(const LeafArgs& a, int n_cu, hipStream_t s) {
  if (a.nb < 0 || a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots ||
      a.level < a.nb || a.nt < 1 || a.nt > kMaxTiles || a.nbu < 1 || a.nbu > (1 << a.nb) || n_cu < 1)
    return hipErrorInvalidValue;
  // As many workgroups of four waves per CU as its registers hold at once:
  // three, or four for rows of at most 512 columns (two slices per lane) and
  // five for at most 256; with fewer the loads in flight do not cover their
  // latency (two, three and four: 0.41 ms against 0.38, 0.44 against 0.41, 0.35
  // against 0.32), with one more the rows spill or wait (six: 0.40).
  // The grid is a multiple of the XCD count: every XCD's workgroups split its
  // entries by blockIdx / 8.
  const bool sorted = a.tile_bits >= 0, narrow = a.dp <= 512;
  const dim3 g(kXcds * ((n_cu * (a.dp <= 256 ? 5 : narrow ? 4 : 3) + kXcds - 1) / kXcds));
  if (a.dp <= 256 && sorted)
    hipLaunchKernelGGL((k_leaf<1, true>), g, dim3(256), 0, s, a);
  else if (a.dp <= 256)
    hipLaunchKernelGGL((k_leaf<1, false>), g, dim3(256), 0, s, a);
  else if (narrow && sorted)
    hipLaunchKernelGGL((k_leaf<2, true>), g, dim3(256), 0, s, a);
  else if (narrow)
    hipLaunchKernelGGL((k_leaf<2, false>), g, dim3(256), 0, s, a);
  else if (sorted)
    hipLaunchKernelGGL((k_leaf<4, true>), g, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_leaf<4, false>), g, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_leaf_sort(const LeafArgs& a, hipStream_t s) {
  if (a.nb < 0 || a.nb > kMaxBucketBits || ((int64_t)a.nt << a.nb) > kMaxSlots ||
      a.level < a.nb || a.nt < 1 || a.nbu < 1 || a.nbu > (1 << a.nb) || a.dense ||
      (1 << a.tile_bits) < a.nt || a.level - a.nb + a.tile_bits > 32 || !a.sort_node ||
      !a.sort_mask || !a.sort_count || a.sort_node == a.in_node || a.sort_mask == a.in_mask)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_leaf_sort, dim3(a.nbu), dim3(1024), 0, s, a,
                     const_cast<uint32_t*>(a.sort_node), const_cast<uint64_t*>(a.sort_mask),
                     const_cast<uint32_t*>(a.sort_count));
  return hipGetLastError();
}

hipError_t launch_recheck(Hit* hits, const uint32_t* band_idx, const unsigned long long* nband,
                          unsigned long long cap, const float* qf, const float* leaves, int d,
                          int dp, const double* ff, const double* rho, QCount qcount,
                          const uint32_t* lvl_count, int first, int levels, const int* qexp, int nq,
                          DevCounters* ctr, hipStream_t s) {
  if (first < 0 || levels > GT_MAX_LEVELS) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_recheck, dim3(kRecheckGroups + (levels > first ? levels - first : 0) + 1),
                     dim3(256), 0, s, hits, band_idx, nband, cap, qf, leaves, d, dp, ff, rho,
                     qcount, lvl_count, first, qexp, nq, ctr);
  return hipGetLastError();
}

hipError_t launch_place(const PlaceArgs& a, hipStream_t s) {
  if (a.nq <= kPlaceQueries) {
    hipLaunchKernelGGL(k_place<true>, dim3(256), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_scan_offsets, dim3(1), dim3(1024), 0, s, a);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(k_place<false>, dim3(256), dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_sort_segments(const int64_t* offs, int nq, uint32_t* id, float* sim,
                                uint32_t* tmp_id, float* tmp_sim, int64_t* ids_out,
                                float* sims_out, const DevCounters* ctr,
                                unsigned long long hit_cap, unsigned long long lim,
                                int64_t id_bound, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  // top 12 bits of the ids below id_bound
  int bits = 0;
  while (bits < 32 && (int64_t(1) << bits) < id_bound) ++bits;
  const int shift = bits > 12 ? bits - 12 : 0;
  const int split = std::max(1, std::min(kSegSplit, 256 / nq));
  hipLaunchKernelGGL(k_sort_segments, dim3(nq, split), dim3(kSegThreads), 0, s, offs, id, sim,
                     tmp_id, tmp_sim, ids_out, sims_out, ctr, hit_cap, lim, shift);
  return hipGetLastError();
}

}  // namespace gt
