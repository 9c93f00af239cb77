// Device helpers shared by the leaf test of the walk and the pair test of the
// exhaustive path: classification against rho and staging of candidate hits.
#pragma once
#include "gt_internal.h"

namespace gt {

// Statistics counters.  Every wave of a walk, dense or leaf launch adds its
// count once.  Adds to one address are served one after another, so the waves
// spread over kStatStripes counters on lines of their own and the offsets
// kernel sums them.  With one counter, one reservation per wave and one
// returning add per accepted pair, a leaf launch was bound by those adds:
// 5,001 entries (256 queries, n = 2^17, d = 2048) took 64 us, now 26; 10,208
// entries (16 queries, d = 512) 94 us, now 39; 0.59 M entries (1024 queries,
// d = 1000) 0.45 ms, now 0.41.
__device__ __forceinline__ void stat_add(unsigned long long* stat, int stride, uint32_t wave,
                                         unsigned long long v) {
  atomicAdd(stat + (size_t)(wave % kStatStripes) * stride, v);
}

// Slots of a wave's accepted pairs among their queries' results, shifted into
// the flag.  Lanes of the same query share one add to its counter for the
// first four queries met (calls of few queries, whose counters would
// otherwise take every result as an add of its own); other lanes add alone.
__device__ __forceinline__ uint32_t accept_slots(bool acc, uint32_t q, QCount qcount,
                                                 DevCounters* ctr, int lane) {
  uint64_t rem = __ballot(acc);
  if (rem == 0ull) return 0u;
  int leader = lane;
  uint32_t rank = 0, add = 1;
#pragma unroll 1
  for (int k = 0; k < 4 && rem; ++k) {
    const int l0 = __ffsll((unsigned long long)rem) - 1;
    const uint32_t q0 = (uint32_t)__shfl((int)q, l0, 64);
    const uint64_t same = __ballot(acc && q == q0);
    if (acc && q == q0) {
      leader = l0;
      rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
      add = (uint32_t)__popcll(same);
    }
    rem &= ~same;
  }
  uint32_t r = 0;
  if (acc && leader == lane) r = atomicAdd(&qcount.p[(size_t)q << qcount.shift], add);
  r = (uint32_t)__shfl((int)r, leader, 64) + rank;
  if (acc && r >= kMaxResultsPerQuery) {
    atomicOr(&ctr->slot_over, 1u);
    r = 0u;
  }
  return r << 2;
}

// Writes the cnt staged hits of a wave to hits[base ..]; an accepted pair
// takes its slot here, for 64 pairs at a time, so that the test rounds do not
// wait for the counters.
__device__ __forceinline__ void write_hits(const Hit* buf, int cnt, unsigned long long base,
                                           QCount qcount, DevCounters* ctr, Hit* hits,
                                           unsigned long long hit_cap, uint32_t* band_idx,
                                           int lane) {
  for (int i0 = 0; i0 < cnt; i0 += 64) {
    const int i = i0 + lane;
    const bool have = i < cnt;
    Hit x = buf[have ? i : i0];
    const bool acc = have && hit_kind(x.flag) == HIT_ACCEPT;
    x.flag |= accept_slots(acc, x.q, qcount, ctr, lane);
    const unsigned long long slot = base + i;
    if (have && slot < hit_cap) {
      hits[slot] = x;
      if (hit_kind(x.flag) == HIT_BAND) {
        const unsigned long long bp = atomicAdd(&ctr->nband, 1ull);
        if (bp < hit_cap) band_idx[bp] = (uint32_t)slot;
      }
    }
  }
}

// Appends up to 64 candidate hits of a wave to its LDS staging buffer and
// flushes the buffer to global memory (one reservation per flush) when it is
// nearly full.  Called by the whole wave.
__device__ __forceinline__ void stage_hits(Hit* buf, int& cnt, bool have, const Hit& h,
                                           QCount qcount, DevCounters* ctr, Hit* hits,
                                           unsigned long long hit_cap, uint32_t* band_idx,
                                           int lane) {
  const uint64_t bal = __ballot(have);
  if (have) buf[cnt + __popcll(bal & ((1ull << lane) - 1ull))] = h;
  cnt += __popcll(bal);
  if (cnt <= kHitStage - 64) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  unsigned long long base = 0;
  if (lane == 0) base = atomicAdd(&ctr->nhits, (unsigned long long)cnt);
  base = __shfl(base, 0, 64);
  write_hits(buf, cnt, base, qcount, ctr, hits, hit_cap, band_idx, lane);
  __builtin_amdgcn_wave_barrier();
  cnt = 0;
}

// Last flush of a workgroup of four waves: one reservation for all of them
// (every wave of the workgroup calls it once, with whatever it has staged).
__device__ __forceinline__ void flush_hits(const Hit* buf, int cnt, QCount qcount,
                                           DevCounters* ctr, Hit* hits,
                                           unsigned long long hit_cap, uint32_t* band_idx,
                                           int lane, int w) {
  __shared__ int counts[4];
  __shared__ unsigned long long first;
  if (lane == 0) counts[w] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int all = counts[0] + counts[1] + counts[2] + counts[3];
    first = all ? atomicAdd(&ctr->nhits, (unsigned long long)all) : 0ull;
  }
  __syncthreads();
  unsigned long long base = first;
  for (int k = 0; k < w; ++k) base += (unsigned long long)counts[k];
  write_hits(buf, cnt, base, qcount, ctr, hits, hit_cap, band_idx, lane);
}

// Slot of one accepted pair among its query's results (the recheck's).
__device__ __forceinline__ uint32_t accept_slot(QCount qcount, uint32_t q, DevCounters* ctr) {
  const uint32_t r = atomicAdd(&qcount.p[(size_t)q << qcount.shift], 1u);
  if (r >= kMaxResultsPerQuery) {
    atomicOr(&ctr->slot_over, 1u);
    return 0u;
  }
  return r << 2;
}

// Classification of a float32 cosine against rho (the float32 value is within
// 1e-6 of the canonical float64 one): accept, reject, or recheck in float64.
__device__ __forceinline__ uint32_t classify(float cs, double rho) {
  const double c64 = (double)cs;
  if (c64 >= rho + 1e-5) return HIT_ACCEPT;
  if (c64 > rho - 1e-5) return HIT_BAND;
  return 0u;
}

}  // namespace gt
