// Exhaustive baseline (the paper's Exh comparison, Sec. 4): every (query,
// vector) dot product with a matrix-core GEMM [nq x d] . [d x n], and a
// threshold epilogue that keeps pairs which may reach rho.  Kept pairs go
// through the same exact test as the leaves of the walk, so both paths return
// identical results.
//
// The products run on the float16 matrix cores (16 times the float32 rate)
// with every float32 operand split in two: x 2^e = hi + lo, hi the nearest
// float16 and lo the nearest float16 of the rest (22 significant bits), and
// q.f = hi.hi + hi.lo + lo.hi, accumulated in float32.  e is a power-of-two
// scale per row that puts the largest element near the top of the float16
// range.  Per product the split and the dropped lo.lo lose at most 3 x 2^-22 of
// |q_k f_k|, and the 3 K / 16 accumulations at most one unit in the last place
// each, well inside the (K + 2) 2^-22 by which the thresholds are lowered.  An
// element far below its row's largest also loses up to half of the least float16
// (2^-38 of |f|, 2^-39 of the query's largest element), which no relative slack
// covers where the score itself is that small: sqrt(K) (2^-38 + 2^-39) |q| |f| in
// all, within half of the slack's share of scores from 1.5 2^-15 sqrt(K) / (K - 6)
// <= 4.3e-6 of |q| |f| on.  Calls with a smaller positive threshold (kSplitRho)
// take float32 matrix cores.  (On an index of signed vectors the slack is
// absolute, and thresholds of at most 0 keep every pair.)  Measured
// against float64 the scores are closer than the float32 matrix cores' (which
// round after every two products): rms error 2.3e-8 against 3.3e-8 on softmax
// rows of d = 1000, 6.0e-8 against 9.0e-7 on centred ones, largest error 5e-7
// against 7e-7 and 1.5e-6 against 2.3e-5, and smaller at each of five widths from
// 128 to 4096 of five distributions.
#include <math.h>

#include "gt_internal.h"
#include "gt_device.h"
#include "gt_numerics.h"

namespace gt {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

constexpr int kET = 256;            // output tile edge (queries x vectors)
constexpr int kEK = 32;             // dimensions per stage: 128 bytes of split row
constexpr int kEBlk = 8 * 128 + 16; // LDS: 32 blocks of 8 rows, skewed by 16 bytes
constexpr int kERegion = 32 * kEBlk;
constexpr int kEStage = 2 * kERegion;
constexpr int kEThreads = 256;

typedef __attribute__((address_space(3))) void* lds_ptr;

// Eight scaled values as hi and lo halves.
__device__ __forceinline__ void split8(const float (&x)[8], f16x8& hi, f16x8& lo) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    hi[k] = (_Float16)x[k];
    lo[k] = (_Float16)(x[k] - (float)hi[k]);
  }
}

// Split rows: 32 dimensions are 128 bytes, for each 8 of them 16 bytes of hi and
// 16 of lo.  One workgroup per query row (rows past nq: zero, never kept).
__global__ __launch_bounds__(256) void k_split_queries(const float* __restrict__ qf, int nq, int dp,
                                                       const float* __restrict__ thr,
                                                       unsigned char* __restrict__ out,
                                                       float* __restrict__ thr_out) {
  __shared__ float mx[4];
  const int b = blockIdx.x, t = threadIdx.x;
  const float* q = qf + (size_t)b * dp;
  float m = 0.0f;
  if (b < nq)
    for (int k = t; k < dp; k += 256) m = fmaxf(m, fabsf(q[k]));
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((t & 63) == 0) mx[t >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
  int e = 0;
  if (m > 0.0f && m < INFINITY) (void)frexpf(m, &e);  // m < 2^e
  e = 15 - e;
  for (int c = t; c < dp / 8; c += 256) {
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = b < nq ? ldexpf(q[8 * c + k], e) : 0.0f;
    f16x8 hi, lo;
    split8(x, hi, lo);
    f16x8* o = reinterpret_cast<f16x8*>(out + (size_t)b * dp * 4 + (size_t)c * 32);
    o[0] = hi;
    o[1] = lo;
  }
  if (t == 0) thr_out[b] = b < nq ? ldexpf(thr[b], e) : INFINITY;
}

// Room for each lane's candidates: a workgroup of four waves reserves with one add.
// False if none has any.
__device__ __forceinline__ bool reserve(uint32_t count, int lane, int wave, DevCounters* ctr,
                                        unsigned long long& pos) {
  __shared__ uint32_t wcount[4];
  __shared__ unsigned long long wbase;
  uint32_t incl = count;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t c = __shfl_up(incl, o, 64);
    if (lane >= o) incl += c;
  }
  if (lane == 63) wcount[wave] = incl;
  __syncthreads();
  const uint32_t all = wcount[0] + wcount[1] + wcount[2] + wcount[3];
  if (all == 0u) return false;
  if (threadIdx.x == 0) wbase = atomicAdd(&ctr->ncand, (unsigned long long)all);
  __syncthreads();
  pos = wbase + incl - count;
  for (int k = 0; k < wave; ++k) pos += wcount[k];
  return true;
}

// Operands of one 16-dimension step of a wave.
struct SplitOps {
  f16x8 ah[4], al[4], bh[4], bl[4];
};

// A workgroup (4 waves, one per SIMD) computes 256 queries x 256 vectors; wave
// w owns queries 128 (w / 2) .. +127 and vectors 128 (w % 2) .. +127, 4 x 4
// blocks of 32x32 products whose accumulators fill its accumulation registers,
// so that the 16 operand reads of a step feed 48 products.  Per stage of 32
// dimensions the split query rows are loaded straight into LDS; the float32
// vector rows pass through registers, are split there between the products of
// the stage's first step, and are written to the next stage's buffer.  Bound
// by the matrix cores.  XCD-aware order: the workgroups of one XCD take all
// query blocks of a vector block in turn, which then passes through one L2.
// 1024 queries x 2^20 vectors, d = 1000: 5.7 ms (1.16 PFLOP/s of float16
// products, the rate of a large library GEMM on this card), on float32 matrix
// cores 16.4 ms (134 TFLOP/s, 0.85 of their peak).
__global__ __launch_bounds__(kEThreads, 1) void k_gemm_threshold(
    const unsigned char* __restrict__ qs, int qblocks, const float* __restrict__ rows, int64_t n,
    int dp, const float* __restrict__ thr, const float* __restrict__ nf, uint2* cand,
    unsigned long long cap, DevCounters* ctr) {
  // (two separate arrays: reads of one do not wait for the loads into the other)
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[kEStage];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[kEStage];
  __shared__ float thr_lds[kET];
  const int64_t rblocks = (n + kET - 1) / kET;
  const int64_t total = rblocks * qblocks;
  const int64_t per_xcd = (total + 7) / 8;
  const int64_t wid = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (wid >= total) return;
  const int qb = (int)(wid % qblocks);
  const int64_t r0 = (wid / qblocks) * kET;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wave >> 1, wr = wave & 1;
  const int r = lane & 31, half = lane >> 5;
  const int nst = dp / kEK;
  thr_lds[tid] = thr[qb * kET + tid];

  // Query loads: instruction m of wave w fills block j = w + 4 m of the query
  // region; lane l brings chunk l % 8 of block row l / 8, region row
  // 32 (l / 8) + j.
  const unsigned char* qbase = qs + (size_t)qb * kET * dp * 4;
  uint32_t qoff[8];
#pragma unroll
  for (int m = 0; m < 8; ++m)
    qoff[m] = (uint32_t)(32 * (lane >> 3) + wave + 4 * m) * (uint32_t)(dp * 4) + 16u * (uint32_t)(lane & 7);
  const uint32_t wave_off = (uint32_t)(wave * kEBlk);
  auto issue_queries = [&](unsigned char* buf, int s) {
    uint32_t wo = wave_off;
    asm volatile("" : "+s"(wo));  // (keeps the destinations from being held in scalar registers)
    const unsigned char* p = qbase + (size_t)s * 128;
#pragma unroll
    for (int m = 0; m < 8; ++m)
      __builtin_amdgcn_global_load_lds((const void*)(p + qoff[m]),
                                       (lds_ptr)(buf + wo + 4 * m * kEBlk), 16, 0, 0);
  };
  // Vector rows: piece m of wave w is 16 rows x 32 dimensions, lane l the 8
  // dimensions 8 (l % 4) of region row R = 64 m + 16 w + l / 4 (rows past the
  // last one re-read it; they are never kept).
  const float* vrow[4];
  uint32_t vdst[4];
  int vexp[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int R = 64 * m + 16 * wave + (lane >> 2);
    const int64_t row = r0 + R < n ? r0 + R : n - 1;
    vrow[m] = rows + (size_t)row * dp + 8 * (lane & 3);
    vdst[m] = (uint32_t)(kERegion + (R & 31) * kEBlk + (R >> 5) * 128 + 32 * (lane & 3));
    int e = 0;
    const float norm = nf[row];
    if (norm > 0.0f) (void)frexpf(norm, &e);  // elements <= |f| <= 2^e
    vexp[m] = 14 - e;
  }
  float4 v[4][2];
  auto load_rows = [&](int s) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      v[m][0] = *reinterpret_cast<const float4*>(vrow[m] + s * kEK);
      v[m][1] = *reinterpret_cast<const float4*>(vrow[m] + s * kEK + 4);
    }
  };
  auto put_rows = [&](unsigned char* buf, int m) {
    const float x[8] = {ldexpf(v[m][0].x, vexp[m]), ldexpf(v[m][0].y, vexp[m]),
                        ldexpf(v[m][0].z, vexp[m]), ldexpf(v[m][0].w, vexp[m]),
                        ldexpf(v[m][1].x, vexp[m]), ldexpf(v[m][1].y, vexp[m]),
                        ldexpf(v[m][1].z, vexp[m]), ldexpf(v[m][1].w, vexp[m])};
    f16x8 hi, lo;
    split8(x, hi, lo);
    *reinterpret_cast<f16x8*>(buf + vdst[m]) = hi;
    *reinterpret_cast<f16x8*>(buf + vdst[m] + 16) = lo;
  };
  // Lane (r, half) reads, for block i of its rows (region row 128 w + 32 i + r:
  // LDS block r, block row 4 w + i), dimensions 16 st + 8 half .. +7.
  const uint32_t abase = (uint32_t)(kEBlk * r + 512 * wq + 32 * half);
  const uint32_t bbase = (uint32_t)(kERegion + kEBlk * r + 512 * wr + 32 * half);
  auto read_ops = [&](const unsigned char* buf, int st, SplitOps& o) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o.ah[i] = *reinterpret_cast<const f16x8*>(buf + abase + 128 * i + 64 * st);
      o.al[i] = *reinterpret_cast<const f16x8*>(buf + abase + 128 * i + 64 * st + 16);
      o.bh[i] = *reinterpret_cast<const f16x8*>(buf + bbase + 128 * i + 64 * st);
      o.bl[i] = *reinterpret_cast<const f16x8*>(buf + bbase + 128 * i + 64 * st + 16);
    }
  };

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.0f;
  // the products of query row block i (small terms first)
  auto products = [&](const SplitOps& o, int i) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.ah[i], o.bl[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.al[i], o.bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.ah[i], o.bh[j], acc[i][j], 0, 0, 0);
  };

  // Stage s is multiplied from buffer cb.  First step: its products, with the
  // rows of stage s + 1 (in registers) split and written to nb between them and
  // the rows of stage s + 2 requested; the second step's operands are read
  // meanwhile.  Then a barrier: stage s + 1 is complete in nb and every wave is
  // done with cb, which takes the queries of stage s + 2; the first operands of
  // stage s + 1 are read while the second step is multiplied.
  SplitOps o0, o1;
  auto stage = [&](unsigned char* cb, unsigned char* nb, int s, bool next, bool next2) {
    products(o0, 0);
    __builtin_amdgcn_sched_barrier(0);
    read_ops(cb, 1, o1);
    if (next) put_rows(nb, 0);
    __builtin_amdgcn_sched_barrier(0);
    products(o0, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (next) put_rows(nb, 1);
    __builtin_amdgcn_sched_barrier(0);
    products(o0, 2);
    __builtin_amdgcn_sched_barrier(0);
    if (next) {
      put_rows(nb, 2);
      put_rows(nb, 3);
    }
    if (next2) load_rows(s + 2);
    __builtin_amdgcn_sched_barrier(0);
    products(o0, 3);
    __builtin_amdgcn_sched_barrier(0);
    if (next) {
      // the queries of stage s + 1 have landed (the rows requested above may
      // still be in flight), and this wave's LDS accesses are complete
      if (next2)
        __builtin_amdgcn_s_waitcnt(0x0078);  // vmcnt(8) lgkmcnt(0)
      else
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (next2) issue_queries(cb, s + 2);
      read_ops(nb, 0, o0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) products(o1, i);
    __builtin_amdgcn_sched_barrier(0);
  };
  issue_queries(lds0, 0);
  load_rows(0);
#pragma unroll
  for (int m = 0; m < 4; ++m) put_rows(lds0, m);
  issue_queries(lds1, 1);
  load_rows(1);
  __builtin_amdgcn_s_waitcnt(0x0070);  // stage 0, and the requests of stage 1
  __syncthreads();
  read_ops(lds0, 0, o0);
  int s = 0;
  for (; s + 2 < nst; s += 2) {
    stage(lds0, lds1, s, true, true);
    stage(lds1, lds0, s + 1, true, true);
  }
  stage(lds0, lds1, s, true, false);
  stage(lds1, lds0, s + 1, false, false);

  // Epilogue: keep (query, vector) if the score may reach rho * |q| * |f|, both
  // sides in the rows' scales.  Register x of block (i, j): query
  // 32 i + 8 (x / 4) + 4 half + x % 4, vector 32 j + r.  Counted first, so that
  // a workgroup reserves its candidates with one add.
  float nfv[4];
  uint32_t rid[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t row = r0 + 128 * wr + 32 * j + r;
    rid[j] = (uint32_t)row;
    float norm = row < n ? nf[row] : 0.0f;
    int e = 0;
    if (norm > 0.0f) (void)frexpf(norm, &e);
    nfv[j] = ldexpf(norm, 14 - e) * (1.0f - 0x1p-20f);
  }
  uint32_t kept[4][2];  // bit 16 (j % 2) + x of word (i, j / 2)
  uint32_t count = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    kept[i][0] = kept[i][1] = 0u;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const float th = thr_lds[128 * wq + 32 * i + 8 * (x >> 2) + 4 * half + (x & 3)];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (nfv[j] > 0.0f && acc[i][j][x] >= th * nfv[j]) kept[i][j >> 1] |= 1u << (16 * (j & 1) + x);
    }
    count += (uint32_t)(__popc(kept[i][0]) + __popc(kept[i][1]));
  }
  unsigned long long pos;
  if (!reserve(count, lane, wave, ctr, pos)) return;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int w = 0; w < 2; ++w)
      for (uint32_t m = kept[i][w]; m; m &= m - 1u) {
        const int bit = __ffs((int)m) - 1, x = bit & 15;
        const int qi = qb * kET + 128 * wq + 32 * i + 8 * (x >> 2) + 4 * half + (x & 3);
        if (pos < cap) cand[pos] = make_uint2((uint32_t)qi, rid[2 * w] + 32u * (uint32_t)(bit >> 4));
        ++pos;
      }
}

constexpr int kFT = 128;    // output tile edge (queries x vectors)
constexpr int kFK = 32;     // dimensions per LDS stage
constexpr int kFStride = kFK + 4;

// The same on float32 matrix cores, for positive thresholds below kSplitRho: no scale
// takes small elements out of the operands' range, so the relative slack holds
// for any score.  1024 queries x 2^20 vectors, d = 1000: 16.4 ms.
//
// One workgroup (4 waves) per 128 x 128 output tile; each wave owns 64 x 64 as
// 2 x 2 blocks of 32 x 32.  Workgroups are dispatched round-robin over the 8
// XCDs; consecutive workgroups of one XCD take the query tiles of one vector
// tile in turn, so each vector tile is fetched into that XCD's L2 once.
__global__ __launch_bounds__(256) void k_gemm_small_rho(const float* __restrict__ qf, int nq_pad,
                                                        const float* __restrict__ rows, int64_t n,
                                                        int dp, const float* __restrict__ thr,
                                                        const float* __restrict__ nf, uint2* cand,
                                                        unsigned long long cap, DevCounters* ctr,
                                                        int nq) {
  __shared__ __attribute__((aligned(16))) float As[kFT * kFStride];
  __shared__ __attribute__((aligned(16))) float Bs[kFT * kFStride];
  const int QT = nq_pad / kFT;
  const int64_t RT = (n + kFT - 1) / kFT;
  const int64_t total = RT * QT;
  const int64_t per_xcd = (total + 7) / 8;
  const int64_t w = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (w >= total) return;
  const int qt = (int)(w % QT);
  const int64_t rt = w / QT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = (wave >> 1) * 64, wr = (wave & 1) * 64;  // wave's sub-tile origin
  const int c = lane & 31, half = lane >> 5;

  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

  // global -> register staging: 128 rows x 32 floats per operand; thread tid
  // moves float4 pieces tid + 256 v (v < 4): row = piece / 8 = tid / 8 + 32 v
  const float* qbase = qf + (size_t)qt * kFT * dp;
  const int64_t r0 = rt * kFT;
  const int prow = tid >> 3, pcol = (tid & 7) * 4;
  const float* qa = qbase + (size_t)prow * dp + pcol;
  const float* fb[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t rr = r0 + prow + 32 * v < n ? r0 + prow + 32 * v : n - 1;
    fb[v] = rows + (size_t)rr * dp + pcol;
  }
  const size_t q32 = (size_t)32 * dp;
  float4 ra0 = *reinterpret_cast<const float4*>(qa);
  float4 ra1 = *reinterpret_cast<const float4*>(qa + q32);
  float4 ra2 = *reinterpret_cast<const float4*>(qa + 2 * q32);
  float4 ra3 = *reinterpret_cast<const float4*>(qa + 3 * q32);
  float4 rb0 = *reinterpret_cast<const float4*>(fb[0]);
  float4 rb1 = *reinterpret_cast<const float4*>(fb[1]);
  float4 rb2 = *reinterpret_cast<const float4*>(fb[2]);
  float4 rb3 = *reinterpret_cast<const float4*>(fb[3]);
  for (int k0 = 0; k0 < dp; k0 += kFK) {
    __syncthreads();
    *reinterpret_cast<float4*>(&As[(prow + 0) * kFStride + pcol]) = ra0;
    *reinterpret_cast<float4*>(&As[(prow + 32) * kFStride + pcol]) = ra1;
    *reinterpret_cast<float4*>(&As[(prow + 64) * kFStride + pcol]) = ra2;
    *reinterpret_cast<float4*>(&As[(prow + 96) * kFStride + pcol]) = ra3;
    *reinterpret_cast<float4*>(&Bs[(prow + 0) * kFStride + pcol]) = rb0;
    *reinterpret_cast<float4*>(&Bs[(prow + 32) * kFStride + pcol]) = rb1;
    *reinterpret_cast<float4*>(&Bs[(prow + 64) * kFStride + pcol]) = rb2;
    *reinterpret_cast<float4*>(&Bs[(prow + 96) * kFStride + pcol]) = rb3;
    __syncthreads();
    if (k0 + kFK < dp) {
      const int kn = k0 + kFK;
      ra0 = *reinterpret_cast<const float4*>(qa + kn);
      ra1 = *reinterpret_cast<const float4*>(qa + q32 + kn);
      ra2 = *reinterpret_cast<const float4*>(qa + 2 * q32 + kn);
      ra3 = *reinterpret_cast<const float4*>(qa + 3 * q32 + kn);
      rb0 = *reinterpret_cast<const float4*>(fb[0] + kn);
      rb1 = *reinterpret_cast<const float4*>(fb[1] + kn);
      rb2 = *reinterpret_cast<const float4*>(fb[2] + kn);
      rb3 = *reinterpret_cast<const float4*>(fb[3] + kn);
    }
#pragma unroll
    for (int t = 0; t < kFK / 8; ++t) {
      float4 fa[2], fb[2];
#pragma unroll
      for (int a = 0; a < 2; ++a)
        fa[a] = *reinterpret_cast<const float4*>(&As[(wq + 32 * a + c) * kFStride + 8 * t + 4 * half]);
#pragma unroll
      for (int b = 0; b < 2; ++b)
        fb[b] = *reinterpret_cast<const float4*>(&Bs[(wr + 32 * b + c) * kFStride + 8 * t + 4 * half]);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a].x, fb[b].x, acc[a][b], 0, 0, 0);
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a].y, fb[b].y, acc[a][b], 0, 0, 0);
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a].z, fb[b].z, acc[a][b], 0, 0, 0);
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a].w, fb[b].w, acc[a][b], 0, 0, 0);
        }
    }
  }

  // Epilogue as above: keep (query, vector) if the score may reach rho * |q| * |f|,
  // counted first (with one add per wave and accumulator register, the add's one
  // address set the time of a call with many candidates: 9.6 M of them 88 ms, now
  // 16.6).
  float nfv[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int64_t row = r0 + wr + 32 * b + c;
    nfv[b] = row < n ? nf[row] : 0.0f;
  }
  uint32_t kept[2], count = 0;  // bit 16 b + i of word a
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    kept[a] = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int qi = qt * kFT + wq + 32 * a + 8 * (i >> 2) + 4 * half + (i & 3);
      const float th = qi < nq ? thr[qi] : INFINITY;
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (nfv[b] > 0.0f && acc[a][b][i] >= th * nfv[b] * (1.0f - 0x1p-20f)) kept[a] |= 1u << (16 * b + i);
    }
    count += (uint32_t)__popc(kept[a]);
  }
  unsigned long long pos;
  if (!reserve(count, lane, wave, ctr, pos)) return;
#pragma unroll
  for (int a = 0; a < 2; ++a)
    for (uint32_t m = kept[a]; m; m &= m - 1u) {
      const int bit = __ffs((int)m) - 1, i = bit & 15;
      const int qi = qt * kFT + wq + 32 * a + 8 * (i >> 2) + 4 * half + (i & 3);
      if (pos < cap) cand[pos] = make_uint2((uint32_t)qi, (uint32_t)(r0 + wr + 32 * (bit >> 4) + c));
      ++pos;
    }
}

// Exact test of explicit (query, vector) pairs: the same float32 dot product
// (in-lane pairwise sums, then the lane reduction) and classification as the
// leaf test of the walk, four pairs per wave at a time.
__global__ __launch_bounds__(256) void k_pair_check(const uint2* cand, const unsigned long long* ncand,
                                                    unsigned long long cap, const float* qf,
                                                    const float* leaves, const float* invn_q,
                                                    const float* invn_f, const double* rho, int dp,
                                                    Hit* hits, unsigned long long hit_cap,
                                                    uint32_t* band_idx, QCount qcount,
                                                    DevCounters* ctr,
                                                    unsigned long long* stat_pairs) {
  __shared__ Hit hstage[4][kHitStage];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned long long n = *ncand < cap ? *ncand : cap;
  const unsigned long long nw = blockDim.x >> 6;
  Hit* buf = hstage[w];
  int cnt = 0;
  unsigned long long npairs = 0;
  // Lane 16 v .. 16 v + 15 hold pair v of the step; a step's pairs are requested
  // a step ahead.
  const int v = lane >> 4;
  const unsigned long long step = gridDim.x * nw * 4ull;
  unsigned long long b0 = (blockIdx.x * nw + w) * 4ull;
  auto pair_at = [&](unsigned long long b) { return cand[b + v < n ? b + v : n - 1]; };
  uint2 nx = make_uint2(0u, 0u);
  if (b0 < n) nx = pair_at(b0);
  for (; b0 < n; b0 += step) {
    const uint2 x = nx;
    if (b0 + step < n) nx = pair_at(b0 + step);
    const float invf = invn_f[x.y], invq = invn_q[x.x];
    const double rh = rho[x.x];
    const float *q[4], *f[4];  // (at scalar bases)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      q[k] = qf + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)x.x, 16 * k) * dp;
      f[k] = leaves + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)x.y, 16 * k) * dp;
    }
    float acc[4];
    for (int c = 0; c * 1024 < dp; ++c) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float part = lane_partial16(q[k], f[k], c, dp, lane);
        acc[k] = c == 0 ? part : __fadd_rn(acc[k], part);
      }
    }
    const float dot = wave_reduce4(acc, lane);
    Hit h;
    uint32_t flag = 0;
    if ((lane & 15) == 0 && b0 + v < n) {
      const float cs = __fmul_rn(__fmul_rn(dot, invq), invf);
      flag = invf != 0.0f ? classify(cs, rh) : 0u;
      h.q = x.x;
      h.id = x.y;
      h.sim = cs;
      h.flag = flag;
      ++npairs;
    }
    stage_hits(buf, cnt, flag != 0u, h, qcount, ctr, hits, hit_cap, band_idx, lane);
  }
  flush_hits(buf, cnt, qcount, ctr, hits, hit_cap, band_idx, lane, w);
  for (int o = 32; o >= 1; o >>= 1) npairs += __shfl_xor(npairs, o, 64);
  if (lane == 0 && npairs)
    stat_add(stat_pairs, kLeafStride, (uint32_t)(blockIdx.x * nw + w), npairs);
}

}  // namespace

hipError_t launch_exhaustive_gemm(const float* qf, int nq_pad, const float* leaves, int64_t n,
                                  int dp, const float* thr_gemm, const float* nf,
                                  unsigned char* qsplit, float* qsplit_thr, uint2* cand,
                                  unsigned long long cand_cap, DevCounters* ctr, int nq,
                                  bool small_rho, hipStream_t s) {
  if (n <= 0 || nq_pad <= 0) return hipSuccess;
  if (dp % 128 != 0 || nq > nq_pad || nq_pad % kFT != 0) return hipErrorInvalidValue;
  if (small_rho) {
    const int64_t tiles = ((n + kFT - 1) / kFT) * (nq_pad / kFT);
    hipLaunchKernelGGL(k_gemm_small_rho, dim3((unsigned)(8 * ((tiles + 7) / 8))), dim3(256), 0, s, qf,
                       nq_pad, leaves, n, dp, thr_gemm, nf, cand, cand_cap, ctr, nq);
    return hipGetLastError();
  }
  const int qblocks = (nq_pad + kET - 1) / kET;
  hipLaunchKernelGGL(k_split_queries, dim3(qblocks * kET), dim3(256), 0, s, qf, nq, dp, thr_gemm,
                     qsplit, qsplit_thr);
  if (hipError_t e = hipGetLastError()) return e;
  const int64_t total = ((n + kET - 1) / kET) * qblocks;
  const int64_t grid = 8 * ((total + 7) / 8);
  hipLaunchKernelGGL(k_gemm_threshold, dim3((unsigned)grid), dim3(kEThreads), 0, s, qsplit, qblocks,
                     leaves, n, dp, qsplit_thr, nf, cand, cand_cap, ctr);
  return hipGetLastError();
}

hipError_t launch_pair_check(const uint2* cand, const unsigned long long* ncand,
                             unsigned long long cap, const float* qf, const float* leaves,
                             const float* invn_q, const float* invn_f, const double* rho, int dp,
                             Hit* hits, unsigned long long hit_cap, uint32_t* band_idx,
                             QCount qcount, DevCounters* ctr,
                             unsigned long long* stat_pairs, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_pair_check, dim3(grid), dim3(256), 0, s, cand, ncand, cap, qf, leaves, invn_q,
                     invn_f, rho, dp, hits, hit_cap, band_idx, qcount, ctr, stat_pairs);
  return hipGetLastError();
}

}  // namespace gt
