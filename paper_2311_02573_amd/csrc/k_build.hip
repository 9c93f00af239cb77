// Index construction and query preparation kernels.
//
// Tree layout (paper Sec. 2: the pools of binary splitting are fixed offline):
// level l (0 = root) has 2^l pools; pool j of level l covers leaves
// [j * 2^(depth-l), (j+1) * 2^(depth-l)).  Level l is stored at rows
// (2^l - 1) .. (2^(l+1) - 2) of one array, so the two children of a pool are
// adjacent rows.  Leaves (level `depth`) are the float32 feature rows.
#include <float.h>
#include <hip/hip_fp16.h>
#include <math.h>

#include <algorithm>

#include "gt_internal.h"
#include "gt_numerics.h"

namespace gt {

namespace {

__global__ void k_zero_u32(uint32_t* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

__device__ __forceinline__ float load_feature(const void* src, int dtype, int64_t idx) {
  if (dtype == GT_F16) return __half2float(reinterpret_cast<const __half*>(src)[idx]);
  if (dtype == GT_BF16)
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(src)[idx] << 16);
  return reinterpret_cast<const float*>(src)[idx];
}

// Four consecutive features of a row (VEC: one aligned load; else one by one,
// zero past the row's d columns).
template <bool VEC>
__device__ __forceinline__ float4 load_feature4(const void* src, int dtype, int64_t row, int d,
                                                int c) {
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (VEC) {
    if (c < d) {
      const int64_t i = row * d + c;
      if (dtype == GT_F32) return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(src) + i);
      const uint2 h = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(src) + i);
      const uint16_t u[4] = {(uint16_t)h.x, (uint16_t)(h.x >> 16), (uint16_t)h.y, (uint16_t)(h.y >> 16)};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = dtype == GT_F16 ? __half2float(__ushort_as_half(u[e]))
                               : __uint_as_float((uint32_t)u[e] << 16);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < d) v[e] = load_feature(src, dtype, row * d + c + e);
  }
  return make_float4(v[0], v[1], v[2], v[3]);
}

__global__ void k_ingest_reset(IngestOut* o) {
  const int t = threadIdx.x;
  if (t < GT_MAX_LEVELS) o->over[t] = 0u;
  if (t == 0) {
    o->mmin = INFINITY;
    o->absmax = 0u;
    o->err = 0u;
  }
}

// Feature rows to float32 leaves, with their canonical squared norm (float64,
// summed sequentially over the columns), inverse norm and lowered norm.
// Values must be finite and >= 0, or only finite with allow_negative (then
// the largest |value| is folded into o->absmax as float bits).
//
// Bound by memory (rows in, leaves out) as long as the sequential sums, one
// lane per row, hide behind it: a workgroup of four waves moves tiles of R
// rows x 4096 / R columns through registers into one of two LDS buffers while
// its first R lanes add up the tile before.  64-row tiles for large inputs
// (200,000 x 1000 float32: 1.66 ms with single-wave workgroups and 4-byte
// loads, now 0.44); 4-row tiles for small ones, whose time is the chain of one
// row (100 x 512: 346 us, now 11).
template <int R, bool VEC>
__global__ __launch_bounds__(256) void k_ingest(const void* src, int dtype, int64_t rows, int d,
                                                int dp, float* leaves, double* ff, float* invn,
                                                float* nf, IngestOut* o, int allow_negative) {
  constexpr int C = 4096 / R, G = C / 4, S = C + 4;  // S: row stride in LDS (16-byte bank spread)
  __shared__ __attribute__((aligned(16))) float tile[2][R * S];
  __shared__ float amax_w[4];
  const int t = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * R;
  bool bad = false;
  float amax = 0.0f;
  const int ntiles = (dp + C - 1) / C;
  float4 v[4];
  auto load = [&](int k) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int i = t + 256 * p, c = k * C + 4 * (i % G);
      const int64_t row = r0 + i / G;
      v[p] = row < rows && c < dp ? load_feature4<VEC>(src, dtype, row, d, c)
                                  : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  };
  auto store = [&](int k) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int i = t + 256 * p, r = i / G, c4 = 4 * (i % G), c = k * C + c4;
      const float x[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (allow_negative) {
          if (!isfinite(x[e])) bad = true;
          amax = fmaxf(amax, fabsf(x[e]));
        } else if (!(x[e] >= 0.0f) || isinf(x[e])) {
          bad = true;
        }
      }
      if (r0 + r < rows && c < dp) *reinterpret_cast<float4*>(leaves + (r0 + r) * dp + c) = v[p];
      *reinterpret_cast<float4*>(&tile[k & 1][r * S + c4]) = v[p];
    }
  };
  load(0);
  store(0);
  __syncthreads();
  double acc = 0.0;
  for (int k = 0; k < ntiles; ++k) {
    if (k + 1 < ntiles) load(k + 1);
    if (t < R) {
      const float* x = &tile[k & 1][t * S];
      const int lim = min(C, d - k * C);
      int c = 0;
      for (; c + 16 <= lim; c += 16) {
        float4 y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = *reinterpret_cast<const float4*>(x + c + 4 * j);
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // (squares of float32 values are exact in float64)
          acc = __fma_rn((double)y[j].x, (double)y[j].x, acc);
          acc = __fma_rn((double)y[j].y, (double)y[j].y, acc);
          acc = __fma_rn((double)y[j].z, (double)y[j].z, acc);
          acc = __fma_rn((double)y[j].w, (double)y[j].w, acc);
        }
      }
      for (; c < lim; ++c) acc = __fma_rn((double)x[c], (double)x[c], acc);
    }
    if (k + 1 < ntiles) store(k + 1);
    __syncthreads();
  }
  if (bad) atomicOr(&o->err, 1u);
  if (allow_negative) {
    for (int s = 32; s >= 1; s >>= 1) amax = fmaxf(amax, __shfl_xor(amax, s, 64));
    if ((t & 63) == 0) amax_w[t >> 6] = amax;
    __syncthreads();
    if (t == 0) {
      const uint32_t m = __float_as_uint(fmaxf(fmaxf(amax_w[0], amax_w[1]), fmaxf(amax_w[2], amax_w[3])));
      if (m > o->absmax) atomicMax(&o->absmax, m);  // (a stale read only adds an atomic)
    }
  }
  if (t < 64) {
    double mn = INFINITY;
    const int64_t row = r0 + t;
    if (t < R && row < rows) {
      ff[row] = acc;
      const double nrm = __dsqrt_rn(acc);
      invn[row] = acc > 0.0 ? (float)__ddiv_rn(1.0, nrm) : 0.0f;
      nf[row] = acc > 0.0 ? f64_to_f32_down(nrm) : 0.0f;
      if (acc > 0.0) mn = nrm;
    }
    for (int s = R / 2; s >= 1; s >>= 1) mn = fmin(mn, __shfl_xor(mn, s, 64));
    if (t == 0 && mn < o->mmin)
      atomicMin(reinterpret_cast<unsigned long long*>(&o->mmin),
                (unsigned long long)__double_as_longlong(mn));
  }
}

// A refused ingest (invalid values, or beyond a signed index's bound) leaves
// the pools as they are: the kernels enqueued behind it do nothing.
__device__ __forceinline__ bool refused(const IngestOut* o, float bound) {
  return o && (o->err != 0u || (bound > 0.0f && __uint_as_float(o->absmax) > bound));
}

// One pool of two children: the element-wise sum rounded up (sum pooling,
// paper Sec. 2) or the element-wise maximum, which is exact (Our-Max pooling).
template <bool MAXP>
__device__ __forceinline__ float4 pool4(const float4& a, const float4& b) {
  if constexpr (MAXP)
    return make_float4(fmaxf(a.x, b.x), fmaxf(a.y, b.y), fmaxf(a.z, b.z), fmaxf(a.w, b.w));
  else
    return make_float4(add_up(a.x, b.x), add_up(a.y, b.y), add_up(a.z, b.z), add_up(a.w, b.w));
}

// Four columns of pool j of level l in every stored format.
__device__ __forceinline__ void store_pool4(const TreeArgs& a, int l, int64_t j, int c,
                                            const float4& v) {
  const size_t at = (size_t)(((int64_t(1) << l) - 1 + j)) * a.w + c;
  *reinterpret_cast<float4*>(a.tree + at) = v;
  if (a.p16) {
    const uint32_t lo = (uint32_t)bf16_up(v.x) | ((uint32_t)bf16_up(v.y) << 16);
    const uint32_t hi = (uint32_t)bf16_up(v.z) | ((uint32_t)bf16_up(v.w) << 16);
    *reinterpret_cast<uint2*>(a.p16 + at) = make_uint2(lo, hi);
  }
  if (a.p8) {
    const int e = a.lexp[l];
    uint32_t q[4] = {e4m3_up_f32(v.x, e), e4m3_up_f32(v.y, e), e4m3_up_f32(v.z, e), e4m3_up_f32(v.w, e)};
    bool over = false;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (q[k] == 0xFFu) {
        over = true;
        q[k] = 0x7Eu;
      }
    *reinterpret_cast<uint32_t*>(a.p8 + at) = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
    if (over) atomicOr(&a.over[l], 1u);
  }
}

// Folds four values into their level's maximum (few threads; a stale read only
// adds an atomic).
__device__ __forceinline__ void raise_level_max(const TreeArgs& a, int l, const float4& v) {
  const float m = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
  if (m > a.level_max[l])
    atomicMax(reinterpret_cast<unsigned int*>(a.level_max + l), __float_as_uint(m));
}

// Pools of K levels above level `child`: each thread reads four columns of the
// 2^K rows below one pool of level child - K and writes every pool of that
// subtree that covers one of the rows [lo, hi), in every stored format, so a
// level is read once for K levels and never again for its reduced copies.
// Bound by memory.  200,000 x 1000, sum pools with a bfloat16 copy: one launch
// per level and a conversion pass took 0.86 ms, now 0.43.
// With `level_max`, the largest value of each written level as float bits (one
// atomic per workgroup, and only where it raises the value): a launch per
// level with one atomic per wave took 6.0 ms.
template <bool MAXP, int K>
__global__ __launch_bounds__(256) void k_tree(TreeArgs a, int child) {
  if (refused(a.gate, a.bound)) return;
  __shared__ float mx[K][4];
  const int top = child - K, g = a.w / 4;
  const int sh = a.depth - top;
  const int64_t first = a.lo >> sh, count = ((a.hi - 1) >> sh) - first + 1;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  float m[K];
#pragma unroll
  for (int k = 0; k < K; ++k) m[k] = 0.0f;
  if (i < count * g) {
    const int64_t j = first + i / g;
    const int c = (int)(i % g) * 4;
    const float* rows = child == a.depth ? a.leaves : a.tree + (size_t)((int64_t(1) << child) - 1) * a.w;
    const float* p = rows + (size_t)(j << K) * a.w + c;
    float4 v[1 << K];
#pragma unroll
    for (int r = 0; r < (1 << K); ++r) v[r] = *reinterpret_cast<const float4*>(p + (size_t)r * a.w);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int l = child - 1 - k;
      const int64_t lo = a.lo >> (a.depth - l), hi = (a.hi - 1) >> (a.depth - l);
#pragma unroll
      for (int r = 0; r < (1 << (K - 1 - k)); ++r) {
        v[r] = pool4<MAXP>(v[2 * r], v[2 * r + 1]);
        const int64_t node = (j << (K - 1 - k)) + r;
        if (node >= lo && node <= hi) {
          store_pool4(a, l, node, c, v[r]);
          m[k] = fmaxf(m[k], fmaxf(fmaxf(v[r].x, v[r].y), fmaxf(v[r].z, v[r].w)));
        }
      }
    }
  }
  if (!a.level_max) return;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    for (int o = 32; o >= 1; o >>= 1) m[k] = fmaxf(m[k], __shfl_xor(m[k], o, 64));
    if ((threadIdx.x & 63) == 0) mx[k][threadIdx.x >> 6] = m[k];
  }
  __syncthreads();
  if (threadIdx.x < K) {
    const int k = threadIdx.x;
    const float v = fmaxf(fmaxf(mx[k][0], mx[k][1]), fmaxf(mx[k][2], mx[k][3]));
    float* out = a.level_max + (child - 1 - k);
    if (v > *out) atomicMax(reinterpret_cast<unsigned int*>(out), __float_as_uint(v));
  }
}

// Every level above `child` of the pools that cover the rows [lo, hi), where
// level child - 1 has at most kPathNodes of them.  Columns do not meet, so a
// workgroup takes 16 columns through all levels by itself: thread (r, q) holds
// columns 4 q .. 4 q + 3 of the level's r-th pool, the levels pass through LDS,
// and the siblings outside the range (at most one at each end of a level,
// which nothing here writes) are read up front.  The time is the chain of
// levels: an insert of 100 rows (21 levels, d = 512, bfloat16 copies) took 42
// launches, about 180 us of the call, now one of 12 us.
template <bool MAXP>
__global__ __launch_bounds__(4 * kPathNodes) void k_tree_path(TreeArgs a, int child) {
  if (refused(a.gate, a.bound)) return;
  __shared__ float4 buf[2][kPathNodes][4];
  __shared__ float4 edge[GT_MAX_LEVELS][2][4];
  const int t = threadIdx.x, q = t & 3, r = t >> 2;
  const int c = blockIdx.x * 16 + 4 * q;
  auto range = [&](int l, int64_t& x, int64_t& y) {
    x = a.lo >> (a.depth - l);
    y = (a.hi - 1) >> (a.depth - l);
  };
  for (int i = t; i < (child - 1) * 8; i += blockDim.x) {
    // siblings of level l = 1 .. child - 1: left (of an odd first pool), right
    // (of an even last one)
    const int l = 1 + (i >> 3), side = (i >> 2) & 1, e = i & 3;
    int64_t x, y;
    range(l, x, y);
    const bool has = side == 0 ? (x & 1) : !(y & 1);
    const int64_t row = (int64_t(1) << l) - 1 + (side == 0 ? x - 1 : y + 1);
    if (has)
      edge[l][side][e] = *reinterpret_cast<const float4*>(a.tree + (size_t)row * a.w + blockIdx.x * 16 + 4 * e);
  }
  int64_t lo, hi;
  range(child - 1, lo, hi);
  if (lo + r <= hi) {
    const float* rows = child == a.depth ? a.leaves : a.tree + (size_t)((int64_t(1) << child) - 1) * a.w;
    const float* p = rows + (size_t)(2 * (lo + r)) * a.w + c;
    const float4 v = pool4<MAXP>(*reinterpret_cast<const float4*>(p),
                                 *reinterpret_cast<const float4*>(p + a.w));
    buf[0][r][q] = v;
    store_pool4(a, child - 1, lo + r, c, v);
    if (a.level_max) raise_level_max(a, child - 1, v);
  }
  for (int l = child - 2, k = 0; l >= 0; --l, k ^= 1) {
    __syncthreads();
    const int64_t clo = lo, chi = hi;  // the children's range
    range(l, lo, hi);
    if (lo + r <= hi) {
      float4 v[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int64_t ch = 2 * (lo + r) + s;
        v[s] = ch < clo ? edge[l + 1][0][q] : ch > chi ? edge[l + 1][1][q] : buf[k][ch - clo][q];
      }
      const float4 x = pool4<MAXP>(v[0], v[1]);
      buf[k ^ 1][r][q] = x;
      store_pool4(a, l, lo + r, c, x);
      if (a.level_max) raise_level_max(a, l, x);
    }
  }
}

// Rows of a tree that cover none of its first n leaves are zero: one grid row
// per level clears the pools past the level's last populated one.
__global__ void k_zero_tails(uint4* tree, int row16, int depth, int64_t n) {
  const int l = blockIdx.y;
  const int64_t first = n > 0 ? ((n - 1) >> (depth - l)) + 1 : 0;
  const int64_t base = ((int64_t(1) << l) - 1 + first) * row16;
  const int64_t count = ((int64_t(1) << l) - first) * row16;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    tree[base + i] = make_uint4(0u, 0u, 0u, 0u);
}

// Bottom level of the max/min tree of a signed index (paper Sec. 2, negative
// descriptors).  Pool j of level depth-1 holds leaves 2j and 2j+1; only leaves
// below n are members.  Row j gets [max_k + B | B - min_k] over its members in
// columns k < d, each term rounded up (every term is >= 0 because |f_k| <= B),
// zero in the padding columns and for a pool without members.  The maximum of
// the shifted rows is taken term by term, which is the shifted max and min.
__global__ void k_signed_bottom(const float* __restrict__ leaves, float* __restrict__ parent,
                                int64_t first, int64_t nodes, int dp, int d, int64_t n,
                                float bound, uint16_t* parent16, const IngestOut* gate) {
  if (refused(gate, bound)) return;
  const int pw = 2 * dp, qd = pw / 4;
  const int64_t total = nodes * qd;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = first + i / qd;
    const int k = (int)(i % qd) * 4;          // column of the shifted row
    const bool hi = k >= dp;                  // second half: B - f
    const int c = hi ? k - dp : k;            // feature column
    float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int m = 0; m < 2; ++m) {
      const int64_t leaf = 2 * j + m;
      if (leaf >= n) break;
      const float4 v = *reinterpret_cast<const float4*>(leaves + leaf * dp + c);
      const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (c + e < d) {
          const float t = hi ? add_up(bound, -x[e]) : add_up(x[e], bound);
          o[e] = fmaxf(o[e], t);
        }
      }
    }
    *reinterpret_cast<float4*>(parent + j * pw + k) = make_float4(o[0], o[1], o[2], o[3]);
    if (parent16)
      *reinterpret_cast<uint2*>(parent16 + j * pw + k) =
          make_uint2((uint32_t)bf16_up(o[0]) | ((uint32_t)bf16_up(o[1]) << 16),
                     (uint32_t)bf16_up(o[2]) | ((uint32_t)bf16_up(o[3]) << 16));
  }
}

// Largest value of a level (a float8 level that an insert outgrew).
__global__ __launch_bounds__(256) void k_level_max(const float4* __restrict__ rows, int64_t count4,
                                                   float* out) {
  __shared__ float mx[4];
  float m = 0.0f;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count4;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float4 v = rows[i];
    m = fmaxf(m, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
  }
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) mx[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
    if (m > *out) atomicMax(reinterpret_cast<unsigned int*>(out), __float_as_uint(m));
  }
}

// float8 scale exponents of all levels from their largest values.
__global__ void k_fp8_exps(const float* level_max, int depth, int* lexp) {
  if ((int)threadIdx.x < depth) lexp[threadIdx.x] = fp8_exp_for(level_max[threadIdx.x]);
}

// float8 copies of the levels first .. last in one pass over their rows; the
// rows past a level's last populated pool are zero.
__global__ void k_quant_fp8(const float* __restrict__ tree, uint8_t* __restrict__ p8, int w,
                            int first, int last, int depth, int64_t n, const int* lexp,
                            unsigned int* over) {
  const int g = w / 4;
  const int64_t row0 = (int64_t(1) << first) - 1;
  const int64_t total = ((int64_t(2) << last) - 1 - row0) * g;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = row0 + i / g;
    const int l = 63 - __clzll((unsigned long long)(row + 1));
    const int64_t j = row + 1 - (int64_t(1) << l);
    const size_t at = (size_t)row * w + (size_t)(i % g) * 4;
    uint32_t q[4] = {0u, 0u, 0u, 0u};
    if (n > 0 && j <= (n - 1) >> (depth - l)) {
      const float4 v = *reinterpret_cast<const float4*>(tree + at);
      const int e = lexp[l];
      q[0] = e4m3_up_f32(v.x, e);
      q[1] = e4m3_up_f32(v.y, e);
      q[2] = e4m3_up_f32(v.z, e);
      q[3] = e4m3_up_f32(v.w, e);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (q[k] == 0xFFu) {
          atomicOr(&over[l], 1u);
          q[k] = 0x7Eu;
        }
    }
    *reinterpret_cast<uint32_t*>(p8 + at) = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
  }
}

// Start of a query call: clears the call's counters and prepares its queries,
// in one launch (every workgroup clears a share; nothing prepared lies in the
// cleared ranges).  A wave takes one (padded) query and a workgroup eight, one
// byte of a tile's mask of live queries, which so needs no atomics and no
// clearing; a query that is not allowed is marked in qexp.  Bound by its round
// trips: 1024 queries of 1000 columns 12.5 us (16 and 3 as two launches), 4096
// 20 (30 and 4), one query 10 (5 and 3, and a launch).
constexpr int kPrepQueries = 8;
typedef __attribute__((address_space(3))) void* lds_ptr;
template <bool KARG>
__global__ __launch_bounds__(64 * kPrepQueries) void k_query_prep(QueryPrep a, RhoArg r) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  {
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + t, step = (int64_t)gridDim.x * blockDim.x;
    for (int k = 0; k < 3; ++k)
      for (int64_t i = i0; i < a.n16[k]; i += step) a.p[k][i] = make_uint4(0u, 0u, 0u, 0u);
  }
  if ((int)blockIdx.x >= a.nq_pad / kPrepQueries) return;
  __shared__ int live[kPrepQueries];
  const int b = blockIdx.x * kPrepQueries + wave, d = a.d, dp = a.dp;
  const bool real = b < a.nq;
  const bool sgn = a.sbound > 0.0f;  // signed index: any finite value
  double rho = 0.0;
  if (real) rho = KARG ? r.v[b] : a.rho_src[b];
  // The wave's row, and the root pool's, in LDS.  (The loads are all in flight
  // from a rolled loop; unrolled to hold them in registers the kernel was 18 KB
  // of code run once, 13 us for one query of 1000 columns, for its fetch.)
  extern __shared__ float rows[];
  float* const row = rows + wave * dp;
  float* const root = rows + kPrepQueries * dp;
  const float* q = a.q + (int64_t)b * d;
#pragma unroll 1
  for (int c = 0; c < dp; c += 64)
    if (real && c + lane < d)
      __builtin_amdgcn_global_load_lds((const void*)(q + c + lane), (lds_ptr)(row + c), 4, 0, 0);
    else
      row[c + lane] = 0.0f;
  if (a.root)
#pragma unroll 1
    for (int c = 64 * wave; c < dp; c += 64 * kPrepQueries)
      __builtin_amdgcn_global_load_lds((const void*)(a.root + c + lane), (lds_ptr)(root + c), 4, 0, 0);
  const double mmin = *a.mmin;
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  __syncthreads();
  // Column k belongs to partial sum (k / 64) % 4 of lane k % 64: |q|^2 and
  // |q|_1 are added in a fixed order (deterministic, relative error below
  // 2^-40 for d <= 4096; the thresholds' slack covers far more).  The
  // canonical sequential sum, which the float64 recheck needs bit for bit,
  // is formed there for the few candidates that reach it.
  float mx = 0.0f;
  bool bad = false;
  double l1[4] = {0.0, 0.0, 0.0, 0.0}, l2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int c = lane; c < dp; c += 256) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = c + 64 * u;
      if (k >= dp) continue;
      const float v = row[k];
      if (sgn ? !isfinite(v) : (!(v >= 0.0f) || isinf(v))) bad = true;
      mx = fmaxf(mx, v);
      l1[u] += (double)fabsf(v);
      l2[u] = __fma_rn((double)v, (double)v, l2[u]);
      a.qf[(int64_t)b * dp + k] = v;
      if (sgn) {
        // walk query [max(q,0) | max(-q,0)] against rows [max + B | B - min]
        const float vp = fmaxf(v, 0.0f), vn = fmaxf(-v, 0.0f);
        const int64_t at = (int64_t)b * a.pw + k;
        if (a.qw) {
          a.qw[at] = vp;
          a.qw[at + dp] = vn;
        }
        if (a.qbf) {
          a.qbf[at] = bf16_up(vp);
          a.qbf[at + dp] = bf16_up(vn);
        }
      } else if (a.qbf) {
        a.qbf[(int64_t)b * dp + k] = bf16_up(v);
      }
    }
  }
  // |q|_1 + |root pool|_1 (only an upper bound is needed); for a signed index
  // |q|_1 alone, which sets the threshold's shift B |q|_1
  if (a.root)
#pragma unroll 1
    for (int c = lane; c < dp; c += 256) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c + 64 * u < dp) l1[u] += (double)root[c + 64 * u];
    }
#pragma unroll 1
  for (int o = 32; o >= 1; o >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, o, 64));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      l1[u] += __shfl_xor(l1[u], o, 64);
      l2[u] += __shfl_xor(l2[u], o, 64);
    }
  }
  bad = __any(bad);
  const double qq = (l2[0] + l2[1]) + (l2[2] + l2[3]);
  // float8 query scale 2^e with qmax / 2^e in (224, 448]
  int e = 0;
  if (mx > 0.0f) {
    int ex;
    const double m = frexp((double)mx / 448.0, &ex);
    e = (m == 0.5) ? ex - 1 : ex;
  }
  if (a.q8)
#pragma unroll 1
    for (int k = 4 * lane; k < dp; k += 256) {
      const float4 v = *reinterpret_cast<const float4*>(row + k);
      *reinterpret_cast<uint32_t*>(a.q8 + (int64_t)b * dp + k) =
          (e4m3_up_f32(v.x, e) & 0xFFu) | (e4m3_up_f32(v.y, e) & 0xFFu) << 8 |
          (e4m3_up_f32(v.z, e) & 0xFFu) << 16 | (e4m3_up_f32(v.w, e) & 0xFFu) << 24;
    }
  const bool on = real && qq > 0.0 && !bad;
  if (lane == 0) {
    live[wave] = on;
    const double nrm = __dsqrt_rn(qq);
    if (real) a.rho[b] = rho;
    a.qq[b] = qq;
    a.qexp[b] = bad ? kBadQuery : e;
    a.invn_q[b] = qq > 0.0 ? (float)__ddiv_rn(1.0, nrm) : 0.0f;
    float th = INFINITY, tg = INFINITY;
    const double l1s = (l1[0] + l1[1]) + (l1[2] + l1[3]);
    if (on) {
      if (rho <= 0.0) {
        th = -INFINITY;
        tg = -INFINITY;
      } else {
        // cos >= rho with the float64 definition implies the real cosine is
        // at least rho * (1 - 2e-11) for d <= 4096; every member norm is at
        // least m_min, so a pool holding a neighbour scores >= tau (reals).
        const double reff = rho * (1.0 - 4e-11);
        const double tau = reff * nrm * mmin * (1.0 - 4e-11);
        if (sgn) {
          // A member's q.f is at most the pool's max/min score U, and the
          // walk computes [q+ | q-] . [max + B | B - min] = U + B |q|_1 over
          // pw non-negative products.  The shift is taken slightly low (the
          // float64 |q|_1 of <= 4096 terms is within 2^-40 of the real one).
          // Products of mixed sign in the leaf GEMM carry an error relative
          // to sum |q_k f_k| <= |q| |f|, hence rho - slack there.
          const double sl = pool_slack(a.pw);
          const double kappa = (double)a.sbound * l1s * (1.0 - 1e-12);
          th = f64_to_f32_down((tau + kappa) * (1.0 - sl) - 2.0 * a.pw * 0x1p-126);
          const double cg = reff * (1.0 - 4e-11) - pool_slack(dp);
          tg = cg > 0.0 ? f64_to_f32_down(cg * nrm) : -INFINITY;
        } else {
          const double sl = pool_slack(dp);
          th = f64_to_f32_down(tau * (1.0 - sl) - 2.0 * dp * 0x1p-126);
          tg = f64_to_f32_down(reff * nrm * (1.0 - 4e-11) * (1.0 - sl));
        }
      }
    }
    a.thr[b] = th;
    a.thr_gemm[b] = tg;
    if (a.sabs && !sgn) {
      // absolute term of the subtraction step's lower bound: 2^-125 (|S|_1 +
      // |q|_1 + dp 2^-126) + 2^-126, a normal float32 rounded up
      const double v = ldexp(1.01 * l1s + (double)dp * 0x1p-126, -125) + 0x1p-126;
      float f = (float)v;
      if ((double)f < v) f = __uint_as_float(__float_as_uint(f) + 1u);
      a.sabs[b] = f;
    }
  }
  __syncthreads();
  if (t == 0) {
    uint32_t m = 0u;
#pragma unroll
    for (int w = 0; w < kPrepQueries; ++w) m |= (uint32_t)live[w] << w;
    uint8_t* tile = reinterpret_cast<uint8_t*>(a.tile_mask + blockIdx.x * kPrepQueries / a.tq);
    const int byte = (int)(blockIdx.x * kPrepQueries % a.tq) / 8;
    tile[byte] = (uint8_t)m;
    if (a.tq == 32) tile[byte + 4] = 0u;
  }
}

inline int grid_for(int64_t work, int block) {
  int64_t g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (int)g;
}

}  // namespace

hipError_t launch_zero_u32(uint32_t* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_ingest_reset(IngestOut* o, hipStream_t s) {
  hipLaunchKernelGGL(k_ingest_reset, dim3(1), dim3(64), 0, s, o);
  return hipGetLastError();
}

template <int R>
hipError_t launch_ingest_rows(const void* src, int dtype, int64_t rows, int d, int dp,
                              float* leaves, double* ff, float* invn, float* nf, IngestOut* o,
                              int allow_negative, hipStream_t s) {
  // wide loads: rows whose starts are all aligned to four features
  const bool vec = d % 4 == 0 && reinterpret_cast<uintptr_t>(src) % (dtype == GT_F32 ? 16 : 8) == 0;
  const dim3 grid((unsigned)((rows + R - 1) / R));
  if (vec)
    hipLaunchKernelGGL((k_ingest<R, true>), grid, dim3(256), 0, s, src, dtype, rows, d, dp, leaves,
                       ff, invn, nf, o, allow_negative);
  else
    hipLaunchKernelGGL((k_ingest<R, false>), grid, dim3(256), 0, s, src, dtype, rows, d, dp, leaves,
                       ff, invn, nf, o, allow_negative);
  return hipGetLastError();
}

hipError_t launch_ingest(const void* src, int dtype, int64_t rows, int d, int dp, float* leaves,
                         double* ff, float* invn, float* nf, IngestOut* o, bool allow_negative,
                         hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  // 64-row tiles once they fill the chip, 4-row tiles below
  if (rows >= 8192)
    return launch_ingest_rows<64>(src, dtype, rows, d, dp, leaves, ff, invn, nf, o, allow_negative, s);
  return launch_ingest_rows<4>(src, dtype, rows, d, dp, leaves, ff, invn, nf, o, allow_negative, s);
}

hipError_t launch_signed_bottom(const float* leaves, float* parent, int64_t first, int64_t nodes,
                                int dp, int d, int64_t n, float bound, uint16_t* parent16,
                                const IngestOut* gate, hipStream_t s) {
  if (nodes <= 0) return hipSuccess;
  if (dp % 4 || d > dp || first < 0 || n < 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_signed_bottom, dim3(grid_for(nodes * (2 * dp / 4), 256)), dim3(256), 0, s,
                     leaves, parent, first, nodes, dp, d, n, bound, parent16, gate);
  return hipGetLastError();
}

// The pools above level `child` that cover the rows [lo, hi), bottom-up: four
// levels a launch while a level has more pools than the path kernel holds.
template <bool MAXP>
hipError_t launch_tree_levels(const TreeArgs& a, int child, hipStream_t s) {
  while (child > 0) {
    const int sh = a.depth - (child - 1);
    if (((a.hi - 1) >> sh) - (a.lo >> sh) + 1 <= kPathNodes) {
      hipLaunchKernelGGL(k_tree_path<MAXP>, dim3(a.w / 16), dim3(4 * kPathNodes), 0, s, a, child);
      return hipGetLastError();
    }
    // (more than kPathNodes pools: at least seven levels are left)
    const int st = a.depth - (child - 4);
    const int64_t threads = (((a.hi - 1) >> st) - (a.lo >> st) + 1) * (a.w / 4);
    hipLaunchKernelGGL((k_tree<MAXP, 4>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       a, child);
    if (hipError_t e = hipGetLastError()) return e;
    child -= 4;
  }
  return hipSuccess;
}

hipError_t launch_tree_update(const TreeArgs& a, bool max_pool, int child, hipStream_t s) {
  if (a.hi <= a.lo || child <= 0) return hipSuccess;
  if (a.lo < 0 || child > a.depth || a.depth > 31 || a.hi > (int64_t(1) << a.depth) || a.w % 16 ||
      (a.p8 && (!a.lexp || !a.over)))
    return hipErrorInvalidValue;
  return max_pool ? launch_tree_levels<true>(a, child, s) : launch_tree_levels<false>(a, child, s);
}

hipError_t launch_zero_tails(void* tree, int row_bytes, int depth, int64_t n, hipStream_t s) {
  if (depth <= 0 || row_bytes % 16) return depth <= 0 ? hipSuccess : hipErrorInvalidValue;
  const int64_t most = ((int64_t(1) << (depth - 1)) - (n > 0 ? ((n - 1) >> 1) + 1 : 0)) * (row_bytes / 16);
  const unsigned gx = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, (most + 1023) / 1024));
  hipLaunchKernelGGL(k_zero_tails, dim3(gx, (unsigned)depth), dim3(256), 0, s,
                     static_cast<uint4*>(tree), row_bytes / 16, depth, n);
  return hipGetLastError();
}

hipError_t launch_level_max(const float* rows, int64_t nrows, int dp, float* out_max,
                            hipStream_t s) {
  const int64_t count = nrows * dp / 4;
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_level_max, dim3((unsigned)std::min<int64_t>(2048, (count + 1023) / 1024)),
                     dim3(256), 0, s, reinterpret_cast<const float4*>(rows), count, out_max);
  return hipGetLastError();
}

hipError_t launch_fp8_exps(const float* level_max, int depth, int* lexp, hipStream_t s) {
  hipLaunchKernelGGL(k_fp8_exps, dim3(1), dim3(64), 0, s, level_max, depth, lexp);
  return hipGetLastError();
}

hipError_t launch_quant_fp8(const float* tree, uint8_t* p8, int w, int first, int last, int depth,
                            int64_t n, const int* lexp, unsigned int* over, hipStream_t s) {
  if (first < 0 || last >= depth || first > last || w % 4) return hipErrorInvalidValue;
  const int64_t total = ((int64_t(2) << last) - (int64_t(1) << first)) * (w / 4);
  hipLaunchKernelGGL(k_quant_fp8, dim3(grid_for(total, 256 * 4)), dim3(256), 0, s, tree, p8, w,
                     first, last, depth, n, lexp, over);
  return hipGetLastError();
}

hipError_t launch_query_prep(QueryPrep a, const double* rho, hipStream_t s) {
  if (a.nq < 0 || a.nq > a.nq_pad || a.nq_pad % kPrepQueries || a.nq_pad % a.tq ||
      (a.tq != 32 && a.tq != 64) || a.d < 1 || a.d > a.dp || a.dp % 128 ||
      (a.sbound > 0.0f && a.pw != 2 * a.dp))
    return hipErrorInvalidValue;
  for (int k = 0; k < 3; ++k)
    if (reinterpret_cast<uintptr_t>(a.p[k]) % 16) return hipErrorInvalidValue;
  if (a.nq == 0) a.nq_pad = 0;  // only clear
  const dim3 grid((unsigned)std::max(128, a.nq_pad / kPrepQueries)), block(64 * kPrepQueries);
  const int lds = (kPrepQueries + 1) * a.dp * 4;
  const void* fn = reinterpret_cast<const void*>(rho ? k_query_prep<true> : k_query_prep<false>);
  if (lds + 1024 > 160 * 1024) return hipErrorInvalidValue;
  if (hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) return err;
  RhoArg r;
  if (rho) {
    if (a.nq > kRhoArg) return hipErrorInvalidValue;
    for (int i = 0; i < a.nq; ++i) r.v[i] = rho[i];
    hipLaunchKernelGGL(k_query_prep<true>, grid, block, lds, s, a, r);
  } else {
    hipLaunchKernelGGL(k_query_prep<false>, grid, block, lds, s, a, r);
  }
  return hipGetLastError();
}

}  // namespace gt
