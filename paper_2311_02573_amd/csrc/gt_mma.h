// Pool formats of the walk kernels and their 16x16 matrix products.
#pragma once
#include "gt_internal.h"

namespace gt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

template <int FMT>
struct WalkFmt;
template <>
struct WalkFmt<GT_POOL_F32> {
  static constexpr int TQ = kQueriesPerTileF32, ESZ = 4, MAXDP = kMaxDpF32;
};
template <>
struct WalkFmt<GT_POOL_BF16> {
  static constexpr int TQ = kQueriesPerTile16, ESZ = 2, MAXDP = kMaxDpBf16;
};
template <>
struct WalkFmt<GT_POOL_FP8E4M3> {
  static constexpr int TQ = kQueriesPerTile16, ESZ = 1, MAXDP = kMaxDpFp8;
};

__device__ __forceinline__ uint4 ld_global16(const unsigned char* p) {
  return *reinterpret_cast<const uint4*>(p);
}
__device__ __forceinline__ uint4 ld_lds16(const unsigned char* p) {
  return *reinterpret_cast<const uint4*>(p);
}

// A tile's query rows (stage_columns: nbytes of each) to LDS rows of stride
// rowbytes + 16 (rs), which spreads the banks, by direct loads of 64 lanes x 16
// bytes: wave w of WAVES copies rows w, w + WAVES, ...  All of a row's loads are
// in flight, and no thread divides an index by the row's length (through
// registers, 32 divisions a thread for 64 x 2 KB: 2^20 x 1000, 1024 queries,
// three subtraction levels 340 us, 351 before; 2^19 x 800 240, 260).
constexpr int kStageChunk = 1024;
template <int ROWS, int WAVES>
__device__ __forceinline__ void stage_columns(unsigned char* lds, int rs, const unsigned char* src,
                                              int rowbytes, int nbytes, int wave, int lane) {
  typedef __attribute__((address_space(3))) void* lds_ptr;
  static_assert(ROWS % WAVES == 0, "whole rows per wave");
#pragma unroll
  for (int m = 0; m < ROWS / WAVES; ++m) {
    const int row = wave + m * WAVES;
    for (int c = 0; c < nbytes; c += kStageChunk)
      if (c + 16 * lane < nbytes)
        __builtin_amdgcn_global_load_lds((const void*)(src + (size_t)row * rowbytes + c + 16 * lane),
                                         (lds_ptr)(lds + row * rs + c), 16, 0, 0);
  }
}
template <int ROWS, int WAVES>
__device__ __forceinline__ void stage_rows(unsigned char* lds, const unsigned char* src, int rowbytes,
                                           int wave, int lane) {
  stage_columns<ROWS, WAVES>(lds, rowbytes + 16, src, rowbytes, rowbytes, wave, lane);
}
// This wave's loads, direct ones too, which a barrier alone does not wait for.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0070); }

// 16x16 forms: one 16-byte slice per lane, 64 bytes of each of 16 rows per
// wave instruction.  Lane l holds row (l % 16) and slice (l / 16) of a 64-byte
// step; the A and B lanes of the same index hold the same dimensions.
// Accumulator: register i of lane l is row 4 (l / 16) + i, column l % 16.
typedef __attribute__((ext_vector_type(4))) float f32x4;
template <int FMT>
__device__ __forceinline__ void mma16x16(const uint4& a, const uint4& b, f32x4& acc);
template <>
__device__ __forceinline__ void mma16x16<GT_POOL_BF16>(const uint4& a, const uint4& b, f32x4& acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma16x16<GT_POOL_FP8E4M3>(const uint4& a, const uint4& b,
                                                          f32x4& acc) {
  const long a0 = (long)(((unsigned long)a.y << 32) | a.x);
  const long a1 = (long)(((unsigned long)a.w << 32) | a.z);
  const long b0 = (long)(((unsigned long)b.y << 32) | b.x);
  const long b1 = (long)(((unsigned long)b.w << 32) | b.z);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a0, b0, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a1, b1, acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma16x16<GT_POOL_F32>(const uint4& a, const uint4& b, f32x4& acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// gfx950 f8f6f4 forms for float8 (e4m3: format 0 for both operands, no
// block scales): 32 bytes per lane, the lane's two 16-byte slices a0, a1 and
// the matching slices b0, b1 of the other operand, so A and B lanes again
// carry the same dimensions.  Same numerics as the fp8 forms above (measured
// equal), twice the products per instruction.
typedef __attribute__((ext_vector_type(8))) int i32x8;
__device__ __forceinline__ i32x8 pack32(const uint4& x0, const uint4& x1) {
  i32x8 v;
  v[0] = (int)x0.x; v[1] = (int)x0.y; v[2] = (int)x0.z; v[3] = (int)x0.w;
  v[4] = (int)x1.x; v[5] = (int)x1.y; v[6] = (int)x1.z; v[7] = (int)x1.w;
  return v;
}
__device__ __forceinline__ void mma_f8_16x16x128(const uint4& a0, const uint4& a1, const uint4& b0,
                                                 const uint4& b1, f32x4& acc) {
  acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(pack32(a0, a1), pack32(b0, b1), acc, 0, 0,
                                                        0, 0, 0, 0);
}

}  // namespace gt
