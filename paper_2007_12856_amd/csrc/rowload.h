// Device helpers shared by the matrix-core kernels that stage rows of NCDHW tensors through registers: row pieces by branch-free
// buffer loads for any width and alignment, their transposition into 16-byte units of 8 channels, the 32x32x16 product.
#pragma once
#include "common.h"

namespace h3d {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int ROW_OOB = (int)0x80000000;   // byte offset beyond every buffer: such a lane reads zeros, its store is dropped

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// g = v where the saved output m is > 0, else v * slope, rounded to bf16; two elements
__device__ __forceinline__ uint32_t mask2(uint32_t v, uint32_t m, float slope) {
  float v0 = __uint_as_float(v << 16), v1 = __uint_as_float(v & 0xffff0000u);
  if (!(__uint_as_float(m << 16) > 0.f)) v0 *= slope;
  if (!(__uint_as_float(m & 0xffff0000u) > 0.f)) v1 *= slope;
  return pack_bf16x2(v0, v1);
}
__device__ __forceinline__ uint4 mask8(uint4 v, uint4 m, float slope) {
  return uint4{mask2(v.x, m.x, slope), mask2(v.y, m.y, slope), mask2(v.z, m.z, slope), mask2(v.w, m.w, slope)};
}
// 8 elements moved down by s (0 .. 7), zeros behind them
__device__ __forceinline__ uint4 shift8(uint4 v, int s) {
  if (s & 4) v = uint4{v.z, v.w, 0u, 0u};
  if (s & 2) v = uint4{v.y, v.z, v.w, 0u};
  if (s & 1) v = uint4{__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16), __builtin_amdgcn_alignbit(v.w, v.z, 16), v.w >> 16};
  return v;
}

// 8 elements of a row of `w` from column c >= 0 on; `off` = element offset of the ROW in the sample, `span` = elements of the
// sample (>= 8).  One 16-byte buffer load without a branch (a branch around each load makes the compiler wait for every one of
// them where the paths meet: stride-2 backward-data, 64->128 on 64^3: 55 -> 48 us, backward-filter 52 -> 46).
//   V16: w % 8 == 0, c % 8 == 0 and 16-byte aligned rows: a group is inside the row or outside as a whole.
//   else: the load may start at any 2-byte address and run over the end of the row into the next one, never past the sample;
//   fix8 then drops what does not belong to the row.
template <bool V16>
__device__ __forceinline__ uint4 row8(__amdgpu_buffer_rsrc_t rs, int off, int c, int w, int span, bool ok) {
  const int f = V16 ? off + c : min(off + c, span - 8);
  const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, ok && c < w ? 2 * f : ROW_OOB, 0, 0);
  return uint4{t.x, t.y, t.z, t.w};
}
template <bool V16>
__device__ __forceinline__ uint4 fix8(uint4 v, int off, int c, int w, int span) {
  if (V16) return v;
  const int s = off + c - min(off + c, span - 8);      // elements the load was moved forward by (the end of the sample only)
  if (__builtin_amdgcn_ballot_w64(s > 0)) v = shift8(v, s);
  const int k = w - c;                                 // elements that belong to the row
  v.x &= k >= 2 ? 0xffffffffu : k == 1 ? 0xffffu : 0u;
  v.y &= k >= 4 ? 0xffffffffu : k == 3 ? 0xffffu : 0u;
  v.z &= k >= 6 ? 0xffffffffu : k == 5 ? 0xffffu : 0u;
  v.w &= k >= 8 ? 0xffffffffu : k == 7 ? 0xffffu : 0u;
  return v;
}
__device__ __forceinline__ uint32_t row1(__amdgpu_buffer_rsrc_t rs, int off, int c, int w, bool ok) {
  return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, ok && c >= 0 && c < w ? 2 * (off + c) : ROW_OOB, 0, 0);
}

// v[e] = 8 consecutive columns of channel e; result: four (all eight) channels of column col
__device__ __forceinline__ uint2 column_half(const uint4* v, int col) {
  uint32_t d[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) d[e] = (col >> 1) == 0 ? v[e].x : (col >> 1) == 1 ? v[e].y : (col >> 1) == 2 ? v[e].z : v[e].w;
  const uint32_t sel = (col & 1) ? 0x07060302u : 0x05040100u;
  return uint2{__builtin_amdgcn_perm(d[1], d[0], sel), __builtin_amdgcn_perm(d[3], d[2], sel)};
}
__device__ __forceinline__ uint4 column_unit(const uint4 (&v)[8], int col) {
  const uint2 lo = column_half(v, col), hi = column_half(v + 4, col);
  return uint4{lo.x, lo.y, hi.x, hi.y};
}

__device__ __forceinline__ f32x16 mfma32(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// row of the accumulator block that register r of this lane holds
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r / 4) + 4 * (lane >> 5) + (r % 4); }


}  // namespace h3d
