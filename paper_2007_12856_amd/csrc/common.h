// Internal definitions shared by the HIP translation units of libh3d (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "h3d.h"

namespace h3d {

h3d_status fail(void* handle, h3d_status st, const char* fmt, ...);

struct Handle {
  int device = 0;
  int num_cu = 256;
  void* scratch = nullptr;    // this device's copy of the library-owned scratch array (static_scratch.hip)
  char err[512] = {0};
  char kernel[160] = {0};     // principal kernel of the last compute call (h3d_last_kernel)
  bool kernel_noted = false;
};

// size of the library-owned scratch array behind h3d_conv3d_bwd_filter_static
#define H3D_STATIC_SCRATCH_BYTES (96u << 20)
h3d_status static_scratch_init(Handle* hd);

// Slab geometry as the kernels see it (element strides, not bytes).
struct Geo {
  int n, c, d, h, w, hlo, hhi;
  int ds;            // stored planes = hlo + d + hhi
  int64_t doff, dglob;
  int64_t plane;     // h*w
  int64_t cstride;   // ds*h*w
  int64_t nstride;   // c*ds*h*w
};

inline Geo make_geo(const h3d_tensor* t) {
  Geo g;
  g.n = t->n; g.c = t->c; g.d = t->d; g.h = t->h; g.w = t->w; g.hlo = t->halo_lo; g.hhi = t->halo_hi;
  g.ds = t->halo_lo + t->d + t->halo_hi;
  g.doff = t->d_offset; g.dglob = t->d_global;
  g.plane = (int64_t)t->h * t->w;
  g.cstride = t->c_stride ? t->c_stride : g.plane * g.ds;
  g.nstride = t->n_stride ? t->n_stride : g.cstride * t->c;
  return g;
}

// elements from a sample's first stored one to behind its last: what a wide load may touch.  A view's nstride is its parent's and reaches
// past the parent's end when the view does not start at channel 0.
__host__ __device__ inline int64_t stored_span(const Geo& g) { return (g.c - 1) * g.cstride + g.ds * g.plane; }

inline bool is_packed(const h3d_tensor* t) { return t->c_stride == 0 && t->n_stride == 0; }
// elements spanned by one sample (all channels), with the tensor's real strides
inline int64_t sample_span(const h3d_tensor* t) {
  const int64_t cs = t->c_stride ? t->c_stride : (int64_t)(t->halo_lo + t->d + t->halo_hi) * t->h * t->w;
  return t->n_stride ? t->n_stride : cs * t->c;
}

inline size_t elt_size(int dtype) { return dtype == H3D_F32 ? 4 : 2; }

h3d_status fail(void* handle, h3d_status st, const char* fmt, ...);
h3d_status check_tensor(void* handle, const h3d_tensor* t, const char* name);          // strided plane runs allowed
h3d_status check_tensor_packed(void* handle, const h3d_tensor* t, const char* name);   // packed tensors only
// every needed in-volume input plane for output planes [lo,hi) (local indices) must be stored
bool halo_covers(const h3d_tensor* in, int64_t lo, int64_t hi);
bool same_shard(const h3d_tensor* a, const h3d_tensor* b);
h3d_status launch_status(void* handle, const char* what);   // also records `what` as the call's kernel unless one was noted
// name of the kernel that does the arithmetic of the call under way (shown by h3d_last_kernel)
void note_kernel(void* handle, const char* fmt, ...);

// raises a kernel's dynamic LDS limit once (`done`: one flag per kernel); a failure is reported and tried again by the next call
template <typename K>
h3d_status raise_lds_limit(void* handle, K kern, size_t bytes, bool* done) {
  if (*done) return H3D_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
    return fail(handle, H3D_EHIP, "cannot raise the dynamic LDS limit to %zu bytes", bytes);
  *done = true;
  return H3D_OK;
}

inline float act_slope(int act, float alpha) { return act == H3D_ACT_LEAKY ? alpha : (act == H3D_ACT_RELU ? 0.f : 1.f); }

// ---- bf16 storage helpers (device) -------------------------------------------------------------
typedef uint16_t bf16_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {  // round to nearest even; NaN stays NaN
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
// two floats -> packed bf16x2 (low half = first), round to nearest even: one v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// ---- global -> LDS copies without registers (buffer_load ... lds) ---------------------------------------------------
// The instruction is issued from inline assembly on purpose: the compiler's wait-count pass treats a copy into LDS as
// aliasing every later LDS read and puts "s_waitcnt vmcnt(0)" in front of the first one, which serialises a prefetch
// with the arithmetic it was meant to hide behind.  Issued this way the copies are invisible to that pass; the kernel
// itself waits (s_waitcnt vmcnt) and synchronises (barrier) before anyone reads the destination.  Hidden operations can
// only make the compiler's own vmcnt waits longer, never shorter: the counter is decremented in issue order.
typedef int h3d_i32x4 __attribute__((ext_vector_type(4)));
// raw buffer resource: byte range [base, base + bytes), accesses beyond it return zeros
__device__ __forceinline__ h3d_i32x4 lds_dma_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  h3d_i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
// LDS byte address of a pointer into shared memory (wave-uniform)
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p);
}
// 64 lanes x 16 bytes from per-lane byte offsets `voff` of the buffer into 1 KB of LDS at `lds_byte_addr` (lane l at + 16 l)
__device__ __forceinline__ void lds_dma16(h3d_i32x4 rs, uint32_t lds_byte_addr, int voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds_byte_addr), "v"(voff), "s"(rs) : "memory", "m0");
}

// the same with a scalar byte offset on top (not part of the range check: the per-lane offset alone decides)
__device__ __forceinline__ void lds_dma16_row(h3d_i32x4 rs, uint32_t lds_byte_addr, int voff, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_byte_addr), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}

// ---- stores of streaming passes ---------------------------------------------------------------------------------------
// A result larger than the last-level cache can keep for its reader goes past it (non-temporal): written through the cache, its
// dirty lines are evicted in the way of the following pass's reads.  Batch normalisation of 4 x 16 x 128^3 bf16, five passes:
// 387 -> 346 us; a result of 2 x 16 x 128^3 (134 MB) 188 -> 169; smaller ones stay in the 256 MB cache for whoever reads them next.
// A wavefront's store has to cover whole lines (pool_bwd_mask_kernel).
constexpr int64_t STREAM_PAST_CACHE_BYTES = (int64_t)1 << 27;
typedef unsigned int h3d_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store16(void* p, const void* v, bool past_cache) {
  h3d_u32x4 t;
  __builtin_memcpy(&t, v, 16);
  if (past_cache) __builtin_nontemporal_store(t, reinterpret_cast<h3d_u32x4*>(p));
  else __builtin_memcpy(p, &t, 16);
}

template <typename T> struct dtype_of;
template <> struct dtype_of<float> { static constexpr int value = H3D_F32; };
template <> struct dtype_of<bf16_t> { static constexpr int value = H3D_BF16; };

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }      // parts of a workspace start at multiples of 256 bytes

}  // namespace h3d

#define H3D_TRY(expr)                       \
  do {                                      \
    h3d_status _s = (expr);                 \
    if (_s != H3D_OK) return _s;            \
  } while (0)
