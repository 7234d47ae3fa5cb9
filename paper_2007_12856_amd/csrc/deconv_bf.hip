// Filter gradient of the 2x2x2 stride-2 transposed convolution (the U-Net's up-sampling layer) on the matrix cores, bf16 and fp32
// tensors of any width and alignment:
//
//   dW[ci][co][a,b,c] = sum over coarse voxels v = (d,h,w) of x[ci][v] * dy[co][2d+a][2h+b][2w+c],   db[co] = sum of dy[co]
//
// A GEMM whose contraction runs over the coarse voxels.  HBM-bound at the sizes that matter (x + dy once: 671 MB at the U-Net shape against
// 69 GFlop), so what counts is how many bytes are in flight:
//   * a plane of x is one contiguous run whatever its width, and voxel v = h W + w of it meets dy at 2 v + 2 W (h + b) of a fine plane.  A
//     tile is therefore TV consecutive voxels of a plane, not a rectangle: no columns are lost to padding, and only the row number of a
//     piece has to be known (one multiplication).  Pieces of VP voxels, where VP divides the width, never cross a row of dy; with the
//     longest ones (16 bytes of dy) a plane holds whole units of x, with others the last unit may have to be cut.
//   * rows = 16 * MRB input channels: x goes through registers into LDS, one tile ahead (16-byte units, odd pitch per channel);
//     columns = 16 output channels: a lane takes the 32 bytes of dy above its unit of voxels straight into registers, one tile ahead, and
//     splits them into the operands of c = 0 and c = 1, so that each byte of dy is loaded by one lane and each x fragment read feeds two
//     products.  A wavefront has one (a,b), a workgroup of four all of them.  The barrier waits for LDS alone: loads stay in flight.
//   * the products of one tile start from zero and their sum is added to the running one by an ordinary addition: a matrix instruction
//     truncates when it adds to a large sum (2^19 voxels in one chain: db 1.7e-5 from 64 bits; here 1e-7).
// Workgroups of one chunk of voxels that differ in their channels read the same x or dy and follow each other on one XCD.
// 128 -> 64 channels from 64x256x256 bf16: 193 -> 189 us (the form before took whole aligned rows only; a bare read of dy in this order takes
// 100 - 120); 64 -> 64 there 167 -> 144; from 64x256x248, which the direct kernel took: 11650 -> 160; 48 -> 32 from 128x64x92 283 -> 27;
// fp32 128 -> 96 from 32x120x32: 447 -> 48.  Two steps a tile and at most 64 channels at three wavefronts a SIMD: 64 -> 64 167 us with four steps
// and two wavefronts, 144 so.  (Rotating where each workgroup starts in its chunk, against equal low address bits: nothing.)
#include <algorithm>

#include "rowload.h"

namespace h3d {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int DB_RU = 2;                 // K-steps of four units (one per 16 lanes) in a tile
constexpr int DB_PITCH = 4 * DB_RU + 1;  // LDS pitch of a channel in 16-byte units (odd: 16 channels -> 16 bank groups)

struct DbfArgs {
  Geo x, y;
  int cin, cout;
  int tiles_p, ntiles, tiles_per_chunk, nchunks;   // tiles of a plane, in all, of a chunk
  int gco, gci;                                    // groups of 16 output channels / of 16 * MRB input channels
  uint32_t magic;                                  // v / W = umulhi(v, magic) >> shift
  int shift;
  int xspan, yspan;                                // elements of a sample
};

template <typename T> struct Unit;                 // 16 bytes of consecutive voxels
template <> struct Unit<bf16_t> {
  static constexpr int N = 8;
  // v moved down by s elements, those from k on zero
  static __device__ __forceinline__ uint4 fix(uint4 v, int s, int k) {
    if (__builtin_amdgcn_ballot_w64(s > 0)) v = shift8(v, s);
    v.x &= k >= 2 ? 0xffffffffu : k == 1 ? 0xffffu : 0u;
    v.y &= k >= 4 ? 0xffffffffu : k == 3 ? 0xffffu : 0u;
    v.z &= k >= 6 ? 0xffffffffu : k == 5 ? 0xffffu : 0u;
    v.w &= k >= 8 ? 0xffffffffu : k == 7 ? 0xffffu : 0u;
    return v;
  }
};
template <> struct Unit<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ uint4 fix(uint4 v, int s, int k) {
    if (s & 2) v = uint4{v.z, v.w, 0u, 0u};
    if (s & 1) v = uint4{v.y, v.z, v.w, 0u};
    return uint4{k > 0 ? v.x : 0u, k > 1 ? v.y : 0u, k > 2 ? v.z : 0u, k > 3 ? v.w : 0u};
  }
};

// acc[c] += A * (dy of parity c), over the unit's voxels
__device__ __forceinline__ void unit_products(uint4 A, const uint4 (&b)[2], f32x4 (&acc)[2], bf16_t) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A), __builtin_bit_cast(bf16x8, b[c]), acc[c], 0, 0, 0);
}
__device__ __forceinline__ void unit_products(uint4 A, const uint4 (&b)[2], f32x4 (&acc)[2], float) {
  const uint32_t av[4] = {A.x, A.y, A.z, A.w};
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const uint32_t bv[4] = {b[c].x, b[c].y, b[c].z, b[c].w};
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(av[j]), __uint_as_float(bv[j]), acc[c], 0, 0, 0);
    }
}
// 32 bytes of dy above a unit -> the elements of c = 0 and of c = 1
__device__ __forceinline__ void split_parity(const uint32_t (&r)[8], uint4 (&b)[2], bf16_t) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const uint32_t sel = c ? 0x07060302u : 0x05040100u;
    b[c] = uint4{__builtin_amdgcn_perm(r[1], r[0], sel), __builtin_amdgcn_perm(r[3], r[2], sel), __builtin_amdgcn_perm(r[5], r[4], sel),
                 __builtin_amdgcn_perm(r[7], r[6], sel)};
  }
}
__device__ __forceinline__ void split_parity(const uint32_t (&r)[8], uint4 (&b)[2], float) {
  b[0] = uint4{r[0], r[2], r[4], r[6]};
  b[1] = uint4{r[1], r[3], r[5], r[7]};
}

template <typename T, int MRB, int VP>
__global__ void __launch_bounds__(256, MRB == 8 ? 2 : MRB == 4 ? 3 : 4) deconv_bf_flat_kernel(const T* __restrict__ x, const T* __restrict__ dy, float* __restrict__ part,
                                                               DbfArgs a) {
  constexpr int CI_WG = 16 * MRB, ES = sizeof(T), VU = Unit<T>::N, NP = VU / VP;      // NP pieces of dy a unit
  constexpr int PD = VP * 2 * ES / 4;                                                 // dwords of a piece: 1, 2 or 4
  constexpr int XBUF = CI_WG * DB_PITCH;
  constexpr int XU = 4 * DB_RU, XC = 256 / XU, NX = CI_WG / XC;                       // a thread stages NX units of x, XC channels apart
  extern __shared__ uint4 lds[];      // [2 buffers][CI_WG][DB_PITCH]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lg = lane >> 4, lc = lane & 15;
  const int groups = a.gco * a.gci;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int grp = slot % groups, chunk = (slot / groups) * 8 + xcd;
  if (chunk >= a.nchunks) return;                         // the grid is padded to a multiple of 8 chunks
  const int co = (grp % a.gco) * 16 + lc, ci0 = (grp / a.gco) * CI_WG;
  const int ta = wave >> 1, tb = wave & 1;
  const int W = a.x.w, plane = (int)a.x.plane, Dc = a.x.d;
  constexpr bool TAIL = PD < 4;      // a plane may end within a unit of x

  const int xu = tid % XU, xc = ci0 + tid / XU;           // this thread's unit, and the first of its channels
  auto load_x = [&](int n, int d, int p0, int lim, uint4 (&dst)[NX]) {
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(x + n * a.x.nstride, (uint32_t)a.xspan * ES);
    const int v0 = p0 + xu * VU, o0 = (d + a.x.hlo) * plane + v0;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int c = xc + XC * i, o = min(o0 + c * (int)a.x.cstride, a.xspan - VU);
      dst[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, ES * o | (v0 < lim && c < a.cin ? 0 : ROW_OOB), 0, 0));
    }
  };
  auto store_x = [&](int d, int p0, const uint4 (&src)[NX], int buf) {
    uint4* dst = lds + buf * XBUF + tid / XU * DB_PITCH + xu;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      uint4 v = src[i];
      if constexpr (TAIL) {
        const int o = (d + a.x.hlo) * plane + p0 + xu * VU + (xc + XC * i) * (int)a.x.cstride;
        v = Unit<T>::fix(v, max(0, o - (a.xspan - VU)), plane - p0 - xu * VU);
      }
      dst[i * XC * DB_PITCH] = v;
    }
  };
  auto load_y = [&](int n, int d, int p0, int lim, uint32_t (&dst)[DB_RU][8]) {
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(dy + n * a.y.nstride, (uint32_t)a.yspan * ES);
    const int base = co * (int)a.y.cstride + (2 * d + ta + a.y.hlo) * (int)a.y.plane + 2 * W * tb;
#pragma unroll
    for (int r = 0; r < DB_RU; ++r)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int v = p0 + (4 * r + lg) * VU + q * VP;
        const int h = (int)(__umulhi((uint32_t)v, a.magic) >> a.shift);
        const int off = ES * (base + 2 * (v + W * h)) | (v < lim && co < a.cout ? 0 : ROW_OOB);
        if constexpr (PD == 4) {
          const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[r][4 * q + e] = t[e];
        } else if constexpr (PD == 2) {
          const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
          dst[r][2 * q] = t[0];
          dst[r][2 * q + 1] = t[1];
        } else {
          dst[r][q] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
        }
      }
  };

  f32x4 acc[MRB][2];
  float accdb[2] = {0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int rb = 0; rb < MRB; ++rb) acc[rb][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t one = ES == 2 ? 0x3f803f80u : 0x3f800000u;
  const uint4 ones = {one, one, one, one};
  const bool do_db = ci0 == 0;

  const int t0 = chunk * a.tiles_per_chunk, t1 = min(t0 + a.tiles_per_chunk, a.ntiles);
  constexpr int TV = 4 * DB_RU * VU;
  int pt = t0 % a.tiles_p, d = t0 / a.tiles_p % Dc, n = t0 / a.tiles_p / Dc;
  uint4 xr[NX];
  uint32_t ya[DB_RU][8], yb[DB_RU][8];
  int buf = 0;
  // the loads behind the last tile are made with nothing in range: where a branch around loads ends, the compiler waits for all of them
  auto step = [&](int tile, const uint32_t (&cur)[DB_RU][8], uint32_t (&nxt)[DB_RU][8]) {
    const int lim = tile + 1 < t1 ? plane : 0;
    pt = tile + 1 < t1 ? pt + 1 : pt;
    if (pt == a.tiles_p) {
      pt = 0;
      if (++d == Dc) { d = 0; ++n; }
    }
    load_x(n, d, pt * TV, lim, xr);
    load_y(n, d, pt * TV, lim, nxt);
    __builtin_amdgcn_sched_barrier(0);
    uint4 B[DB_RU][2];
#pragma unroll
    for (int r = 0; r < DB_RU; ++r) split_parity(cur[r], B[r], T());
    if (do_db) {
      f32x4 t[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int r = 0; r < DB_RU; ++r) unit_products(ones, B[r], t, T());
#pragma unroll
      for (int c = 0; c < 2; ++c) accdb[c] += t[c][0];
    }
    const uint4* ap = lds + buf * XBUF + lc * DB_PITCH + lg;
    uint4 A[2][DB_RU];
#pragma unroll
    for (int r = 0; r < DB_RU; ++r) A[0][r] = ap[4 * r];
#pragma unroll
    for (int rb = 0; rb < MRB; ++rb) {
      // (one row block ahead and no further: the fragments of all at once spill registers)
      if (rb + 1 < MRB)
#pragma unroll
        for (int r = 0; r < DB_RU; ++r) A[(rb + 1) & 1][r] = ap[(rb + 1) * 16 * DB_PITCH + 4 * r];
      f32x4 t[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int r = 0; r < DB_RU; ++r) unit_products(A[rb & 1][r], B[r], t, T());
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[rb][c] += t[c];
      __builtin_amdgcn_sched_barrier(0);
    }
    store_x(d, pt * TV, xr, buf ^ 1);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    buf ^= 1;
  };
  load_x(n, d, pt * TV, plane, xr);
  load_y(n, d, pt * TV, plane, ya);
  store_x(d, pt * TV, xr, 0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  for (int tile = t0; tile < t1; tile += 2) {       // (behind an odd number of tiles a step of zeros: a second exit would be such a branch too)
    step(tile, ya, yb);
    step(tile + 1, yb, ya);
  }

  // ---- partial sums -> workspace [chunk][cin][cout][8] (+ [chunk][cout][8] for the bias partials behind them)
  if (co < a.cout) {
    float* pw = part + (int64_t)chunk * a.cin * a.cout * 8;
#pragma unroll
    for (int rb = 0; rb < MRB; ++rb)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int ci = ci0 + rb * 16 + 4 * lg + rr;
        if (ci < a.cin) *reinterpret_cast<float2*>(pw + ((int64_t)ci * a.cout + co) * 8 + 2 * wave) = float2{acc[rb][0][rr], acc[rb][1][rr]};
      }
    if (do_db && lg == 0) {
      float* pb = part + (int64_t)a.nchunks * a.cin * a.cout * 8 + (int64_t)chunk * a.cout * 8;
      *reinterpret_cast<float2*>(pb + co * 8 + 2 * wave) = float2{accdb[0], accdb[1]};
    }
  }
}

// dw[i] = sum over chunks of part[chunk][i]; db[co] = sum over chunks and the 8 taps of the bias partials behind them.  Fixed order: each of
// a block's 16 thread groups adds every 16th chunk in increasing order, then the group sums are added in group order.  A thread takes four
// neighbouring outputs.
__global__ void __launch_bounds__(256) deconv_bf_flat_reduce_kernel(const float* __restrict__ part, float* __restrict__ dw, float* __restrict__ db,
                                                                   int64_t nw, int cout, int nchunks) {
  constexpr int G = 16;
  __shared__ float4 red[G][16];
  const int o = threadIdx.x & 15, cg = threadIdx.x >> 4;
  const int64_t wblocks = (nw + 63) / 64;
  const bool bias = blockIdx.x >= wblocks;                              // blocks behind the weights: 8 channels each, two threads a channel
  const int64_t i = bias ? ((blockIdx.x - wblocks) * 16 + o) * 4 : ((int64_t)blockIdx.x * 16 + o) * 4;
  const int64_t len = bias ? (int64_t)cout * 8 : nw;
  const float* base = part + (bias ? (int64_t)nchunks * nw : 0) + i;
  float4 s = {0.f, 0.f, 0.f, 0.f};
  if (i < len) {
    int c = cg;
    for (; c + 3 * G < nchunks; c += 4 * G) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(base + (c + u * G) * len);
#pragma unroll
      for (int u = 0; u < 4; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
    for (; c < nchunks; c += G) {
      const float4 v = *reinterpret_cast<const float4*>(base + c * len);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  red[cg][o] = s;
  __syncthreads();
  if (cg != 0 || i >= len) return;
  float4 r = red[0][o];
#pragma unroll
  for (int k = 1; k < G; ++k) { r.x += red[k][o].x; r.y += red[k][o].y; r.z += red[k][o].z; r.w += red[k][o].w; }
  if (!bias) {
    // dw may start at any 4-byte address
    dw[i] = r.x; dw[i + 1] = r.y; dw[i + 2] = r.z; dw[i + 3] = r.w;
  } else {
    const float half = (r.x + r.y) + (r.z + r.w);
    const float other = __shfl_xor(half, 1, 64);
    if (db && (o & 1) == 0) db[i / 8] = half + other;
  }
}

__global__ void deconv_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

struct DbfPlan {
  int ci_wg, tiles_p, ntiles, tiles_per_chunk, nchunks, gco, gci;
};

DbfPlan dbf_plan(const h3d_tensor* x, const h3d_tensor* dy) {
  DbfPlan p;
  p.ci_wg = x->c > 64 ? 128 : (x->c > 32 ? 64 : 32);
  p.tiles_p = (int)cdiv((int64_t)x->h * x->w, 4 * DB_RU * (x->dtype == H3D_F32 ? 4 : 8));
  p.ntiles = (int)((int64_t)x->n * x->d * p.tiles_p);
  p.gco = (int)cdiv(dy->c, 16);
  p.gci = (int)cdiv(x->c, p.ci_wg);
  // one round of resident workgroups (two a CU), as long as the partial sums stay a small part of the traffic
  const int64_t per_chunk_bytes = std::max<int64_t>(1, ((int64_t)x->c * dy->c + dy->c) * 8 * 4);
  int64_t want = std::max<int64_t>(1, (p.ci_wg == 128 ? 512 : 768) / ((int64_t)p.gco * p.gci));
  want = std::min<int64_t>(want, std::max<int64_t>(1, ((int64_t)64 << 20) / per_chunk_bytes));
  // bf16: .. and no chunks of less than four tiles, six where that still gives every CU a workgroup: their sums cost more than the products, and push
  // the operands of the calls behind out of the cache.  us of all three passes, from one tile on, four and six: 96 -> 64 channels from 64x16x16 52.7, 47.0
  // and 47.9, 128 -> 64 from 8x16x16 42.8, 40.5 and 44.3, 64 -> 24 from 32x112x32 59.1, 59.0 and 54.6, 53 -> 128 from 2 x 16x18x32, three sets of
  // tensors in turn, 91.7, 94.0 and 86.3.  (fp32 tiles are half as long and four times the work: 32 -> 32 from 8x16x16 48.8, 49.7 and 53.6)
  if (x->dtype == H3D_BF16) {
    const int64_t least = p.ntiles / 6 * (int64_t)(p.gco * p.gci) >= 256 ? 6 : 4;
    want = std::min<int64_t>(want, std::max<int64_t>(1, p.ntiles / least));
  }
  p.tiles_per_chunk = (int)std::max<int64_t>(1, cdiv(p.ntiles, want));
  // the kernel takes two tiles a turn: an odd number from three on costs as much as the next even one
  if (p.tiles_per_chunk > 2) p.tiles_per_chunk += p.tiles_per_chunk & 1;
  p.nchunks = (int)std::max<int64_t>(1, cdiv(p.ntiles, p.tiles_per_chunk));
  return p;
}

template <typename T, int MRB, int VP>
h3d_status dbf_launch(void* handle, const h3d_tensor* x, const h3d_tensor* dy, float* part, const DbfArgs& a, hipStream_t stream) {
  constexpr size_t lds_bytes = (size_t)2 * 16 * MRB * DB_PITCH * 16;
  static bool done = false;
  H3D_TRY(raise_lds_limit(handle, deconv_bf_flat_kernel<T, MRB, VP>, lds_bytes, &done));
  const int64_t grid = cdiv(a.nchunks, 8) * 8 * (int64_t)(a.gco * a.gci);
  if (grid >= ((int64_t)1 << 31)) return fail(handle, H3D_EINVAL, "deconv2_bwd_filter: too many workgroups");
  hipLaunchKernelGGL((deconv_bf_flat_kernel<T, MRB, VP>), dim3((unsigned)grid), dim3(256), lds_bytes, stream, (const T*)x->data,
                     (const T*)dy->data, part, a);
  note_kernel(handle, "deconv_bf_flat_kernel<%s,%d,%d>", sizeof(T) == 4 ? "f32" : "bf16", 16 * MRB, VP);
  return H3D_OK;
}
template <typename T, int VP>
h3d_status dbf_ci(void* handle, const h3d_tensor* x, const h3d_tensor* dy, float* part, const DbfArgs& a, int ci_wg, hipStream_t stream) {
  if (ci_wg == 128) return dbf_launch<T, 8, VP>(handle, x, dy, part, a, stream);
  if (ci_wg == 64) return dbf_launch<T, 4, VP>(handle, x, dy, part, a, stream);
  return dbf_launch<T, 2, VP>(handle, x, dy, part, a, stream);
}

}  // namespace

// everything whose sample 32-bit byte offsets reach; a sample has to hold one 16-byte unit, a row two voxels.  The direct kernel takes the rest.
bool deconv_bf_flat_supported(const h3d_tensor* x, const h3d_tensor* dy) {
  if (x->c < 1 || dy->c < 1 || x->w < 2) return false;
  const int64_t es = elt_size(x->dtype), xs = stored_span(make_geo(x)), ys = stored_span(make_geo(dy));
  const int64_t ntiles = (int64_t)x->n * x->d * cdiv((int64_t)x->h * x->w, 32);
  return xs * es >= 16 && xs * es < ((int64_t)1 << 31) && ys * es < ((int64_t)1 << 31) && ntiles < ((int64_t)1 << 30) &&
         cdiv(dy->c, 16) * cdiv(x->c, 32) < 65536;
}

size_t deconv_bf_flat_ws_bytes(const h3d_tensor* x, const h3d_tensor* dy) {
  return (size_t)dbf_plan(x, dy).nchunks * ((size_t)x->c * dy->c + dy->c) * 8 * sizeof(float);
}

h3d_status deconv_bf_flat(void* handle, const h3d_tensor* x, const h3d_tensor* dy, float* dw, float* db, void* ws, size_t ws_bytes,
                          hipStream_t stream) {
  const DbfPlan p = dbf_plan(x, dy);
  if (!ws || ws_bytes < deconv_bf_flat_ws_bytes(x, dy) || (uintptr_t)ws % 16)
    return fail(handle, H3D_EWORKSPACE, "deconv2_bwd_filter: workspace too small or misaligned");
  DbfArgs a;
  a.x = make_geo(x); a.y = make_geo(dy);
  a.cin = x->c; a.cout = dy->c;
  a.tiles_p = p.tiles_p; a.ntiles = p.ntiles; a.tiles_per_chunk = p.tiles_per_chunk; a.nchunks = p.nchunks;
  a.gco = p.gco; a.gci = p.gci;
  a.xspan = (int)stored_span(a.x); a.yspan = (int)stored_span(a.y);
  const int64_t nw = (int64_t)a.cin * a.cout * 8;
  if (p.ntiles == 0) {
    // a fill kernel, not a memset: the call may be recorded into a graph by the caller
    hipLaunchKernelGGL(deconv_zero_kernel, dim3((unsigned)cdiv(nw, 256)), dim3(256), 0, stream, dw, nw);
    if (db) hipLaunchKernelGGL(deconv_zero_kernel, dim3((unsigned)cdiv(a.cout, 256)), dim3(256), 0, stream, db, (int64_t)a.cout);
    return launch_status(handle, "deconv2_bwd_filter");
  }
  // floor(v / W) for v < 2^31: magic = ceil(2^(31 + l) / W), 2^l >= W, is off by less than W / 2^(31 + l) <= 2^-31 a voxel
  int l = 1;
  while (((int64_t)1 << l) < a.x.w) ++l;
  a.magic = (uint32_t)((((uint64_t)1 << (31 + l)) + a.x.w - 1) / a.x.w);
  a.shift = l - 1;
  const int w = a.x.w;
  const bool whole = a.x.plane % (x->dtype == H3D_F32 ? 4 : 8) == 0;      // whole units of x in a plane
  float* part = (float*)ws;
  if (x->dtype == H3D_F32) {
    if (w % 2 == 0 && whole) H3D_TRY((dbf_ci<float, 2>(handle, x, dy, part, a, p.ci_wg, stream)));
    else H3D_TRY((dbf_ci<float, 1>(handle, x, dy, part, a, p.ci_wg, stream)));
  } else {
    if (w % 4 == 0 && whole) H3D_TRY((dbf_ci<bf16_t, 4>(handle, x, dy, part, a, p.ci_wg, stream)));
    else if (w % 2 == 0) H3D_TRY((dbf_ci<bf16_t, 2>(handle, x, dy, part, a, p.ci_wg, stream)));
    else H3D_TRY((dbf_ci<bf16_t, 1>(handle, x, dy, part, a, p.ci_wg, stream)));
  }
  hipLaunchKernelGGL(deconv_bf_flat_reduce_kernel, dim3((unsigned)(cdiv(nw, 64) + cdiv(a.cout, 8))), dim3(256), 0, stream, (const float*)part, dw,
                     db, nw, a.cout, a.nchunks);
  return launch_status(handle, "deconv2_bwd_filter");
}

}  // namespace h3d
