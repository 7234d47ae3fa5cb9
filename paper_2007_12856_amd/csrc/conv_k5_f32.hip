// 5x5x5 convolution passes of fp32 tensors on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums).  2 * 125 * cin * cout flop a
// voxel: far right of the fp32 ridge, so what bounds all three is the product rate (157 TFLOP/s published), and, in volumes of few tiles, how
// much of the chip they occupy.
//  * forward / backward-data (one kernel; backward-data: the filter reversed and transposed by the pack kernel, g = dz * act'(z) made while
//    staging): rows = 16 voxels, columns = 16 result channels, K = 4 contraction channels of one tap.  A workgroup of four wavefronts owns 4
//    planes x TR rows x 16 HV columns x 16 CB channels, a wavefront one plane.  Per group of 4 channels the tile with its halo is staged (8
//    planes, zeros outside the volume); per (kd, kw) its TR + 4 rows are read once for the five kh.  Weights go from the packed copy (fragment
//    order, L2) straight into registers, one (kd, kw) ahead: in LDS they would need a buffer and a barrier for each kd.  Two workgroups a CU
//    stage and multiply in turn.  Volumes of few tiles: 2-row tiles, and the channel groups split over workgroups whose sums a second kernel
//    adds in order.
//  * backward-filter: rows = 16 input channels, columns = 16 output channels, K = voxels of a row (in the order of conv_f32_mfma.hip: a lane
//    group holds consecutive columns, so that a few wide LDS reads feed 5 products a voxel).  A workgroup owns a 16 x 16 block of one kd and a
//    chunk of tiles; 25 accumulator tiles and one for db; next tile's loads in flight, two LDS buffers, one barrier a tile.
// us of the three masked passes, on the vector ALU and here: 128 -> 32 on 54x16x12 4137 and 560, 32 -> 96 on 48x32x16 3955 and 774, 64 -> 24 on
// 38x58x32 3008 and 1272, 24 -> 64 on 2 x 16x32x10 2228 and 298.
#include <algorithm>

#include "rowload.h"
#include "taps.h"

namespace h3d {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// (the range check looks at voff alone)
__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t rs, int voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, (int)__builtin_amdgcn_readfirstlane(soff), 0));
}
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

struct K5FArgs {
  Geo in, mask, out;
  int cin, cout, ncig;       // contraction / result channels, groups of 4 contraction channels
  int pmin, pmax;            // planes of `in` that are read
  int npg, nhg, nwg;         // plane, row and column groups
  int per_split;             // channel groups of a split
  int64_t split_elems;       // elements of one split's sums (0: not split)
  float slope_in, slope_out;
  int vec;                   // 16-byte stores allowed
};

// wk: [result group][channel group][kd][kw][kh][block of 16 results][lane]: lane l = channel l / 16 of the group, result l % 16
__global__ void __launch_bounds__(256) k5f_pack_kernel(const float* __restrict__ w, float* __restrict__ wk, int cin, int cout, int transposed, int ncig,
                                                      int cb, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  int64_t r = i >> 6;
  const int lane = (int)(i & 63), b = (int)(r % cb); r /= cb;
  const int kh = (int)(r % 5); r /= 5;
  const int kw = (int)(r % 5); r /= 5;
  const int kd = (int)(r % 5); r /= 5;
  const int cig = (int)(r % ncig), cog = (int)(r / ncig);
  const int res = (cog * cb + b) * 16 + (lane & 15), c = cig * 4 + (lane >> 4), t = kd * 25 + kh * 5 + kw;
  const int co = transposed ? c : res, ci = transposed ? res : c;
  wk[i] = co < cout && ci < cin ? w[((int64_t)co * cin + ci) * 125 + (transposed ? 124 - t : t)] : 0.f;
}

template <int CB, int TR, int HV, bool MASKED>
__global__ void __launch_bounds__(256, 2) k5f_conv_kernel(const float* __restrict__ in, const float* __restrict__ mask, const float* __restrict__ wk,
                                                         const float* __restrict__ bias, float* __restrict__ out, float* __restrict__ part, K5FArgs a) {
  constexpr int XR = TR + 4, XC = 16 * HV + 4, XPL = XR * XC, SP = 8 * XPL, PT = (SP + 255) / 256;      // staged voxels of a channel
  constexpr int CS = (SP + 63) / 64 * 64 + 16;      // channel pitch: the four channels of a fragment read meet four bank groups
  extern __shared__ float lds[];                    // [4 channels][CS]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = a.out.w, H = a.out.h;
  int t = blockIdx.x;
  const int w0 = t % a.nwg * 16 * HV; t /= a.nwg;
  const int h0 = t % a.nhg * TR; t /= a.nhg;
  const int p0 = t % a.npg * 4, n = t / a.npg, cog = blockIdx.y;

  int xoff[PT], moff[MASKED ? PT : 1];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int s = tid + 256 * i, col = s % XC, row = s / XC % XR, q = p0 - 2 + s / XPL;
    const int hh = h0 - 2 + row, ww = w0 - 2 + col;
    const bool ok = s < SP && q >= a.pmin && q < a.pmax && hh >= 0 && hh < H && ww >= 0 && ww < W;
    xoff[i] = ok ? 4 * (int)((q + a.in.hlo) * a.in.plane + (int64_t)hh * W + ww) : ROW_OOB;
    if (MASKED) moff[i] = ok ? 4 * (int)((q + a.mask.hlo) * a.mask.plane + (int64_t)hh * W + ww) : ROW_OOB;
  }
  const int p = p0 + wave;
  const bool live = p < a.out.d;

  f32x4 acc[CB][TR][HV];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int co = (cog * CB + cb) * 16 + (lane & 15);
    const float b = bias && !a.split_elems && co < a.cout ? bias[co] : 0.f;
#pragma unroll
    for (int r = 0; r < TR; ++r)
#pragma unroll
      for (int hf = 0; hf < HV; ++hf) acc[cb][r][hf] = f32x4{b, b, b, b};
  }
  const __amdgpu_buffer_rsrc_t rs_in = row_rsrc(in + (int64_t)n * a.in.nstride, (uint32_t)(a.in.nstride * 4));
  const __amdgpu_buffer_rsrc_t rs_mk = row_rsrc(MASKED ? mask + (int64_t)n * a.mask.nstride : in, (uint32_t)(a.mask.nstride * 4));
  const float* xw = lds + (lane >> 4) * CS + wave * XPL + (lane & 15);

  const int cig1 = min(a.ncig, (int)(blockIdx.z + 1) * a.per_split);
  for (int cig = blockIdx.z * a.per_split; cig < cig1; ++cig) {
    const float* wp = wk + ((int64_t)cog * a.ncig + cig) * (125 * CB * 64) + lane;
    float wc[5][CB], wn[5][CB];
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) wc[k][cb] = wp[(k * CB + cb) * 64];
    __syncthreads();                                       // everyone is done with the previous group's tile
#pragma unroll
    for (int c2 = 0; c2 < 4; c2 += 2) {
      float v[2][PT], m[2][MASKED ? PT : 1];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int ci = cig * 4 + c2 + c;
        const bool ok = ci < a.cin;                        // uniform
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          v[c][i] = buf_load(rs_in, ok ? xoff[i] : ROW_OOB, 4u * ci * (uint32_t)a.in.cstride);
          if (MASKED) m[c][i] = buf_load(rs_mk, ok ? moff[i] : ROW_OOB, 4u * ci * (uint32_t)a.mask.cstride);
        }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          float x = v[c][i];
          if (MASKED) x = m[c][i] > 0.f ? x : x * a.slope_in;
          if (SP % 256 == 0 || tid + 256 * i < SP) lds[(c2 + c) * CS + tid + 256 * i] = x;
        }
    }
    __syncthreads();
    if (!live) continue;
#pragma unroll 1
    for (int kd = 0; kd < 5; ++kd) {
#pragma unroll
      for (int kw = 0; kw < 5; ++kw) {
        const int next = min(kd * 5 + kw + 1, 24);         // the weights of the next (kd, kw)
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) wn[k][cb] = wp[((next * 5 + k) * CB + cb) * 64];
        float bx[XR][HV];
#pragma unroll
        for (int r = 0; r < XR; ++r)
#pragma unroll
          for (int hf = 0; hf < HV; ++hf) bx[r][hf] = xw[kd * XPL + r * XC + hf * 16 + kw];
#pragma unroll
        for (int kh = 0; kh < 5; ++kh)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
              for (int hf = 0; hf < HV; ++hf) acc[cb][r][hf] = mfma4(bx[r + kh][hf], wc[kh][cb], acc[cb][r][hf]);
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) wc[k][cb] = wn[k][cb];
      }
    }
  }

  if (!live) return;
  const bool split = a.split_elems != 0;
  const int64_t plane = (int64_t)H * W;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int co = (cog * CB + cb) * 16 + (lane & 15);
    if (co >= a.cout) continue;
    float* dst = split ? part + blockIdx.z * a.split_elems + (((int64_t)n * a.cout + co) * a.out.d + p) * plane
                       : out + (int64_t)n * a.out.nstride + (int64_t)co * a.out.cstride + (int64_t)(p + a.out.hlo) * plane;
#pragma unroll
    for (int r = 0; r < TR; ++r) {
      const int h = h0 + r;
      if (h >= H) continue;
#pragma unroll
      for (int hf = 0; hf < HV; ++hf) {
        const int wc = w0 + hf * 16 + 4 * (lane >> 4);
        if (wc >= W) continue;
        f32x4 o = acc[cb][r][hf];
        if (!split)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (!(o[j] > 0.f)) o[j] *= a.slope_out;
        float* q = dst + (int64_t)h * W + wc;
        if (a.vec && wc + 3 < W) {
          *reinterpret_cast<f32x4*>(q) = o;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (wc + j < W) q[j] = o[j];
        }
      }
    }
  }
}

// out = activation(bias + the splits' sums in order)
__global__ void __launch_bounds__(256) k5f_split_kernel(const float* __restrict__ part, const float* __restrict__ bias, float* __restrict__ out, K5FArgs a,
                                                       int nsplit) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.split_elems) return;
  const int64_t v = i % a.out.plane, r = i / a.out.plane;
  const int p = (int)(r % a.out.d), co = (int)(r / a.out.d % a.cout), n = (int)(r / a.out.d / a.cout);
  float s = bias ? bias[co] : 0.f;
  for (int k = 0; k < nsplit; ++k) s += part[k * a.split_elems + i];
  out[n * a.out.nstride + co * a.out.cstride + (p + a.out.hlo) * a.out.plane + v] = s > 0.f ? s : s * a.slope_out;
}

// ------------------------------------------------------------------------------------------------ backward-filter
struct K5FBfArgs {
  Geo x, g, z;
  int cin, cout, pmin, pmax;
  int nhg, nwg, cip, cop;
  int64_t tiles;            // n * d * nhg * nwg
  int tiles_per_chunk;
  float slope;
};
constexpr int BG_CS = 128 + 4;      // channel pitch of g (4 mod 32 floats: the 8 lanes of a 16-byte read's phase meet 8 bank groups)
constexpr int bx_floats(bool narrow) { return narrow ? 12 * 20 : 8 * 36; }      // a channel of the x window: (rows + 4) x (columns + 4)

// tile: 4 rows x 32 columns of one plane, a row a wavefront; NARROW (at most 16 columns): 8 rows x 16, two rows a wavefront
template <bool MASKED, bool NARROW>
__global__ void __launch_bounds__(256, 2) k5f_bwf_kernel(const float* __restrict__ x, const float* __restrict__ dz, const float* __restrict__ z,
                                                        float* __restrict__ part, float* __restrict__ part_db, K5FBfArgs a) {
  constexpr int BW = NARROW ? 16 : 32, BR = NARROW ? 8 : 4, RW = BR / 4, CPL = BW / 4, XC = BW + 4, XF = bx_floats(NARROW), XS = 2 * XF + 4;
  static_assert(XS % 32 == 4 && 16 * XS >= 26 * 256, "LDS layout of x");
  extern __shared__ __attribute__((aligned(16))) float lds[];      // x: [16 channels][2 buffers][rows][XC] (+ 4), then g: [2 buffers][16][BG_CS]
  float* lds_g = lds + 16 * XS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = blockIdx.x, cog = blockIdx.y, cig = blockIdx.z / 5, kd = blockIdx.z % 5;
  const int W = a.x.w, H = a.x.h, D = a.x.d;
  const bool do_db = kd == 2 && cig == 0;
  f32x4 acc[26];
#pragma unroll
  for (int t = 0; t < 26; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this thread's part of the staging: one voxel of 16 channels of x (wide tiles: and two voxels of the last four columns), one voxel of 8
  // channels of g
  const int xrow = NARROW ? tid / XC : tid >> 5, xcol = NARROW ? tid % XC : tid & 31;
  const bool xmine = !NARROW || tid < 12 * XC;
  const int gs = tid & 127, gc0 = (tid >> 7) * 8;
  const int nci = min(16, a.cin - cig * 16), nco = min(16, a.cout - cog * 16);
  float xv[16], xe[2], gv[8], zv[8];
  auto load_tile = [&](int64_t tile, bool ok) {
    int64_t r = tile;
    const int w0 = (int)(r % a.nwg) * BW; r /= a.nwg;
    const int h0 = (int)(r % a.nhg) * BR; r /= a.nhg;
    const int p = (int)(r % D), n = (int)(r / D), q = p + kd - 2;
    const __amdgpu_buffer_rsrc_t rs_x = row_rsrc(x + (int64_t)n * a.x.nstride, (uint32_t)(a.x.nstride * 4));
    const __amdgpu_buffer_rsrc_t rs_g = row_rsrc(dz + (int64_t)n * a.g.nstride, (uint32_t)(a.g.nstride * 4));
    const __amdgpu_buffer_rsrc_t rs_z = row_rsrc(MASKED ? z + (int64_t)n * a.z.nstride : dz, (uint32_t)(a.z.nstride * 4));
    const bool pok = ok && q >= a.pmin && q < a.pmax;
    const uint32_t xp = (uint32_t)max(q + a.x.hlo, 0) * (uint32_t)a.x.plane;
    auto offset = [&](int row, int col) {
      const int hh = h0 - 2 + row, ww = w0 - 2 + col;
      return pok && hh >= 0 && hh < H && ww >= 0 && ww < W ? 4 * (hh * W + ww) : ROW_OOB;
    };
    const int vo = xmine ? offset(xrow, xcol) : ROW_OOB;
#pragma unroll
    for (int c = 0; c < 16; ++c) xv[c] = buf_load(rs_x, c < nci ? vo : ROW_OOB, 4u * ((cig * 16 + c) * (uint32_t)a.x.cstride + xp));
    if (!NARROW) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = (tid + 256 * j) >> 5, eo = offset((tid >> 2) & 7, 32 + (tid & 3));
        xe[j] = buf_load(rs_x, c < nci && eo != ROW_OOB ? eo + 4 * c * (int)a.x.cstride : ROW_OOB, 4u * (cig * 16 * (uint32_t)a.x.cstride + xp));
      }
    }
    const int hg = h0 + gs / BW, wg = w0 + gs % BW;
    const int go = ok && hg < H && wg < W ? 4 * (hg * W + wg) : ROW_OOB;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int off = gc0 + j < nco ? go : ROW_OOB;
      gv[j] = buf_load(rs_g, off == ROW_OOB ? ROW_OOB : off + 4 * gc0 * (int)a.g.cstride,
                       4u * ((cog * 16 + j) * (uint32_t)a.g.cstride + (p + a.g.hlo) * (uint32_t)a.g.plane));
      if (MASKED)      // 0 where g is 0
        zv[j] = buf_load(rs_z, off == ROW_OOB ? ROW_OOB : off + 4 * gc0 * (int)a.z.cstride,
                         4u * ((cog * 16 + j) * (uint32_t)a.z.cstride + (p + a.z.hlo) * (uint32_t)a.z.plane));
    }
  };
  auto store_tile = [&](int buf) {
    if (xmine) {
      float* d = lds + buf * XF + xrow * XC + xcol;
#pragma unroll
      for (int c = 0; c < 16; ++c) d[c * XS] = xv[c];
    }
    if (!NARROW)
#pragma unroll
      for (int j = 0; j < 2; ++j) lds[((tid + 256 * j) >> 5) * XS + buf * XF + ((tid >> 2) & 7) * XC + 32 + (tid & 3)] = xe[j];
    float* d = lds_g + buf * 16 * BG_CS + gc0 * BG_CS + gs;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float v = gv[j];
      if (MASKED && !(zv[j] > 0.f)) v *= a.slope;
      d[j * BG_CS] = v;
    }
  };

  const float* xr = lds + (lane & 15) * XS + wave * RW * XC + CPL * (lane >> 4);
  const float* gr = lds_g + (lane & 15) * BG_CS + wave * RW * BW + CPL * (lane >> 4);
  const int64_t t0 = (int64_t)chunk * a.tiles_per_chunk, t1 = min(t0 + a.tiles_per_chunk, a.tiles);
  load_tile(t0, t0 < t1);
  store_tile(0);
  __syncthreads();
  int buf = 0;
  for (int64_t tile = t0; tile < t1; ++tile, buf ^= 1) {
    load_tile(tile + 1, tile + 1 < t1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      float g[CPL], xf[2][CPL + 4];
      auto read_x = [&](int kh, float (&v)[CPL + 4]) {
#pragma unroll
        for (int k = 0; k < CPL + 4; k += 4) *reinterpret_cast<f32x4*>(v + k) = *reinterpret_cast<const f32x4*>(xr + buf * XF + (kh + rr) * XC + k);
      };
#pragma unroll
      for (int k = 0; k < CPL; k += 4) *reinterpret_cast<f32x4*>(g + k) = *reinterpret_cast<const f32x4*>(gr + buf * 16 * BG_CS + rr * BW + k);
      read_x(0, xf[0]);
#pragma unroll
      for (int kh = 0; kh < 5; ++kh) {
        if (kh < 4) read_x(kh + 1, xf[(kh + 1) & 1]);
        const float (&v)[CPL + 4] = xf[kh & 1];
#pragma unroll
        for (int j = 0; j < CPL; ++j)
#pragma unroll
          for (int kw = 0; kw < 5; ++kw) acc[kh * 5 + kw] = mfma4(v[j + kw], g[j], acc[kh * 5 + kw]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (do_db) {      // a row's sum by itself first: shorter chains (db of 600000 voxels 4.9e-7 from 64 bits in one chain, 1.6e-7 so)
        f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < CPL; ++j) t = mfma4(1.f, g[j], t);
        acc[25] += t;
      }
    }
    store_tile(buf ^ 1);
    __syncthreads();
  }

  // ---- the four wavefronts' sums, added in wavefront order through LDS (the x tile's space: 26 KB)
  for (int wv = 0; wv < 4; ++wv) {
    __syncthreads();
    if (wave == wv) {
#pragma unroll
      for (int t = 0; t < 26; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int idx = (t * 4 + j) * 64 + lane;
          if (wv == 0) lds[idx] = acc[t][j];
          else if (wv < 3) lds[idx] += acc[t][j];
          else acc[t][j] += lds[idx];
        }
    }
  }
  if (wave != 3) return;
  // lane holds input channels 4 (lane / 16) .. + 3 and output channel lane % 16 of every tap; channels the tensors do not have are padding
  const int co = cog * 16 + (lane & 15), ci = cig * 16 + 4 * (lane >> 4);
#pragma unroll
  for (int t = 0; t < 25; ++t)
    *reinterpret_cast<f32x4*>(part + (((int64_t)chunk * 125 + kd * 25 + t) * a.cop + co) * a.cip + ci) = acc[t];
  if (do_db && lane < 16) part_db[(int64_t)chunk * a.cop + co] = acc[25][0];
}

bool sample_fits(const h3d_tensor* t) { return sample_span(t) < ((int64_t)1 << 29); }      // 32-bit byte offsets

struct K5FPlan {
  int cb, tr, hv, npg, nhg, nwg, ncig, ncog, nsplit, per_split;
  int64_t tiles;
  size_t wk_bytes, part_bytes;
};
// cin_k / cout: contraction channels / the written tensor
K5FPlan k5f_plan(int cin_k, const h3d_tensor* out) {
  K5FPlan p;
  p.cb = out->c <= 16 ? 1 : 2;
  p.hv = out->w <= 16 ? 1 : 2;
  p.ncig = (int)cdiv(cin_k, 4);
  p.ncog = (int)cdiv(out->c, 16 * p.cb);
  p.npg = (int)cdiv(out->d, 4); p.nwg = (int)cdiv(out->w, 16 * p.hv);
  // 8-row tiles hold more products per staged row; with fewer than two of them per CU 2-row tiles occupy more CUs, then splits of at least two
  // channel groups do
  const int64_t tall = (int64_t)out->n * p.npg * cdiv(out->h, 8) * p.nwg * p.ncog;
  p.tr = tall < 512 ? 2 : 8;
  p.nhg = (int)cdiv(out->h, p.tr);
  p.tiles = (int64_t)out->n * p.npg * p.nhg * p.nwg;
  const int64_t wgs = std::max<int64_t>(1, p.tiles * p.ncog);
  p.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>({cdiv(512, wgs), (int64_t)p.ncig / 2, (int64_t)8}));
  p.per_split = (int)cdiv(p.ncig, p.nsplit);
  p.nsplit = (int)cdiv(p.ncig, p.per_split);
  p.wk_bytes = up256((size_t)p.ncog * p.ncig * 125 * p.cb * 64 * sizeof(float));
  p.part_bytes = p.nsplit > 1 ? up256((size_t)p.nsplit * out->n * out->c * out->d * out->h * out->w * sizeof(float)) : 0;
  return p;
}

template <int CB, int TR, int HV, bool MASKED>
h3d_status k5f_launch(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const float* wk, const float* bias, h3d_tensor* out, float* part,
                      const K5FArgs& a, const K5FPlan& p, hipStream_t s) {
  constexpr size_t lds = (size_t)4 * ((8 * (TR + 4) * (16 * HV + 4) + 63) / 64 * 64 + 16) * sizeof(float);
  static bool done = false;
  H3D_TRY(raise_lds_limit(handle, k5f_conv_kernel<CB, TR, HV, MASKED>, lds, &done));
  hipLaunchKernelGGL((k5f_conv_kernel<CB, TR, HV, MASKED>), dim3((unsigned)p.tiles, (unsigned)p.ncog, (unsigned)p.nsplit), dim3(256), lds, s,
                     (const float*)in->data, (const float*)(mask ? mask->data : nullptr), wk, bias, (float*)out->data, part, a);
  note_kernel(handle, "k5f_conv_kernel<%d,%d,%d>", CB, TR, HV);
  return H3D_OK;
}
template <int CB, int TR, int HV>
h3d_status k5f_launch_m(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const float* wk, const float* bias, h3d_tensor* out, float* part,
                        const K5FArgs& a, const K5FPlan& p, hipStream_t s) {
  return mask ? k5f_launch<CB, TR, HV, true>(handle, in, mask, wk, bias, out, part, a, p, s)
              : k5f_launch<CB, TR, HV, false>(handle, in, mask, wk, bias, out, part, a, p, s);
}

struct K5FBfPlan {
  int nhg, nwg, cigs, cogs, tiles_per_chunk, nchunks;
  int64_t tiles;
  size_t part_bytes, db_bytes;
};
K5FBfPlan k5f_bf_plan(const h3d_tensor* x, int cout) {
  K5FBfPlan p;
  const bool narrow = x->w <= 16;
  p.nhg = (int)std::max<int64_t>(1, cdiv(x->h, narrow ? 8 : 4)); p.nwg = (int)std::max<int64_t>(1, cdiv(x->w, narrow ? 16 : 32));
  p.tiles = (int64_t)x->n * x->d * cdiv(x->h, narrow ? 8 : 4) * cdiv(x->w, narrow ? 16 : 32);
  p.cigs = (int)cdiv(x->c, 16); p.cogs = (int)cdiv(cout, 16);
  const int64_t blocks = 5 * (int64_t)p.cigs * p.cogs, per_chunk = (int64_t)p.cigs * p.cogs * 256 * 125 * 4;
  int64_t want = std::max<int64_t>(1, cdiv(1024, blocks));      // two rounds of resident workgroups
  want = std::min<int64_t>(want, std::max<int64_t>(1, ((int64_t)64 << 20) / per_chunk));
  want = std::min<int64_t>(want, std::max<int64_t>(p.tiles, 1));
  p.tiles_per_chunk = (int)std::max<int64_t>(1, cdiv(p.tiles, want));
  p.nchunks = (int)std::max<int64_t>(1, cdiv(p.tiles, p.tiles_per_chunk));
  p.part_bytes = up256((size_t)p.nchunks * per_chunk);
  p.db_bytes = up256((size_t)p.nchunks * p.cogs * 16 * sizeof(float));
  return p;
}

template <bool MASKED, bool NARROW>
h3d_status k5f_bf_launch(void* handle, const h3d_tensor* x, const h3d_tensor* dz, const h3d_tensor* z, float* part, float* part_db, const K5FBfArgs& a,
                         const K5FBfPlan& p, hipStream_t s) {
  constexpr size_t lds = (size_t)(16 * (2 * bx_floats(NARROW) + 4) + 2 * 16 * BG_CS) * sizeof(float);
  static bool done = false;
  H3D_TRY(raise_lds_limit(handle, k5f_bwf_kernel<MASKED, NARROW>, lds, &done));
  hipLaunchKernelGGL((k5f_bwf_kernel<MASKED, NARROW>), dim3((unsigned)p.nchunks, (unsigned)p.cogs, (unsigned)(5 * p.cigs)), dim3(256), lds, s,
                     (const float*)x->data, (const float*)dz->data, (const float*)(z ? z->data : nullptr), part, part_db, a);
  return H3D_OK;
}

}  // namespace

// in / out: the staged and the written tensor (backward-filter: x and dz).  Samples within 32-bit byte offsets; the vector-ALU kernels of
// conv_k5.hip take the others.
bool k5f_supported(const h3d_tensor* in, const h3d_tensor* out) {
  return in->dtype == H3D_F32 && in->c >= 1 && out->c >= 1 && in->c <= 65536 && out->c <= 65536 && sample_fits(in) && sample_fits(out) &&
         (int64_t)in->n * cdiv(in->d, 4) * cdiv(in->h, 2) * cdiv(in->w, 16) < ((int64_t)1 << 31);
}
size_t k5f_conv_bytes(int cin_k, const h3d_tensor* out) {
  const K5FPlan p = k5f_plan(cin_k, out);
  return p.wk_bytes + p.part_bytes;
}
// .. without the sums of the splits: a call that has no room for those is not split (a workspace that is large enough for a larger volume)
size_t k5f_filter_bytes(int cin_k, const h3d_tensor* out) { return k5f_plan(cin_k, out).wk_bytes; }
size_t k5f_bf_bytes(const h3d_tensor* x, int cout) {
  const K5FBfPlan p = k5f_bf_plan(x, cout);
  return p.part_bytes + p.db_bytes;
}

// cin / cout: channels of the layer; pmin, pmax: planes of `in` (and of the mask) that are stored and inside the volume
h3d_status k5f_conv(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const void* w, int cin, int cout, bool transposed, const float* bias,
                    h3d_tensor* out, int pmin, int pmax, float slope_in, float slope_out, void* ws, size_t ws_bytes,
                    hipStream_t s) {
  K5FPlan p = k5f_plan(in->c, out);
  if (ws_bytes < p.wk_bytes + p.part_bytes) { p.nsplit = 1; p.per_split = p.ncig; p.part_bytes = 0; }
  if (p.tiles >= ((int64_t)1 << 31) || p.ncog > 65535) return fail(handle, H3D_EINVAL, "conv3d_k5: too many blocks");
  K5FArgs a;
  a.in = make_geo(in); a.mask = mask ? make_geo(mask) : a.in; a.out = make_geo(out);
  a.cin = in->c; a.cout = out->c; a.ncig = p.ncig;
  a.pmin = pmin; a.pmax = pmax; a.npg = p.npg; a.nhg = p.nhg; a.nwg = p.nwg; a.per_split = p.per_split;
  a.split_elems = p.nsplit > 1 ? (int64_t)out->n * out->c * out->d * out->h * out->w : 0;
  a.slope_in = slope_in; a.slope_out = slope_out;
  a.vec = out->w % 4 == 0 && (p.nsplit > 1 || ((uintptr_t)out->data % 16 == 0 && a.out.cstride % 4 == 0 && a.out.nstride % 4 == 0));
  float* wk = (float*)ws;
  float* part = (float*)((char*)ws + p.wk_bytes);
  const int64_t total = (int64_t)p.ncog * p.ncig * 125 * p.cb * 64;
  hipLaunchKernelGGL(k5f_pack_kernel, dim3((unsigned)cdiv(total, 256)), dim3(256), 0, s, (const float*)w, wk, cin, cout, transposed ? 1 : 0, p.ncig, p.cb, total);
#define H3D_K5F(CB, TR, HV) H3D_TRY((k5f_launch_m<CB, TR, HV>(handle, in, mask, wk, bias, out, part, a, p, s)))
  if (p.cb == 2 && p.tr == 8) { if (p.hv == 2) H3D_K5F(2, 8, 2); else H3D_K5F(2, 8, 1); }
  else if (p.cb == 2) { if (p.hv == 2) H3D_K5F(2, 2, 2); else H3D_K5F(2, 2, 1); }
  else if (p.tr == 8) { if (p.hv == 2) H3D_K5F(1, 8, 2); else H3D_K5F(1, 8, 1); }
  else { if (p.hv == 2) H3D_K5F(1, 2, 2); else H3D_K5F(1, 2, 1); }
#undef H3D_K5F
  if (p.nsplit > 1)
    hipLaunchKernelGGL(k5f_split_kernel, dim3((unsigned)cdiv(a.split_elems, 256)), dim3(256), 0, s, (const float*)part, bias, (float*)out->data, a, p.nsplit);
  return H3D_OK;
}

h3d_status k5f_bwd_filter(void* handle, const h3d_tensor* x, const h3d_tensor* dz, const h3d_tensor* z, float* dw, float* db, int pmin, int pmax,
                          float slope, void* ws, hipStream_t s) {
  const K5FBfPlan p = k5f_bf_plan(x, dz->c);
  if (p.cogs > 65535 || 5 * (int64_t)p.cigs > 65535) return fail(handle, H3D_EINVAL, "conv3d_k5_bwd_filter: too many channels");
  K5FBfArgs a;
  a.x = make_geo(x); a.g = make_geo(dz); a.z = z ? make_geo(z) : a.g;
  a.x.d = std::max(a.x.d, 1);      // (an empty shard has no tiles)
  a.cin = x->c; a.cout = dz->c; a.pmin = pmin; a.pmax = pmax;
  a.nhg = p.nhg; a.nwg = p.nwg; a.cip = p.cigs * 16; a.cop = p.cogs * 16;
  a.tiles = p.tiles; a.tiles_per_chunk = p.tiles_per_chunk; a.slope = slope;
  float* part = (float*)ws;
  float* part_db = (float*)((char*)ws + p.part_bytes);
  const bool narrow = x->w <= 16;
  if (z && narrow) H3D_TRY((k5f_bf_launch<true, true>(handle, x, dz, z, part, part_db, a, p, s)));
  else if (z) H3D_TRY((k5f_bf_launch<true, false>(handle, x, dz, z, part, part_db, a, p, s)));
  else if (narrow) H3D_TRY((k5f_bf_launch<false, true>(handle, x, dz, z, part, part_db, a, p, s)));
  else H3D_TRY((k5f_bf_launch<false, false>(handle, x, dz, z, part, part_db, a, p, s)));
  note_kernel(handle, "k5f_bwf_kernel");
  taps_reduce(part, part_db, dw, db, 125, x->c, dz->c, a.cip, a.cop, p.nchunks, p.nchunks, 1.f, s);
  return H3D_OK;
}

}  // namespace h3d
