// Forward and data gradient of the 2x2x2 stride-2 transposed convolution on the matrix cores (bf16); the filter gradient: deconv_bf.hip.
//
// Data gradient of the transposed convolution:
//
//   dx[ci][v] = sum over co and the 8 taps k = (a,b,c) of W[ci][co][k] * dy[co][2d+a][2h+b][2w+c]
//
// a GEMM whose contraction index (co, k) needs no re-layout on either side: with
// v_mfma_f32_32x32x16_bf16 a lane feeds the 8 taps of ONE output channel — for the B operand the
// 2x2x2 block of dy above its coarse voxel (four dword loads, consecutive lanes = consecutive dwords),
// for the A operand 16 contiguous bytes of W[ci][co][0..8).  Rows = input channels, columns = 32 coarse
// voxels along W, one K-step = two output channels.  W^T sits in LDS for the whole (persistent)
// workgroup, as [co][ci] units with an odd pitch; every dy element is loaded exactly once.
#include <algorithm>

#include "rowload.h"

namespace h3d {
namespace {

// whole aligned 16-byte pieces in every row of t
bool rows_v16(const h3d_tensor* t) {
  const Geo g = make_geo(t);
  return t->w % 8 == 0 && (uintptr_t)t->data % 16 == 0 && g.cstride % 8 == 0 && g.nstride % 8 == 0;
}
// a sample, with the strides of the tensor that a view is part of, is reached by 31-bit byte offsets: offsets at and past 2 GiB are what the kernels give to
// lanes that have nothing to load or store
bool fits31(const h3d_tensor* t) { return sample_span(t) < ((int64_t)1 << 30); }
// rows read in pieces that may run past their end: a sample holds at least one piece, and 32-bit byte offsets reach all of it
bool rows_any(const h3d_tensor* t) {
  const int64_t span = stored_span(make_geo(t));
  return span >= 8 && span < ((int64_t)1 << 30);
}

constexpr int DD_NW = 8;
constexpr int DD_BATCH = 8;      // K-steps (pairs of output channels) whose dy loads are in flight together

struct DbdArgs {
  Geo x, y;          // x: coarse tensor (dx), y: fine tensor (dy)
  int cin, cout;
  int wblks;         // 32-voxel column blocks per coarse row
  int64_t ncb;       // column blocks in total
};

// STREAM (dy of at least STREAM_PAST_CACHE_BYTES): dy is read past the last-level cache; it is read once, and kept there it displaces what
// is being written.  128 -> 64 channels from 64x256x256 (537 MB): 171 -> 156 us; 2 x 32 channels from 32x128x128 (67 MB) 18.9 -> 20.2.
template <int MRB, bool STREAM>
__global__ void __launch_bounds__(64 * DD_NW, 2) deconv_bd_mfma_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ w,
                                                                     bf16_t* __restrict__ dx, DbdArgs a) {
  constexpr int CP = (32 * MRB) | 1;          // LDS pitch of an output channel in 16-byte units
  extern __shared__ uint4 lds[];              // [cout rounded up to even][CP]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int nks = (a.cout + 1) / 2;
  // this workgroup's channels of dx
  const int ci0 = (int)blockIdx.y * 32 * MRB, ncin = min(a.cin - ci0, 32 * MRB);
  const uint32_t x_bytes = (uint32_t)(a.x.nstride - ci0 * a.x.cstride) * 2;
  dx += ci0 * a.x.cstride;

  // ---- W[ci][co][8] -> LDS [co][ci]; rows of a padding channel are zero (their dy operand is zero too)
  {
    const uint4* wu = reinterpret_cast<const uint4*>(w) + (int64_t)ci0 * a.cout;
    const int total = ncin * a.cout;
    for (int i = tid; i < total; i += 64 * DD_NW) {
      const int ci = i / a.cout, co = i % a.cout;
      lds[co * CP + ci] = wu[i];
    }
    if (a.cout & 1)
      for (int i = tid; i < CP; i += 64 * DD_NW) lds[a.cout * CP + i] = uint4{0, 0, 0, 0};
  }
  __syncthreads();

  const int Wc = a.x.w, Hc = a.x.h, Dc = a.x.d, Wf = a.y.w;
  const char* a_base = reinterpret_cast<const char*>(lds) + 16 * (half * CP + col);
  for (int64_t cb = (int64_t)blockIdx.x * DD_NW + wave; cb < a.ncb; cb += (int64_t)gridDim.x * DD_NW) {
    int64_t r = cb;
    const int wb = (int)(r % a.wblks); r /= a.wblks;
    const int h = (int)(r % Hc); r /= Hc;
    const int d = (int)(r % Dc);
    const int n = (int)(r / Dc);
    const int wv = wb * 32 + col;
    const __amdgpu_buffer_rsrc_t rs_y = row_rsrc(dy + n * a.y.nstride, (uint32_t)a.y.nstride * 2);
    const int vbase = wv < Wc ? 2 * (half * (int)a.y.cstride + (2 * d + a.y.hlo) * (int)a.y.plane + 2 * h * Wf + 2 * wv) : ROW_OOB;

    f32x16 acc[MRB];
#pragma unroll
    for (int rb = 0; rb < MRB; ++rb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rb][i] = 0.f;

    uint32_t bqa[DD_BATCH][4], bqb[DD_BATCH][4];     // two batches of dy operands: one in flight, one being multiplied
    auto load_batch = [&](int s0, uint32_t (&dst)[DD_BATCH][4]) {
#pragma unroll
      for (int j = 0; j < DD_BATCH; ++j) {
        const int s = s0 + j;
        // the channel pair of this K-step is a scalar offset; lanes of a missing channel read nothing
        const int vo = (s < nks && 2 * s + half < a.cout) ? vbase : ROW_OOB;
        const int so = __builtin_amdgcn_readfirstlane(2 * (2 * s) * (int)a.y.cstride);
#pragma unroll
        for (int ab = 0; ab < 4; ++ab)
          dst[j][ab] = __builtin_amdgcn_raw_buffer_load_b32(rs_y, vo, so + 2 * ((ab >> 1) * (int)a.y.plane + (ab & 1) * Wf), STREAM ? 2 : 0);
      }
    };
    auto read_a = [&](int s, uint4 (&dst)[MRB]) {
#pragma unroll
      for (int rb = 0; rb < MRB; ++rb) dst[rb] = *reinterpret_cast<const uint4*>(a_base + 16 * (2 * s * CP + rb * 32));
    };
    auto mul_batch = [&](int s0, const uint32_t (&src)[DD_BATCH][4]) {
      uint4 af[2][MRB];       // weight fragments of this K-step and of the next
      if (s0 < nks) read_a(s0, af[0]);
#pragma unroll
      for (int j = 0; j < DD_BATCH; ++j) {
        const int s = s0 + j;
        if (s < nks) {
          if (s + 1 < nks && j + 1 < DD_BATCH) read_a(s + 1, af[(j + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          const uint4 bu = {src[j][0], src[j][1], src[j][2], src[j][3]};
          const bf16x8 B = __builtin_bit_cast(bf16x8, bu);
#pragma unroll
          for (int rb = 0; rb < MRB; ++rb)
            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[j & 1][rb]), B, acc[rb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    load_batch(0, bqa);
    for (int s0 = 0; s0 < nks; s0 += 2 * DD_BATCH) {
      load_batch(s0 + DD_BATCH, bqb);
      mul_batch(s0, bqa);
      load_batch(s0 + 2 * DD_BATCH, bqa);
      mul_batch(s0 + DD_BATCH, bqb);
    }

    // ---- dx[ci][d][h][wv]: accumulator register r of row block rb is channel 32 rb + 8 (r/4) + 4 half + r % 4
    // (buffer stores: the lane's voxel offset plus a scalar channel offset; a store to a channel beyond Cin or a
    //  column beyond W gets an out-of-range offset and is dropped)
    {
      const __amdgpu_buffer_rsrc_t rs_x = row_rsrc(dx + n * a.x.nstride, x_bytes);
      const int vo = wv < Wc ? 2 * (4 * half * (int)a.x.cstride + (d + a.x.hlo) * (int)a.x.plane + h * Wc + wv) : ROW_OOB;
#pragma unroll
      for (int rb = 0; rb < MRB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int ci_u = rb * 32 + 8 * (i / 4) + (i % 4);      // wave-uniform part of the channel
          const bool ch_ok = ci_u + 4 * half < ncin;
          __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(acc[rb][i]), rs_x, ch_ok ? vo : ROW_OOB,
                                                __builtin_amdgcn_readfirstlane(2 * ci_u * (int)a.x.cstride), 0);
        }
    }
  }
}

template <int MRB, bool STREAM>
h3d_status dbd_launch_as(void* handle, const bf16_t* dy, const bf16_t* w, bf16_t* dx, const DbdArgs& a, size_t lds_bytes,
                      hipStream_t stream) {
  static size_t attr_bytes = 0;
  if (lds_bytes > attr_bytes) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(deconv_bd_mfma_kernel<MRB, STREAM>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_bytes) != hipSuccess)
      return fail(handle, H3D_EHIP, "deconv2_bwd_data: cannot set the dynamic LDS size to %zu bytes", lds_bytes);
    attr_bytes = lds_bytes;
  }
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  const int64_t groups = cdiv(a.cin, 32 * MRB);
  const int64_t grid = std::max<int64_t>(1, std::min<int64_t>(num_cu / groups, cdiv(a.ncb, DD_NW)));
  hipLaunchKernelGGL((deconv_bd_mfma_kernel<MRB, STREAM>), dim3((unsigned)grid, (unsigned)groups), dim3(64 * DD_NW), lds_bytes, stream, dy, w, dx, a);
  note_kernel(handle, "deconv_bd_mfma_kernel<%d,%d>", MRB, (int)STREAM);
  return H3D_OK;
}
static int64_t fine_bytes(const Geo& y, int c) { return (int64_t)y.n * c * y.d * y.plane * (int64_t)sizeof(bf16_t); }
template <int MRB>
h3d_status dbd_launch(void* handle, const bf16_t* dy, const bf16_t* w, bf16_t* dx, const DbdArgs& a, size_t lds_bytes, hipStream_t stream) {
  // (groups of channels of dx read dy at about the same time: through the cache)
  return a.cin <= 32 * MRB && fine_bytes(a.y, a.cout) >= STREAM_PAST_CACHE_BYTES ? dbd_launch_as<MRB, true>(handle, dy, w, dx, a, lds_bytes, stream)
                                                            : dbd_launch_as<MRB, false>(handle, dy, w, dx, a, lds_bytes, stream);
}

// The filter lies in LDS, 32 MRB channels of dx of it a workgroup: all blocks of 32 where up to four fit, else groups of blocks in blockIdx.y, each of which
// reads dy.  us, direct kernel and here: 128 -> 128 channels (of dx and of dy) from 32x64x64 634 and 68 (402 MB of dy in two passes), 128 -> 96 460 and 51,
// 96 -> 128 from 16x32x64 139 and 22, 256 -> 64 from 8x32x32 55 and 15, 200 -> 33 from 4x20x24 22 and 12.
size_t dbd_lds_bytes(int mrb, int cout) { return (size_t)((cout + 1) / 2 * 2) * ((32 * mrb) | 1) * 16; }
int dbd_mrb(int cin, int cout) {
  const int64_t blocks = cdiv(cin, 32);
  int64_t mrb = std::min<int64_t>(4, blocks);
  while (mrb > 0 && dbd_lds_bytes((int)mrb, cout) > 160 * 1024) --mrb;
  return mrb == 0 ? 0 : (int)cdiv(blocks, cdiv(blocks, mrb));      // groups alike
}

}  // namespace

bool deconv_bd_mfma_supported(const h3d_tensor* dx, const h3d_tensor* dy, const void* w) {
  if (dx->dtype != H3D_BF16 || dx->c < 1 || dx->c > 1024 || dy->c < 1) return false;
  if ((uintptr_t)dy->data % 4 != 0 || (uintptr_t)w % 16 != 0) return false;
  if (dbd_mrb(dx->c, dy->c) == 0) return false;
  return fits31(dx) && fits31(dy);
}

h3d_status deconv_bd_mfma(void* handle, const h3d_tensor* dy, const void* w, h3d_tensor* dx, hipStream_t stream) {
  DbdArgs a;
  a.x = make_geo(dx); a.y = make_geo(dy);
  a.cin = dx->c; a.cout = dy->c;
  a.wblks = (int)cdiv(dx->w, 32);
  a.ncb = (int64_t)dx->n * dx->d * dx->h * a.wblks;
  if (a.ncb == 0) return H3D_OK;
  const int mrb = dbd_mrb(a.cin, a.cout);
  const size_t lds_bytes = dbd_lds_bytes(mrb, a.cout);
  const bf16_t* yp = (const bf16_t*)dy->data;
  const bf16_t* wp = (const bf16_t*)w;
  bf16_t* xp = (bf16_t*)dx->data;
  h3d_status st;
  if (mrb == 4) st = dbd_launch<4>(handle, yp, wp, xp, a, lds_bytes, stream);
  else if (mrb == 3) st = dbd_launch<3>(handle, yp, wp, xp, a, lds_bytes, stream);
  else if (mrb == 2) st = dbd_launch<2>(handle, yp, wp, xp, a, lds_bytes, stream);
  else st = dbd_launch<1>(handle, yp, wp, xp, a, lds_bytes, stream);
  if (st != H3D_OK) return st;
  return launch_status(handle, "deconv2_bwd_data_mfma");
}

}  // namespace h3d

// ---------------------------------------------------------------------------------------------------
// Forward of the transposed convolution:
//
//   y[co][2d+a][2h+b][2w+c] = bias[co] + sum over ci of W[ci][co][a,b,c] * x[ci][d,h,w]
//
// a GEMM with rows (co, k = (a,b,c)), columns = coarse voxels and the contraction over ci.  NCDHW keeps
// channels a whole volume apart, so (as in the 3x3x3 kernels) the x tile is transposed on its way into
// LDS: 16-byte units of 8 channels, [ci-group][voxel].  Eight wavefronts share the staged tile; wavefront
// w owns the row blocks w, w+8, ... and keeps their weight fragments (pre-packed in fragment order) in
// registers for the whole persistent workgroup.  In an accumulator the two parities c of a (co,a,b) are
// adjacent registers of one lane, so every lane stores whole dwords and consecutive lanes write
// consecutive dwords of a fine row.
namespace h3d {
namespace {

constexpr int DF_NW = 8;
constexpr int DF_GRP = 16;       // row blocks (of 4 output channels) of a workgroup
constexpr int DF_CBI = 8;        // 32-voxel column blocks staged per iteration (one per wavefront)

struct DfwArgs {
  Geo x, y;
  int cin, cout;
  int wblks;
  int64_t ncb;
};

// wp: [row block][K-step][lane][8] bf16; lane l, element e: row 32 rb + l % 32 = 8 co + k, channel 16 ks + 8 (l/32) + e
__global__ void deconv_fw_pack_kernel(const bf16_t* __restrict__ w, bf16_t* __restrict__ wp, int cin, int cout, int nrb, int ks) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)nrb * ks * 512) return;
  const int e = (int)(i & 7), lane = (int)((i >> 3) & 63);
  int64_t r = i >> 9;
  const int s = (int)(r % ks), rb = (int)(r / ks);
  const int row = rb * 32 + (lane & 31), co = row >> 3, k = row & 7, ci = s * 16 + (lane >> 5) * 8 + e;
  wp[i] = (co < cout && ci < cin) ? w[((int64_t)ci * cout + co) * 8 + k] : (bf16_t)0;
}

// STREAM (y of at least STREAM_PAST_CACHE_BYTES): written past the last-level cache (whole lines of a fine row leave at once): 128 -> 64
// channels onto 64x256x256 (537 MB) 171 -> 138 us.
// V16: rows of whole aligned 16-byte pieces; otherwise a piece may run into the next row (those columns are computed and dropped) but
// not past the sample.  The direct kernel, which such widths had to take, reads x once per 8 output channels: 128 -> 64 channels onto
// 64x256x248 1088 -> 204 us, 64 -> 32 onto 32x192x196 104 -> 29.
template <int RBW, int KS, bool STREAM, bool V16>
__global__ void __launch_bounds__(64 * DF_NW, 2) deconv_fw_mfma_kernel(const bf16_t* __restrict__ x, const uint4* __restrict__ wp,
                                                                     const float* __restrict__ bias, bf16_t* __restrict__ y,
                                                                     DfwArgs a) {
  constexpr int NCIG = 2 * KS;                     // groups of 8 input channels
  constexpr int CBU = NCIG * 32 + 4;               // LDS units of one column block: [ci-group][32 voxels] (+4: staggers the blocks)
  extern __shared__ uint4 lds[];                   // [2 buffers][DF_CBI][CBU]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int Wc = a.x.w, Hc = a.x.h, Dc = a.x.d, Wf = a.y.w;
  const int nrb = (8 * a.cout + 31) / 32, rb0 = (int)blockIdx.y * DF_GRP + wave;      // a workgroup has up to 64 output channels

  // ---- this wavefront's weight fragments
  uint4 A[RBW][KS];
#pragma unroll
  for (int j = 0; j < RBW; ++j) {
    const int rb = rb0 + DF_NW * j;
#pragma unroll
    for (int s = 0; s < KS; ++s) A[j][s] = rb < nrb ? wp[((int64_t)rb * KS + s) * 64 + lane] : uint4{0, 0, 0, 0};
  }

  float bv[RBW][4];
#pragma unroll
  for (int j = 0; j < RBW; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int co = 4 * (rb0 + DF_NW * j) + q;
      bv[j][q] = (bias && co < a.cout) ? bias[co] : 0.f;
    }

  const int ncb = (int)a.ncb;
  const int it0 = blockIdx.x * DF_CBI, it_stride = gridDim.x * DF_CBI;
  auto decode = [&](int cb, int& n, int& d, int& h, int& w0) {
    int r = cb;
    w0 = (r % a.wblks) * 32; r /= a.wblks;
    h = r % Hc; r /= Hc;
    d = r % Dc;
    n = r / Dc;
  };
  // staging: a lane takes one (ci-group, group of 8 voxels) item of its wavefront's column block per round
  constexpr int SROUNDS = (NCIG * 4 + 63) / 64;
  u32x4 sv[SROUNDS][8];
  const int xspan = (int)stored_span(a.x);
  auto stage_load = [&](int cb0) {
    const int cb = cb0 + wave;
    int n, d, h, w0;
    decode(cb < ncb ? cb : 0, n, d, h, w0);
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(x + n * a.x.nstride, (uint32_t)(V16 ? a.x.nstride : xspan) * 2);
#pragma unroll
    for (int r = 0; r < SROUNDS; ++r) {
      const int item = lane + 64 * r, cig = item >> 2, vg = item & 3;
      const int wv = w0 + 8 * vg;
      if constexpr (!V16) {
        const int o = cig * 8 * (int)a.x.cstride + (d + a.x.hlo) * (int)a.x.plane + h * Wc;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          sv[r][e] = __builtin_bit_cast(u32x4, row8<false>(rs, o + e * (int)a.x.cstride, wv, Wc, xspan, cb < ncb && cig < NCIG && cig * 8 + e < a.cin));
        continue;
      }
      const bool ok = cb < ncb && cig < NCIG && wv + 8 <= Wc;
      const int base = 2 * (cig * 8 * (int)a.x.cstride + (d + a.x.hlo) * (int)a.x.plane + h * Wc + wv);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        sv[r][e] = __builtin_amdgcn_raw_buffer_load_b128(rs, (ok && cig * 8 + e < a.cin) ? base : ROW_OOB,
                                                         __builtin_amdgcn_readfirstlane(2 * e * (int)a.x.cstride), 0);
    }
  };
  auto stage_store = [&](int cb0, int buf) {
    int n, d, h, w0;
    if constexpr (!V16) decode(cb0 + wave < ncb ? cb0 + wave : 0, n, d, h, w0);
    uint4* dst0 = lds + (buf * DF_CBI + wave) * CBU;
#pragma unroll
    for (int r = 0; r < SROUNDS; ++r) {
      const int item = lane + 64 * r, cig = item >> 2, vg = item & 3;
      if (cig >= NCIG) continue;
      if constexpr (!V16) {
        const int o = cig * 8 * (int)a.x.cstride + (d + a.x.hlo) * (int)a.x.plane + h * Wc;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          sv[r][e] = __builtin_bit_cast(u32x4, fix8<false>(__builtin_bit_cast(uint4, sv[r][e]), o + e * (int)a.x.cstride, w0 + 8 * vg, Wc, xspan));
      }
      uint4* dst = dst0 + cig * 32 + 8 * vg;
#pragma unroll
      for (int j = 0; j < 4; ++j) {       // dword j of each channel = voxels 2j, 2j+1 of the group
        uint4 u0, u1;
        u0.x = __builtin_amdgcn_perm(sv[r][1][j], sv[r][0][j], 0x05040100); u1.x = __builtin_amdgcn_perm(sv[r][1][j], sv[r][0][j], 0x07060302);
        u0.y = __builtin_amdgcn_perm(sv[r][3][j], sv[r][2][j], 0x05040100); u1.y = __builtin_amdgcn_perm(sv[r][3][j], sv[r][2][j], 0x07060302);
        u0.z = __builtin_amdgcn_perm(sv[r][5][j], sv[r][4][j], 0x05040100); u1.z = __builtin_amdgcn_perm(sv[r][5][j], sv[r][4][j], 0x07060302);
        u0.w = __builtin_amdgcn_perm(sv[r][7][j], sv[r][6][j], 0x05040100); u1.w = __builtin_amdgcn_perm(sv[r][7][j], sv[r][6][j], 0x07060302);
        dst[2 * j] = u0;
        dst[2 * j + 1] = u1;
      }
    }
  };

  if (it0 < ncb) { stage_load(it0); stage_store(it0, 0); }
  __syncthreads();
  int buf = 0;
  for (int cb0 = it0; cb0 < ncb; cb0 += it_stride, buf ^= 1) {
    const bool more = cb0 + it_stride < ncb;
    if (more) stage_load(cb0 + it_stride);       // in flight during this iteration's MFMAs
#pragma unroll 1
    for (int c = 0; c < DF_CBI; ++c) {
      const int cb = cb0 + c;
      if (cb >= ncb) break;
      int n, d, h, w0;
      decode(cb, n, d, h, w0);
      const uint4* bp = lds + (buf * DF_CBI + c) * CBU + half * 32 + col;
      f32x16 acc[RBW];
#pragma unroll
      for (int j = 0; j < RBW; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 B = __builtin_bit_cast(bf16x8, bp[s * 64]);
#pragma unroll
        for (int j = 0; j < RBW; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, A[j][s]), B, acc[j], 0, 0, 0);
      }
      // ---- rows 32 rb + 8 (i/4) + 4 half + i % 4 = 8 co + k: co = 4 rb + i / 4, a = half, b = (i % 4) / 2, c = i % 2
      const __amdgpu_buffer_rsrc_t rs_y = row_rsrc(y + n * a.y.nstride, (uint32_t)a.y.nstride * 2);
      const int wv = w0 + col;
      const int vo = wv < Wc ? 2 * ((2 * d + half + a.y.hlo) * (int)a.y.plane + 2 * h * Wf + 2 * wv) : ROW_OOB;
#pragma unroll
      for (int j = 0; j < RBW; ++j) {
        const int rb = rb0 + DF_NW * j;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int co = 4 * rb + q;
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const uint32_t pk = pack_bf16x2(acc[j][4 * q + 2 * b] + bv[j][q], acc[j][4 * q + 2 * b + 1] + bv[j][q]);
            __builtin_amdgcn_raw_buffer_store_b32(pk, rs_y, co < a.cout ? vo : ROW_OOB,
                                                  __builtin_amdgcn_readfirstlane(2 * (co * (int)a.y.cstride + b * Wf)), STREAM ? 2 : 0);
          }
        }
      }
    }
    if (more) stage_store(cb0 + it_stride, buf ^ 1);
    __syncthreads();
  }
}

template <int RBW, int KS, bool STREAM, bool V16>
h3d_status dfw_launch_as(void* handle, const bf16_t* x, const uint4* wp, const float* bias, bf16_t* y, const DfwArgs& a,
                      hipStream_t stream) {
  constexpr size_t lds_bytes = (size_t)2 * DF_CBI * (2 * KS * 32 + 4) * 16;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(deconv_fw_mfma_kernel<RBW, KS, STREAM, V16>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_bytes) != hipSuccess)
      return fail(handle, H3D_EHIP, "deconv2_fwd: cannot set the dynamic LDS size to %zu bytes", lds_bytes);
    attr_set = true;
  }
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  const int64_t groups = cdiv(a.cout, 4 * DF_GRP);      // one resident round over all of them
  const int64_t grid = std::max<int64_t>(1, std::min<int64_t>(num_cu / groups, cdiv(a.ncb, DF_CBI)));
  hipLaunchKernelGGL((deconv_fw_mfma_kernel<RBW, KS, STREAM, V16>), dim3((unsigned)grid, (unsigned)groups), dim3(64 * DF_NW), lds_bytes, stream, x, wp, bias, y, a);
  note_kernel(handle, "deconv_fw_mfma_kernel<%d,%d,%d,%d>", RBW, KS, (int)STREAM, (int)V16);
  return H3D_OK;
}
template <int RBW, int KS>
h3d_status dfw_launch(void* handle, const bf16_t* x, const uint4* wp, const float* bias, bf16_t* y, const DfwArgs& a, bool v16, hipStream_t stream) {
  if (!v16) return dfw_launch_as<RBW, KS, false, false>(handle, x, wp, bias, y, a, stream);
  // only where a fine row is whole 64-byte pieces: past the cache a piece that two rows share is written twice (us, past the cache and
  // through it: 128 -> 64 channels onto 64x240x240 299 and 182, 64 -> 32 onto 64x256x208 136 and 74, but 58 -> 24 onto 128x172x160 59 and 62)
  const bool pieces = a.y.w % 32 == 0 && (uintptr_t)y % 64 == 0 && a.y.cstride % 32 == 0 && a.y.nstride % 32 == 0;
  return pieces && fine_bytes(a.y, a.cout) >= STREAM_PAST_CACHE_BYTES ? dfw_launch_as<RBW, KS, true, true>(handle, x, wp, bias, y, a, stream)
                                                                     : dfw_launch_as<RBW, KS, false, true>(handle, x, wp, bias, y, a, stream);
}

}  // namespace

// Up to 1024 output channels, 64 a workgroup (each group reads x again, less than it writes).  us, direct kernel and here: 128->128 on 32x64x64 545 and 63,
// 64->96 on 16x48x80 112 and 29, 28->102 on 4 x 26x26x84 219 and 118, 32->128 on 12x16x80 29.7 and 14.5, 24->96 on 4x8x8 14.7 and 11.7 (few input channels: below).
constexpr int DF_COUT = 1024;
bool deconv_fw_mfma_supported(const h3d_tensor* x, const h3d_tensor* y) {
  if (x->dtype != H3D_BF16 || x->c < 1 || x->c > 128 || y->c < 1 || y->c > DF_COUT || (uintptr_t)y->data % 4 != 0) return false;
  if (make_geo(y).cstride % 2 != 0 || make_geo(y).nstride % 2 != 0) return false;      // results leave as pairs in one dword
  // Few input channels stay with the direct kernel, which reads x once per 8 output channels; this one pads them to 64.  More than 64 output channels
  // pay from 16 on, in aligned rows of large volumes from 8.  us, direct and here: 2->96 on 16^3 9.6 and 12.3, 8->128 on 8^3 9.6 and 11.8, 12->65 on 8^3
  // 10.8 and 11.7, 14->192 there 11.7 and 11.9, 16->128 on 16^3 13.1 and 12.8; 8->96 on 16x32x32 13.5 and 14.1, on 32x48x64 43 and 38, 6->65 on 32x64x64 37 and
  // 33, 4->96 there 44 and 46; ragged 8->65 on 32x64x66 43 and 54, 16->72 on 8x10x14 12.2 and 12.7, 17->1000 on 16x18x22 48 and 33.
  // Up to 64: 8->16 on 8x9x10 8.9 and 10.0, 16->16 there 12.3 and 10.0; 16->16 on 32x62x66 21 and 26, 16->32 there 33 and 26; 4->4 on 2 x 24x70x90 13 and 37.
  const int64_t voxels = (int64_t)x->n * x->d * x->h * x->w;
  const bool v16 = rows_v16(x);
  if (!v16 && !rows_any(x)) return false;
  if (y->c > 64) {
    if (x->c < (v16 && voxels >= 98304 ? 8 : 16)) return false;
  } else if (!v16 && (voxels < 49152 ? x->c < 16 : x->c * y->c < 512)) {
    return false;
  }
  const int64_t ncb = (int64_t)x->n * x->d * x->h * cdiv(x->w, 32);
  return fits31(x) && fits31(y) && ncb < ((int64_t)1 << 30);
}

size_t deconv_fw_mfma_ws_bytes(const h3d_tensor* x, const h3d_tensor* y) {
  const int ks = x->c > 64 ? 8 : 4, nrb = (int)cdiv(8 * (int64_t)y->c, 32);
  return (size_t)nrb * ks * 1024;
}

h3d_status deconv_fw_mfma(void* handle, const h3d_tensor* x, const void* w, const float* bias, h3d_tensor* y, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
  DfwArgs a;
  a.x = make_geo(x); a.y = make_geo(y);
  a.cin = x->c; a.cout = y->c;
  a.wblks = (int)cdiv(x->w, 32);
  a.ncb = (int64_t)x->n * x->d * x->h * a.wblks;
  if (a.ncb == 0) return H3D_OK;
  if (!ws || ws_bytes < deconv_fw_mfma_ws_bytes(x, y) || (uintptr_t)ws % 16) return fail(handle, H3D_EWORKSPACE, "deconv2_fwd: workspace too small or misaligned");
  const int ks = a.cin > 64 ? 8 : 4, nrb = (int)cdiv(8 * (int64_t)a.cout, 32), rbw = nrb > DF_NW ? 2 : 1;
  hipLaunchKernelGGL(deconv_fw_pack_kernel, dim3((unsigned)cdiv((int64_t)nrb * ks * 512, 256)), dim3(256), 0, stream, (const bf16_t*)w,
                     (bf16_t*)ws, a.cin, a.cout, nrb, ks);
  const bf16_t* xp = (const bf16_t*)x->data;
  bf16_t* yp = (bf16_t*)y->data;
  const uint4* wq = (const uint4*)ws;
  h3d_status st;
  const bool v16 = rows_v16(x);
  if (ks == 8) st = rbw == 2 ? dfw_launch<2, 8>(handle, xp, wq, bias, yp, a, v16, stream) : dfw_launch<1, 8>(handle, xp, wq, bias, yp, a, v16, stream);
  else st = rbw == 2 ? dfw_launch<2, 4>(handle, xp, wq, bias, yp, a, v16, stream) : dfw_launch<1, 4>(handle, xp, wq, bias, yp, a, v16, stream);
  if (st != H3D_OK) return st;
  return launch_status(handle, "deconv2_fwd_mfma");
}

}  // namespace h3d
