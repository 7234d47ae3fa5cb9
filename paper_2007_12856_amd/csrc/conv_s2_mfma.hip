// Stride-2 3x3x3 convolution of bf16 tensors on the matrix cores, all three passes, straight from the caller's tensors
// (y[p] = sum_k w[k] x~[2p+k-1]).  Per axis an even fine position 2c meets tap k = 1 of coarse position c, an odd one 2c+1
// taps k = 2 of c and k = 0 of c+1, so 27 of the 8 x 27 (parity, shift) products exist.  The rewriting as a stride-1
// convolution over the eight parity sub-lattices (conv_s2.hip, still the route of fp32 tensors and large first layers) executes all 216
// of them and moves both tensors through memory three times; these kernels execute the 27.
//
// 64 -> 128 channels on 64^3 (14.5 GFlop and 42 MB a pass: 6 us of matrix cores, 6 us of memory), all three passes of a masked
// layer: 818 us by the rewriting, 104 us here (profiled, a few per cent slower: 29 forward, 30 backward-data, 34 + 10 backward-filter, 4 + 3 packing).
// At that size what bounds them is the serial chain of a workgroup (fetch a tile, transpose it into LDS, multiply): there are
// one to two workgroups per CU, and every one lives for two to eight stages.
#include <algorithm>

#include "rowload.h"
#include "taps.h"

namespace h3d {

struct S2Args {
  Geo x, y, m;                      // fine side, coarse side (y or dy), saved output (mask)
  int cin, cout;
  int nchunk;                       // 16-channel chunks of the contraction (forward: of cin, padded to 2; backward-data: of cout)
  int tiles_w, tiles_h, ntiles;
  float slope;
  int vec;                          // result rows are 4-byte aligned pairs
  // backward-filter
  int segs, band, bands, nstrips, strips_per_chunk, nchunks, cogroups, cigroups;
};

// How a saved output is read (MASK): not at all; by row8 / row1 like the gradient; or, where it stores so many or so few elements that those do
// not reach it (s2_mask_fits), one by one at 64-bit addresses.  That form is slow and rare, and it needs no other workspace: the size
// query does not see the saved output.
enum { S2_NO_MASK = 0, S2_MASK = 1, S2_FAR_MASK = 2 };
__device__ __forceinline__ uint4 s2_far8(const bf16_t* row, int c, int w, bool ok) {
  uint32_t e[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) e[i] = ok && c + i < w ? (uint32_t)row[c + i] : 0u;
  return uint4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
}

// tile index of a workgroup: the workgroups of one XCD (linear index mod 8) take a contiguous run, so that neighbouring tiles,
// which share halo rows, meet in one L2
__device__ __forceinline__ int xcd_tile(int i, int n) {
  const int per = (n + 7) / 8, t = (i & 7) * per + (i >> 3);
  return t;      // may be >= n: such a workgroup has nothing to do
}

// ---------------------------------------------------------------------------------------------------------- forward
// A workgroup owns 4 rows x 32 columns of one output plane and up to 128 output channels.  Per stage of 32 input channels the
// 3 x 9 x 65 input patch is transposed into LDS (16-byte units of 8 channels); even and odd columns lie apart, so that the
// columns 2q + kw - 1 of 32 neighbouring outputs are 32 neighbouring units for every kw.  The contraction is split over the
// wavefronts: two of them take the two 16-channel halves of a stage each (a volume of 32^3 outputs has 256 tiles: with the
// channels in one wavefront half of the SIMDs would idle), and add their accumulators through LDS at the end, in order.
//   NCO = 2: two wavefront pairs take 64 channels each (CB = 2 blocks of 32) and all four rows;
//   NCO = 1: at most 64 output channels (CB = 1: 32): the pairs take two rows each.
// Weight fragments come from L2 in packed order, two (kd,kw) steps ahead, also into the next stage, whose rows are requested behind the last fragments of
// this one, three steps before they are needed.  us, one step ahead (and loads that the compiler had moved next to their use) and this:
// 64->128 on 64^3 31.6 and 30.2, 128->256 on 32^3 50 and 42, 256->256 on 16x32x32 88 and 71, 64->64 on 4 x 16x32x32 23.8 and 18.9, 48->40 on 16x40x72 23.4 and 18.4.
// The form of more than 64 output channels in aligned rows fills all 512 registers with it and keeps nine in scratch.
constexpr int SF_PITCH = 66, SF_ROWS = 9, SF_CIG = 3 * SF_ROWS * SF_PITCH, SF_UNITS = 4 * SF_CIG;   // row: 33 odd columns (from 2 w0 - 1), 32 even ones
constexpr size_t SF_LDS = (size_t)SF_UNITS * 16;

template <int NCO, int CB, bool V16>
__global__ void __launch_bounds__(256, 1) s2_fwd_kernel(const bf16_t* __restrict__ x, const uint4* __restrict__ wp, const float* __restrict__ bias,
                                                        bf16_t* __restrict__ y, S2Args a) {
  constexpr int R = NCO == 2 ? 4 : 2, T = CB * R;
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int khalf = wave & 1, pair = wave >> 1;
  int t = xcd_tile(blockIdx.x, a.ntiles);
  if (t >= a.ntiles) return;
  const int w0 = (t % a.tiles_w) * 32; t /= a.tiles_w;
  const int h0 = (t % a.tiles_h) * 4; t /= a.tiles_h;
  const int z = t % a.y.d, n = t / a.y.d;
  const int W = a.x.w, H = a.x.h;
  const int ncoblk = (a.cout + 31) / 32;
  const int blk0 = ((int)blockIdx.y * NCO + (NCO == 2 ? pair : 0)) * CB;
  const bf16_t* xs = x + (int64_t)n * a.x.nstride;
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(xs, (uint32_t)a.x.nstride * 2);
  const int cstride = (int)a.x.cstride, plane = (int)a.x.plane;

  // ---- staging plan: 4 x 27 rows of 8 column groups, and the one odd column in front of them
  constexpr int NITEM = 4 * 27 * 8, NR = (NITEM + 255) / 256;
  int off[NR], meta[NR];                  // element offset of the row (channel group included); cig | ok << 8 | unit << 9
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int item = tid + 256 * r;
    const int cg = item & 7;
    int q = item >> 3;
    const int row = q % SF_ROWS; q /= SF_ROWS;
    const int dz = q % 3, cig = q / 3;
    const int p = 2 * z + dz - 1, h = 2 * h0 + row - 1;
    const bool ok = item < NITEM && a.x.doff + p >= 0 && h >= 0 && h < H;
    off[r] = cig * 8 * cstride + (p + a.x.hlo) * plane + h * W;
    meta[r] = cig | (ok ? 256 : 0) | ((cig * SF_CIG + (dz * SF_ROWS + row) * SF_PITCH + 4 * cg) << 9);
  }
  int loff, lmeta;
  {
    int q = tid;
    const int row = q % SF_ROWS; q /= SF_ROWS;
    const int dz = q % 3, cig = q / 3;
    const int p = 2 * z + dz - 1, h = 2 * h0 + row - 1;
    const bool ok = tid < 4 * 27 && a.x.doff + p >= 0 && h >= 0 && h < H;
    loff = cig * 8 * cstride + (p + a.x.hlo) * plane + h * W;
    lmeta = cig | (ok ? 256 : 0) | ((cig * SF_CIG + (dz * SF_ROWS + row) * SF_PITCH) << 9);
  }
  uint4 v[NR][8];
  uint32_t lv[8];
  auto load_stage = [&](int st) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c0 = st * 32 + e;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const bool ok = (meta[r] & 256) && c0 + 8 * (meta[r] & 7) < a.cin;
        v[r][e] = row8<V16>(rs, off[r] + c0 * cstride, 2 * w0 + 8 * ((tid + 256 * r) & 7), W, (int)stored_span(a.x), ok);
      }
      lv[e] = row1(rs, loff + c0 * cstride, 2 * w0 - 1, W, (lmeta & 256) && c0 + 8 * (lmeta & 7) < a.cin);
    }
  };
  auto store_stage = [&](int st) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (tid + 256 * r >= NITEM) continue;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[r][e] = fix8<V16>(v[r][e], off[r] + (st * 32 + e) * cstride, 2 * w0 + 8 * ((tid + 256 * r) & 7), W, (int)stored_span(a.x));
      uint4* dst = lds + (meta[r] >> 9);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        dst[33 + k] = column_unit(v[r], 2 * k);
        dst[1 + k] = column_unit(v[r], 2 * k + 1);
      }
    }
    if (tid < 4 * 27)
      lds[lmeta >> 9] = uint4{lv[0] | (lv[1] << 16), lv[2] | (lv[3] << 16), lv[4] | (lv[5] << 16), lv[6] | (lv[7] << 16)};
  };

  f32x16 acc[CB][R];
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][r][i] = 0.f;

  const uint4* wbase[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c)
    wbase[c] = wp + ((int64_t)min(__builtin_amdgcn_readfirstlane(blk0) + c, ncoblk - 1) * a.nchunk + __builtin_amdgcn_readfirstlane(khalf)) * 27 * 64;
  const uint4* bbase = lds + (2 * khalf + (lane >> 5)) * SF_CIG + (NCO == 2 ? 0 : pair * 2 * R) * SF_PITCH + (lane & 31);

  const int nst = a.nchunk / 2;
  uint4 A[3][3][CB], B[2][2 * R + 1];
  auto load_a = [&](int st, int step) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const __amdgpu_buffer_rsrc_t rw = row_rsrc(wbase[c] + (int64_t)st * (2 * 27 * 64), 27 * 1024);
#pragma unroll
      for (int kh = 0; kh < 3; ++kh)
        A[step % 3][kh][c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16, ((step / 3) * 9 + kh * 3 + step % 3) * 1024, 0));
    }
  };
  load_a(0, 0);
  load_a(0, 1);
  load_stage(0);
  for (int st = 0; st < nst; ++st) {
    if (st) __syncthreads();
    store_stage(st);
    __syncthreads();
    auto load_b = [&](int step) {
      const int kw = step % 3;
#pragma unroll
      for (int r = 0; r < 2 * R + 1; ++r) B[step & 1][r] = bbase[((step / 3) * SF_ROWS + r) * SF_PITCH + (kw == 1 ? 33 : kw / 2)];
    };
    load_b(0);
#pragma unroll
    for (int step = 0; step < 9; ++step) {
      if (step + 2 < 9) load_a(st, step + 2);
      if (step + 1 < 9) load_b(step + 1);
      // Requests return in order: the next stage's rows are asked for behind the last weight fragments of this one, and the next stage's first
      // fragments behind them.
      if (step == 6 && st + 1 < nst) load_stage(st + 1);
      if (step >= 7 && st + 1 < nst) load_a(st + 1, step - 7);
      __builtin_amdgcn_sched_barrier(0);      // (or the compiler puts the loads next to their use)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
#pragma unroll
          for (int c = 0; c < CB; ++c) acc[c][r] = mfma32(A[step % 3][kh][c], B[step & 1][2 * r + kh], acc[c][r]);
    }
  }

  // ---- the two channel halves exchange half of their accumulators and finish the other half
  __syncthreads();
  float4* xch = reinterpret_cast<float4*>(lds);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (khalf == k) continue;               // what wavefront half k keeps goes out from the other one
#pragma unroll
    for (int i = 0; i < T / 2; ++i) {
      const int ti = k * (T / 2) + i;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        xch[((wave * (T / 2) + i) * 4 + q) * 64 + lane] = float4{acc[ti / R][ti % R][4 * q], acc[ti / R][ti % R][4 * q + 1], acc[ti / R][ti % R][4 * q + 2], acc[ti / R][ti % R][4 * q + 3]};
    }
  }
  __syncthreads();
  bf16_t* ys = y + (int64_t)n * a.y.nstride;
  const __amdgpu_buffer_rsrc_t ro = row_rsrc(ys, (uint32_t)a.y.nstride * 2);
  const int ycs = (int)a.y.cstride, W2 = a.y.w, H2 = a.y.h, j = lane & 31;
  const bool odd = lane & 1;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (khalf != k) continue;
#pragma unroll
    for (int i = 0; i < T / 2; ++i) {
      const int ti = k * (T / 2) + i, cb = ti / R, r = ti % R;
      if (blk0 + cb >= ncoblk) continue;
      float f[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 o = xch[(((wave ^ 1) * (T / 2) + i) * 4 + q) * 64 + lane];
        const float ov[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int co = (blk0 + cb) * 32 + acc_row(4 * q + e, lane);
          const float mine = acc[cb][r][4 * q + e];
          float s = (k == 0 ? mine + ov[e] : ov[e] + mine) + ((bias && co < a.cout) ? bias[co] : 0.f);
          if (!(s > 0.f)) s *= a.slope;
          f[4 * q + e] = s;
        }
      }
      const int h = h0 + (NCO == 2 ? 0 : pair * R) + r;
      const int base = (z + a.y.hlo) * (int)a.y.plane + h * W2;
      if (a.vec) {      // neighbouring lanes swap one value, so that a lane stores two neighbouring voxels of one channel
        const int w = w0 + j - (odd ? 1 : 0);
        const bool in = h < H2 && w < W2;
#pragma unroll
        for (int q = 0; q < 16; q += 2) {
          const int co = (blk0 + cb) * 32 + acc_row(q, lane) + (odd ? 1 : 0);
          const float give = odd ? f[q] : f[q + 1];
          const float got = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(give), 0xB1, 0xF, 0xF, true));
          const uint32_t pk = odd ? pack_bf16x2(got, f[q + 1]) : pack_bf16x2(f[q], got);
          __builtin_amdgcn_raw_buffer_store_b32(pk, ro, in && co < a.cout ? 2 * (co * ycs + base + w) : ROW_OOB, 0, 0);
        }
      } else {
        const int w = w0 + j;
        const bool in = h < H2 && w < W2;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int co = (blk0 + cb) * 32 + acc_row(q, lane);
          __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(f[q]), ro, in && co < a.cout ? 2 * (co * ycs + base + w) : ROW_OOB, 0, 0);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------------ backward-data
// A workgroup of 8 wavefronts owns 8 coarse rows x 32 coarse columns of one coarse plane, i.e. 2 x 16 x 64 voxels of dx, and 32
// input channels; a wavefront one coarse row, with one accumulator block for each of the eight parities (128 registers).  Per
// chunk of 16 output channels the 2 x 9 x 33 patch of g = dy act'(y) and the chunk's 27 weight fragments (27 KB) pass through
// LDS (two buffers): the eight fragments of g at the shifts {0,1}^3 feed 27 products.  The two W parities of a lane are
// neighbouring voxels and leave as one dword.
constexpr int SD_PITCH = 34, SD_ROWS = 9, SD_CIG = 2 * SD_ROWS * SD_PITCH, SD_W = 27 * 64, SD_BUF = SD_W + 2 * SD_CIG;
constexpr size_t SD_LDS = (size_t)2 * SD_BUF * 16;

template <int MASK, bool V16>
__global__ void __launch_bounds__(512) s2_bwd_data_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ m, const uint4* __restrict__ wp,
                                                          bf16_t* __restrict__ dx, S2Args a) {
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int t = xcd_tile(blockIdx.x, a.ntiles);
  if (t >= a.ntiles) return;
  const int w0 = (t % a.tiles_w) * 32; t /= a.tiles_w;
  const int h0 = (t % a.tiles_h) * 8; t /= a.tiles_h;
  const int z = t % a.y.d, n = t / a.y.d;
  const int ci0 = blockIdx.y * 32;
  const int W2 = a.y.w, H2 = a.y.h;
  const bf16_t* ys = dy + (int64_t)n * a.y.nstride;
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(ys, (uint32_t)a.y.nstride * 2);
  const int cstride = (int)a.y.cstride;

  // ---- staging plan: threads 0..287 take 8 columns of 4 channels, 288..359 the column behind the tile (with all 8 channels of a
  //      unit in one thread three wavefronts do the masking while five wait: 48 against 35 us at the size above)
  const bool full = tid < 288, tail = tid >= 288 && tid < 360;
  const int cg = full ? tid & 3 : 4;
  int q = full ? tid >> 2 : tid - 288;
  const int row = q % SD_ROWS; q /= SD_ROWS;
  const int pl = q % 2, cq = q / 2;
  const bool ok0 = (full || tail) && h0 + row < H2 && a.y.doff + z + pl < a.y.dglob;
  const int off = cq * 4 * cstride + (z + pl + a.y.hlo) * (int)a.y.plane + (h0 + row) * W2;
  const int col = w0 + 8 * cg;
  const bf16_t* ms = MASK ? m + (int64_t)n * a.m.nstride : ys;
  const __amdgpu_buffer_rsrc_t rm = row_rsrc(ms, (uint32_t)a.m.nstride * 2);
  const int mcs = (int)a.m.cstride, moff = cq * 4 * mcs + (z + pl + a.m.hlo) * (int)a.m.plane + (h0 + row) * W2;
  auto far_row = [&](int co) { return ms + (int64_t)co * a.m.cstride + (int64_t)(z + pl + a.m.hlo) * a.m.plane + (int64_t)(h0 + row) * W2; };
  const int unit = SD_W + (cq >> 1) * SD_CIG + (pl * SD_ROWS + row) * SD_PITCH + 8 * cg;
  // The loads of a chunk are the same buffer loads in every thread, without a branch around them: plain loads, and loads under a condition that returns
  // at their use, the compiler moves behind the products (or issues again there), and the chunk then waits for all of its latency.  us with a mask and without, before
  // and after: 128 -> 64 channels onto 64^3 34.7, 30.1 and 30.3, 25.4; 256 -> 128 onto 32^3 53, 45 and 46.9, 37.9; 256 -> 256 onto 16x32x32 60.5, 52.7 and 49.8, 40.9;
  // 64 -> 32 onto 64x64x128 22.7, 20.1 and 21.5, 18.4; 16 -> 16 onto 64x128x128 19.7, 17.4 and 19.6, 17.2.  Rows two chunks ahead (a second set of registers)
  // are slower: 31.8, 25.9 on the first, 24.8, 20.0 on the last.
  uint4 v[4], mv[4], wv[4];
  const uint4* wsrc = wp + (int64_t)blockIdx.y * a.nchunk * SD_W;
  const int last_unit = min(1536 + tid, SD_W - 1);      // the threads beyond the filter all take its last unit
  auto load_weights = [&](int c) {
    const __amdgpu_buffer_rsrc_t rw = row_rsrc(wsrc + (int64_t)c * SD_W, SD_W * 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) wv[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, 16 * (k < 3 ? tid + 512 * k : last_unit), 0, 0));
  };
  auto load_rows = [&](int c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = ok0 && c * 16 + cq * 4 + e < a.cout;
      v[e] = row8<V16>(rs, off + (c * 16 + e) * cstride, col, W2, (int)stored_span(a.y), ok);
      if (MASK == S2_MASK) mv[e] = row8<V16>(rm, moff + (c * 16 + e) * mcs, col, W2, (int)stored_span(a.m), ok);
      if (MASK == S2_FAR_MASK) mv[e] = s2_far8(far_row(c * 16 + cq * 4 + e), col, W2, ok);
    }
  };
  auto store_chunk = [&](int c) {
    uint4* dst = lds + (c & 1) * SD_BUF;
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[tid + 512 * k] = wv[k];
    dst[last_unit] = wv[3];
    uint4 g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      g[e] = fix8<V16>(v[e], off + (c * 16 + e) * cstride, col, W2, (int)stored_span(a.y));
      if (MASK) g[e] = mask8(g[e], MASK == S2_MASK ? fix8<V16>(mv[e], moff + (c * 16 + e) * mcs, col, W2, (int)stored_span(a.m)) : mv[e], a.slope);
    }
    uint2* half = reinterpret_cast<uint2*>(dst + unit) + (cq & 1);
    if (full || tail) half[0] = column_half(g, 0);
    if (full)
#pragma unroll
      for (int k = 1; k < 8; ++k) half[2 * k] = column_half(g, k);
  };

  f32x16 acc[8];                  // parity (pd, ph, pw)
#pragma unroll
  for (int p = 0; p < 8; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[p][i] = 0.f;

  load_weights(0);
  load_rows(0);
  store_chunk(0);
  for (int c = 0; c < a.nchunk; ++c) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (c + 1 < a.nchunk) {
      load_weights(c + 1);
      load_rows(c + 1);
    }
    const uint4* wl = lds + (c & 1) * SD_BUF + lane;
    const uint4* bl = lds + (c & 1) * SD_BUF + SD_W + (lane >> 5) * SD_CIG + wave * SD_PITCH + (lane & 31);
#pragma unroll
    for (int od = 0; od < 2; ++od)
#pragma unroll
      for (int oh = 0; oh < 2; ++oh) {
        const uint4 b0 = bl[(od * SD_ROWS + oh) * SD_PITCH], b1 = bl[(od * SD_ROWS + oh) * SD_PITCH + 1];
#pragma unroll
        for (int pd = od; pd < 2; ++pd)
#pragma unroll
          for (int ph = oh; ph < 2; ++ph) {
            const int kd = od ? 0 : 1 + pd, kh = oh ? 0 : 1 + ph, tap = kd * 9 + kh * 3;
            acc[pd * 4 + ph * 2] = mfma32(wl[(tap + 1) * 64], b0, acc[pd * 4 + ph * 2]);
            acc[pd * 4 + ph * 2 + 1] = mfma32(wl[(tap + 2) * 64], b0, acc[pd * 4 + ph * 2 + 1]);
            acc[pd * 4 + ph * 2 + 1] = mfma32(wl[tap * 64], b1, acc[pd * 4 + ph * 2 + 1]);
          }
      }
    if (c + 1 < a.nchunk) store_chunk(c + 1);
  }

  bf16_t* xs = dx + (int64_t)n * a.x.nstride;
  const __amdgpu_buffer_rsrc_t ro = row_rsrc(xs, (uint32_t)a.x.nstride * 2);
  const int W = a.x.w, H = a.x.h, ch = h0 + wave, w = 2 * (w0 + (lane & 31));
#pragma unroll
  for (int pd = 0; pd < 2; ++pd)
#pragma unroll
    for (int ph = 0; ph < 2; ++ph) {
      const int h = 2 * ch + ph;
      const int base = (2 * z + pd + a.x.hlo) * (int)a.x.plane + h * W + w;
      const bool in = h < H && w < W;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int ci = ci0 + acc_row(i, lane);
        const int vo = in && ci < a.cin ? 2 * (ci * (int)a.x.cstride + base) : ROW_OOB;
        const uint32_t pk = pack_bf16x2(acc[pd * 4 + ph * 2][i], acc[pd * 4 + ph * 2 + 1][i]);
        if (a.vec) {
          __builtin_amdgcn_raw_buffer_store_b32(pk, ro, vo, 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b16((short)(pk & 0xffffu), ro, vo, 0, 0);
          __builtin_amdgcn_raw_buffer_store_b16((short)(pk >> 16), ro, w + 1 < W ? vo == ROW_OOB ? ROW_OOB : vo + 2 : ROW_OOB, 0, 0);
        }
      }
    }
}

// ---------------------------------------------------------------------------------------------------- backward-filter
// Contraction over coarse voxels with both operands in NCDHW: rows = 32 output channels (A = g, 8 consecutive columns a lane),
// columns = 32 input channels (B = x at every second column: the even and the odd elements of 16 consecutive ones, taken apart
// with v_perm; even columns are tap kw = 1, odd ones kw = 2, and against g shifted by one column kw = 0), K = 16 coarse columns.
// The tap plane kd is a grid dimension (27 accumulator blocks do not fit); a workgroup's four wavefronts hold the 9 (kh,kw)
// blocks of 2 x 2 channel blocks (144 registers) and walk down the rows of a strip (32 coarse columns x a band of rows of one
// plane): fine row 2h is kh = 1 of g row h, fine row 2h + 1 is kh = 2 of it and kh = 0 of row h + 1, which stays in registers
// for the next step, so x and g are read once.  Rows pass through LDS (two buffers, one barrier a step); row pitches of 9 and 5
// units keep the 16-byte reads of neighbouring channels on different banks.
// Partial sums [chunk][27][co][ci] per chunk of strips, added in chunk order: identical bits on every run.
constexpr int SB_XP = 9, SB_GP = 5, SB_X = 2 * 64 * SB_XP, SB_BUF = SB_X + 64 * SB_GP;

template <int MASK, bool V16>
__global__ void __launch_bounds__(256, 2) s2_bwd_filter_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dy, const bf16_t* __restrict__ m,
                                                               float* __restrict__ part, float* __restrict__ part_db, S2Args a) {
  __shared__ uint4 lds[2 * SB_BUF];
  __shared__ float dbl[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cog = blockIdx.y / a.cigroups, cig = blockIdx.y % a.cigroups, kd = blockIdx.z, chunk = blockIdx.x;
  const int W = a.x.w, H = a.x.h, W2 = a.y.w, H2 = a.y.h;
  const bool want_db = kd == 1 && cig == 0;

  const int g_co = cog * 64 + (tid >> 2), g_piece = tid & 3;
  const int x_piece = tid & 7, x_ci = cig * 64 + (tid >> 3);
  int strip = chunk * a.strips_per_chunk;
  const int strip_end = min(strip + a.strips_per_chunk, a.nstrips);

  // position of the step whose rows are being FETCHED
  int n = 0, z = 0, w0 = 0, h = 0, hend = 0;
  bool xrow_ok = false;
  __amdgpu_buffer_rsrc_t rx = row_rsrc(x, 0), rg = row_rsrc(dy, 0), rm = rg;
  auto open_strip = [&]() {
    int t = strip;
    const int band = t % a.bands; t /= a.bands;
    w0 = (t % a.segs) * 32; t /= a.segs;
    z = t % a.y.d; n = t / a.y.d;
    h = band * a.band - 1;                       // first step of a strip: only g row h + 1 is fetched
    hend = min((band + 1) * a.band, H2);
    rx = row_rsrc(x + (int64_t)n * a.x.nstride, (uint32_t)a.x.nstride * 2);
    rg = row_rsrc(dy + (int64_t)n * a.y.nstride, (uint32_t)a.y.nstride * 2);
    if (MASK == S2_MASK) rm = row_rsrc(m + (int64_t)n * a.m.nstride, (uint32_t)a.m.nstride * 2);
    const int p = 2 * z + kd - 1;
    xrow_ok = a.x.doff + p >= 0;
  };

  uint4 xv[4], gv, mv;
  uint32_t ge = 0, me = 0;
  bool count_db = false;
  int xo = 0, go = 0, mo = 0, xc = 0, gc = 0;       // where the fetched groups lie: element offsets of their rows, columns
  auto fetch = [&](bool first) {
    xo = x_ci * (int)a.x.cstride + (2 * z + kd - 1 + a.x.hlo) * (int)a.x.plane + 2 * h * W;
    xc = 2 * w0 + 8 * x_piece;
    gc = w0 + 8 * g_piece;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ci = x_ci + 32 * (i & 1), row = 2 * h + (i >> 1);
      xv[i] = row8<V16>(rx, xo + 32 * (i & 1) * (int)a.x.cstride + (i >> 1) * W, xc, W, (int)stored_span(a.x), !first && xrow_ok && ci < a.cin && row < H);
    }
    const bool gok = g_co < a.cout && h + 1 < H2;
    go = g_co * (int)a.y.cstride + (z + a.y.hlo) * (int)a.y.plane + (h + 1) * W2;
    gv = row8<V16>(rg, go, gc, W2, (int)stored_span(a.y), gok);
    ge = row1(rg, go, w0 + 32, W2, gok && g_piece == 3);
    if (MASK == S2_FAR_MASK) {
      const bf16_t* row = m + (int64_t)n * a.m.nstride + (int64_t)g_co * a.m.cstride + (int64_t)(z + a.m.hlo) * a.m.plane + (int64_t)(h + 1) * W2;
      mv = s2_far8(row, gc, W2, gok);
      me = s2_far8(row, w0 + 32, min(w0 + 33, W2), gok && g_piece == 3).x;
    }
    if (MASK == S2_MASK) {
      mo = g_co * (int)a.m.cstride + (z + a.m.hlo) * (int)a.m.plane + (h + 1) * W2;
      mv = row8<V16>(rm, mo, gc, W2, (int)stored_span(a.m), gok);
      me = row1(rm, mo, w0 + 32, W2, gok && g_piece == 3);
    }
    count_db = h + 1 < hend;
  };
  float dbsum = 0.f;
  auto put = [&](int buf) {
    uint4* dst = lds + buf * SB_BUF;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dst[((i >> 1) * 64 + (tid >> 3) + 32 * (i & 1)) * SB_XP + x_piece] =
          fix8<V16>(xv[i], xo + 32 * (i & 1) * (int)a.x.cstride + (i >> 1) * W, xc, W, (int)stored_span(a.x));
    uint4 g = fix8<V16>(gv, go, gc, W2, (int)stored_span(a.y));
    uint32_t e = ge;
    if (MASK) {
      g = mask8(g, MASK == S2_MASK ? fix8<V16>(mv, mo, gc, W2, (int)stored_span(a.m)) : mv, a.slope);
      e = mask2(e, me, a.slope) & 0xffffu;
    }
    dst[SB_X + (tid >> 2) * SB_GP + g_piece] = g;
    if (g_piece == 3) *reinterpret_cast<uint32_t*>(dst + SB_X + (tid >> 2) * SB_GP + 4) = e;
    if (want_db && count_db) {
      const uint32_t d[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) dbsum += __uint_as_float(d[k] << 16) + __uint_as_float(d[k] & 0xffff0000u);
    }
  };

  f32x16 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
  uint4 G[2], Gs[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) G[k] = Gs[k] = uint4{0u, 0u, 0u, 0u};

  const int cow = wave >> 1, ciw = wave & 1, lc = lane & 31, half = lane >> 5;
  // g has no row behind the volume's last and no column behind its last: the zeros that stand for them must not meet the last row and
  // column of x, which may be infinite.  A step without a next row leaves its products out; for kw = 0 the last odd column of x is
  // cut, with a mask set when a strip opens.  With V16 it can only be the last element of a lane's eight.  (64 -> 128 channels on 64^3,
  // call with a mask 40.2 -> 40.8 us, without 37.1 -> 37.6.)
  constexpr int CUT0 = V16 ? 3 : 0;
  uint32_t cut[2][4];
  // a block of channels beyond the tensors' has no products and leaves no sums (three passes of 16 -> 26 channels on 16x128x104, masked:
  // 67 -> 64 us)
  const bool block_used = __builtin_amdgcn_readfirstlane(cog * 64 + cow * 32 < a.cout && cig * 64 + ciw * 32 < a.cin);
  bool live = strip < strip_end;
  bool first = true, cur_first = true;
  if (live) {
    open_strip();
    fetch(true);
    put(0);
  }
  int buf = 0;
  while (live) {
    __syncthreads();
    cur_first = first;
    const bool cur_next = h + 1 < H2;
    if (cur_first) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int last = W2 - 1 - (w0 + 16 * k + 8 * half);      // element of the last column, if it is among this lane's eight
#pragma unroll
        for (int i = CUT0; i < 4; ++i) cut[k][i] = last == 2 * i ? 0xffff0000u : last == 2 * i + 1 ? 0xffffu : 0xffffffffu;
      }
    }
    // next step
    bool more = true;
    if (h + 1 < hend) {
      ++h;
      first = false;
    } else if (++strip < strip_end) {
      open_strip();
      first = true;
    } else {
      more = false;
    }
    if (more) fetch(first);
    const uint4* xl = lds + buf * SB_BUF + (ciw * 32 + lc) * SB_XP;
    const uint4* gl = lds + buf * SB_BUF + SB_X + (cow * 32 + lc) * SB_GP;
    uint4 N[2], Ns[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      N[k] = gl[2 * k + half];
      const uint32_t nx = *reinterpret_cast<const uint32_t*>(gl + 2 * k + half + 1);
      Ns[k] = uint4{__builtin_amdgcn_alignbit(N[k].y, N[k].x, 16), __builtin_amdgcn_alignbit(N[k].z, N[k].y, 16),
                    __builtin_amdgcn_alignbit(N[k].w, N[k].z, 16), __builtin_amdgcn_alignbit(nx, N[k].w, 16)};
    }
    if (!cur_first && block_used) {
#pragma unroll
      for (int row = 0; row < 2; ++row)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const uint4 p0 = xl[row * 64 * SB_XP + 4 * k + 2 * half], p1 = xl[row * 64 * SB_XP + 4 * k + 2 * half + 1];
          const uint4 E = {__builtin_amdgcn_perm(p0.y, p0.x, 0x05040100u), __builtin_amdgcn_perm(p0.w, p0.z, 0x05040100u),
                           __builtin_amdgcn_perm(p1.y, p1.x, 0x05040100u), __builtin_amdgcn_perm(p1.w, p1.z, 0x05040100u)};
          const uint4 O = {__builtin_amdgcn_perm(p0.y, p0.x, 0x07060302u), __builtin_amdgcn_perm(p0.w, p0.z, 0x07060302u),
                           __builtin_amdgcn_perm(p1.y, p1.x, 0x07060302u), __builtin_amdgcn_perm(p1.w, p1.z, 0x07060302u)};
          const uint4 P = {V16 ? O.x : O.x & cut[k][0], V16 ? O.y : O.y & cut[k][1], V16 ? O.z : O.z & cut[k][2], O.w & cut[k][3]};
          const int kh = row == 0 ? 1 : 2;
          acc[kh * 3 + 1] = mfma32(G[k], E, acc[kh * 3 + 1]);
          acc[kh * 3 + 2] = mfma32(G[k], O, acc[kh * 3 + 2]);
          acc[kh * 3] = mfma32(Gs[k], P, acc[kh * 3]);
          if (row == 1 && cur_next) {
            acc[1] = mfma32(N[k], E, acc[1]);
            acc[2] = mfma32(N[k], O, acc[2]);
            acc[0] = mfma32(Ns[k], P, acc[0]);
          }
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      G[k] = N[k];
      Gs[k] = Ns[k];
    }
    if (more) put(buf ^ 1);
    buf ^= 1;
    live = more;
  }

  const int cop = a.cogroups * 64, cip = a.cigroups * 64;
  float* pp = part + (((int64_t)chunk * 27 + kd * 9) * cop + cog * 64 + cow * 32) * cip + cig * 64 + ciw * 32 + lc;
  if (block_used)
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) pp[((int64_t)t * cop + acc_row(i, lane)) * cip] = acc[t][i];
  if (want_db) {
    dbl[tid] = dbsum;
    __syncthreads();
    if (tid < 64) part_db[(int64_t)chunk * cop + cog * 64 + tid] = (dbl[4 * tid] + dbl[4 * tid + 1]) + (dbl[4 * tid + 2] + dbl[4 * tid + 3]);
  }
}

// ------------------------------------------------------------------------------------------------------------- host
// Byte offsets inside a sample are 32-bit (channels are counted up to the next multiple of 64).
static bool s2_offsets_fit(const h3d_tensor* t, int bits) { return cdiv(t->c, 64) * 64 * make_geo(t).cstride < ((int64_t)1 << bits) && stored_span(make_geo(t)) >= 8; }
// x: fine side, y: coarse side.  A saved output may store more or fewer halo planes than the gradient it belongs to: its own test
// (s2_mask_fits) leaves it four times the room, and one that does not pass is read by the S2_FAR_MASK form.
static bool s2_mask_fits(const h3d_tensor* m) { return s2_offsets_fit(m, 30); }
bool s2_mfma_supported(const h3d_tensor* x, const h3d_tensor* y) {
  if (x->dtype != H3D_BF16) return false;
  if (x->n < 1 || x->c < 1 || y->c < 1 || y->d < 1 || x->h < 1 || x->w < 1) return false;
  if (!s2_offsets_fit(x, 30) || !s2_offsets_fit(y, 28)) return false;
  return (int64_t)x->n * y->d * cdiv(y->h, 4) * cdiv(y->w, 32) < ((int64_t)1 << 28) && cdiv(x->c, 64) * cdiv(y->c, 64) <= 65535;
}

struct S2BfPlan { int segs, band, bands, nstrips, per, nchunks, cogroups, cigroups; };
// chunks: two workgroups per CU (256 CUs).  A step is shorter than the latency of the rows it prefetches, so a second workgroup
// pays although it doubles the partial sums: one per CU 46 us (+ 7 for the reduction), two 33 (+ 10) at the size above.
static S2BfPlan s2_bf_plan(const h3d_tensor* x, const h3d_tensor* y) {
  S2BfPlan p;
  p.cogroups = (int)cdiv(y->c, 64); p.cigroups = (int)cdiv(x->c, 64);
  p.segs = (int)cdiv(y->w, 32);
  const int64_t groups = (int64_t)3 * p.cogroups * p.cigroups;
  // Small layers: bands of 8 or 4 rows, shorter chains of steps in more workgroups.  Each band costs a step more, and its chunk 442 KB of
  // partial sums.  us, bands of 16, 8 and 4 rows: 16->16 on 16x32x32 (24 workgroups at 16 rows) 24.8, 17.0, 14.2; 64->64 on 32^3 (48) 28.0, 23.4,
  // 24.7; 16->8 on 32x64x64 (96) 27.1, 21.6, 23.5; 4->64 on 16x128x128 (192), 16 and 8: 31, 34.
  for (p.band = 16;; p.band /= 2) {
    p.bands = (int)cdiv(y->h, p.band);
    p.nstrips = x->n * y->d * p.segs * p.bands;
    if (p.band == 4 || p.nstrips * groups >= (p.band == 16 ? 160 : 64)) break;
  }
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>(p.nstrips, 512 / groups));
  p.per = (int)cdiv(p.nstrips, want);
  p.nchunks = (int)cdiv(p.nstrips, p.per);
  return p;
}

static size_t s2_wp_bytes(int rows, int contraction, int step) { return up256((size_t)cdiv(rows, 32) * cdiv(contraction, step) * (step / 16) * 27 * 1024); }

size_t s2_mfma_ws_bytes(int op, const h3d_tensor* x, const h3d_tensor* y) {
  if (op == H3D_OP_FWD) return s2_wp_bytes(y->c, x->c, 32);
  if (op == H3D_OP_BWD_DATA) return s2_wp_bytes(x->c, y->c, 16);
  const S2BfPlan p = s2_bf_plan(x, y);
  return up256((size_t)p.nchunks * 27 * p.cogroups * p.cigroups * 4096 * sizeof(float)) + up256((size_t)p.nchunks * p.cogroups * 64 * sizeof(float));
}

static S2Args s2_args(const h3d_tensor* x, const h3d_tensor* y, const h3d_tensor* m, float slope) {
  S2Args a;
  memset(&a, 0, sizeof(a));
  a.x = make_geo(x); a.y = make_geo(y); a.m = m ? make_geo(m) : a.y;
  a.cin = x->c; a.cout = y->c; a.slope = slope;
  return a;
}
static bool rows16(const h3d_tensor* t) { return t->w % 8 == 0 && (uintptr_t)t->data % 16 == 0; }
static unsigned xcd_grid(int n) { return (unsigned)(cdiv(n, 8) * 8); }

template <int NCO, int CB, bool V16>
static h3d_status s2_launch_fwd(void* handle, const h3d_tensor* x, const uint4* wp, const float* bias, h3d_tensor* y, const S2Args& a, hipStream_t s) {
  static bool lds_set = false;
  H3D_TRY(raise_lds_limit(handle, s2_fwd_kernel<NCO, CB, V16>, SF_LDS, &lds_set));
  hipLaunchKernelGGL((s2_fwd_kernel<NCO, CB, V16>), dim3(xcd_grid(a.ntiles), (unsigned)cdiv(y->c, 32 * NCO * CB)), dim3(256), SF_LDS, s,
                     (const bf16_t*)x->data, wp, bias, (bf16_t*)y->data, a);
  note_kernel(handle, "s2_fwd_kernel<%d,%d,%d>", NCO, CB, (int)V16);
  return launch_status(handle, "conv3d_s2_fwd");
}

h3d_status s2_mfma_fwd(void* handle, const h3d_tensor* x, const void* w, const float* bias, h3d_tensor* y, float slope, void* ws, hipStream_t s) {
  S2Args a = s2_args(x, y, nullptr, slope);
  a.nchunk = 2 * (int)cdiv(x->c, 32);
  a.tiles_w = (int)cdiv(y->w, 32); a.tiles_h = (int)cdiv(y->h, 4);
  a.ntiles = y->n * y->d * a.tiles_h * a.tiles_w;
  a.vec = y->w % 2 == 0 && (uintptr_t)y->data % 4 == 0;
  taps_pack(taps_pack_job(w, ws, x->c, y->c, TAPS_FWD, a.nchunk, 27), s);
  const uint4* wp = (const uint4*)ws;
  const bool v16 = rows16(x);
  if (y->c > 64) return v16 ? s2_launch_fwd<2, 2, true>(handle, x, wp, bias, y, a, s) : s2_launch_fwd<2, 2, false>(handle, x, wp, bias, y, a, s);
  if (y->c > 32) return v16 ? s2_launch_fwd<1, 2, true>(handle, x, wp, bias, y, a, s) : s2_launch_fwd<1, 2, false>(handle, x, wp, bias, y, a, s);
  return v16 ? s2_launch_fwd<1, 1, true>(handle, x, wp, bias, y, a, s) : s2_launch_fwd<1, 1, false>(handle, x, wp, bias, y, a, s);
}

template <int MASK, bool V16>
static h3d_status s2_launch_bd(void* handle, const h3d_tensor* dy, const h3d_tensor* m, const uint4* wp, h3d_tensor* dx, const S2Args& a, hipStream_t s) {
  static bool lds_set = false;
  H3D_TRY(raise_lds_limit(handle, s2_bwd_data_kernel<MASK, V16>, SD_LDS, &lds_set));
  hipLaunchKernelGGL((s2_bwd_data_kernel<MASK, V16>), dim3(xcd_grid(a.ntiles), (unsigned)cdiv(dx->c, 32)), dim3(512), SD_LDS, s,
                     (const bf16_t*)dy->data, (const bf16_t*)(m ? m->data : nullptr), wp, (bf16_t*)dx->data, a);
  note_kernel(handle, "s2_bwd_data_kernel<%d,%d>", MASK, (int)V16);
  return launch_status(handle, "conv3d_s2_bwd_data");
}

h3d_status s2_mfma_bwd_data(void* handle, const h3d_tensor* dy, const h3d_tensor* y, const void* w, h3d_tensor* dx, float slope, void* ws, hipStream_t s) {
  S2Args a = s2_args(dx, dy, y, slope);
  a.nchunk = (int)cdiv(dy->c, 16);
  a.tiles_w = (int)cdiv(dy->w, 32); a.tiles_h = (int)cdiv(dy->h, 8);
  a.ntiles = dy->n * dy->d * a.tiles_h * a.tiles_w;
  a.vec = dx->w % 2 == 0 && (uintptr_t)dx->data % 4 == 0;
  taps_pack(taps_pack_job(w, ws, dx->c, dy->c, TAPS_TRANSPOSED, a.nchunk, 27), s);
  const uint4* wp = (const uint4*)ws;
  const bool v16 = rows16(dy) && (!y || rows16(y));
  if (y && !s2_mask_fits(y)) return s2_launch_bd<S2_FAR_MASK, false>(handle, dy, y, wp, dx, a, s);
  if (y) return v16 ? s2_launch_bd<S2_MASK, true>(handle, dy, y, wp, dx, a, s) : s2_launch_bd<S2_MASK, false>(handle, dy, y, wp, dx, a, s);
  return v16 ? s2_launch_bd<S2_NO_MASK, true>(handle, dy, y, wp, dx, a, s) : s2_launch_bd<S2_NO_MASK, false>(handle, dy, y, wp, dx, a, s);
}

h3d_status s2_mfma_bwd_filter(void* handle, const h3d_tensor* x, const h3d_tensor* dy, const h3d_tensor* y, float* dw, float* db, float slope,
                              void* ws, hipStream_t s) {
  S2Args a = s2_args(x, dy, y, slope);
  const S2BfPlan p = s2_bf_plan(x, dy);
  a.segs = p.segs; a.band = p.band; a.bands = p.bands; a.nstrips = p.nstrips; a.strips_per_chunk = p.per; a.nchunks = p.nchunks;
  a.cogroups = p.cogroups; a.cigroups = p.cigroups;
  float* part = (float*)ws;
  const int cop = p.cogroups * 64, cip = p.cigroups * 64;
  float* part_db = (float*)((char*)ws + up256((size_t)p.nchunks * 27 * cop * cip * sizeof(float)));
  const bool v16 = rows16(x) && rows16(dy) && (!y || rows16(y));
  const dim3 grid((unsigned)p.nchunks, (unsigned)(p.cogroups * p.cigroups), 3);
#define S2_BF(M, V) hipLaunchKernelGGL((s2_bwd_filter_kernel<M, V>), grid, dim3(256), 0, s, (const bf16_t*)x->data, (const bf16_t*)dy->data, \
                                       (const bf16_t*)(y ? y->data : nullptr), part, part_db, a)
  const int mask = !y ? S2_NO_MASK : s2_mask_fits(y) ? S2_MASK : S2_FAR_MASK;
  if (mask == S2_FAR_MASK) S2_BF(S2_FAR_MASK, false);
  else if (mask == S2_MASK) { if (v16) S2_BF(S2_MASK, true); else S2_BF(S2_MASK, false); }
  else { if (v16) S2_BF(S2_NO_MASK, true); else S2_BF(S2_NO_MASK, false); }
#undef S2_BF
  note_kernel(handle, "s2_bwd_filter_kernel<%d,%d>", mask, (int)(v16 && mask != S2_FAR_MASK));
  taps_reduce(part, part_db, dw, db, 27, x->c, dy->c, cip, cop, p.nchunks, p.nchunks, 1.f, s);
  return launch_status(handle, "conv3d_s2_bwd_filter");
}

}  // namespace h3d
