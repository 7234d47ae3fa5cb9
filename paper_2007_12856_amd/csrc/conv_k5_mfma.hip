// 5x5x5 convolution of bf16 tensors on the matrix cores: forward, backward-data (the same kernel on g = dz act'(z) with the filter
// reversed and transposed) and backward-filter, for any width and alignment.  Bound by the matrix cores: 2 * 125 * Cin * Cout flop per
// voxel against 2 (Cin + Cout) bytes, 32 -> 32 channels: 2000 flop/B.
#include <algorithm>

#include "rowload.h"
#include "taps.h"

namespace h3d {

struct K5MArgs {
  Geo in, out;              // staged tensor (x or g), written tensor (backward-filter: out = g)
  int pmin, pmax;           // planes of `in` inside the volume and stored, interior-relative
  int cin, cout;            // channels of the contraction / of the result (backward-filter: of x / of g)
  int nchunk;               // 16-channel chunks of the contraction
  int tiles_w, tiles_h, ntiles;
  float slope;
  int vec;                  // result rows are 4-byte aligned pairs
  // backward-filter.  Chunks from `half` on contract with the second part of a gradient in two parts, `neg` elements behind the first.
  int segs, chunks, half, cobs, cibs;
  int64_t neg;
};

// --------------------------------------------------------------------------------------------- forward / backward-data
// A workgroup of 8 wavefronts owns 8 RB rows x 32 columns of one output plane and 32 output channels; a wavefront RB rows (RB
// accumulator blocks of v_mfma_f32_32x32x16_bf16: output channels x voxels of a row, K = 16 input channels of one tap).  Per stage =
// (16-channel chunk, kd) the (8 RB + 4) x 36 patch of that input plane is transposed into LDS (16-byte units of 8 channels) and the
// stage's 25 weight fragments are copied beside it; the rows of the next stage are requested as whole 16-byte pieces of 8 columns
// (8 requests a thread and stage) and written to the other buffer behind this stage's products, one barrier a stage.  Per kw a
// wavefront reads RB + 4 row fragments and 5 weight fragments for 5 RB products.
// 32 -> 32 channels on 32 x 128 x 128 (134 GFlop), call with its packing: 185 -> 126 us (1.06 PFLOP/s; 64 -> 64: 587 -> 440, 1.22);
// matrix pipes busy 51 % at 2.0 GHz.  Two rounds of workgroups with ten stages each: first fetch and result stand out.  Taller
// wavefront tiles (8 rows, one wavefront a SIMD) measured 174 us.
template <int RB>
struct K5Tile {
  static constexpr int ROWS = 8 * RB + 4, PITCH = 46, CIG = ROWS * PITCH, WU = 25 * 64, BUF = 2 * CIG + WU, ITEMS = 2 * ROWS * 6;
  static constexpr int TRASH = 2 * BUF;                    // 64 units that nobody reads
  static constexpr size_t LDS = (size_t)(2 * BUF + 64) * 16;
  static_assert(ITEMS <= 512, "one column group a thread");
};

template <int RB, bool V16>
__global__ void __launch_bounds__(512) k5_conv_mfma_kernel(const bf16_t* __restrict__ in, const uint4* __restrict__ wp, const float* __restrict__ bias,
                                                           bf16_t* __restrict__ out, K5MArgs a) {
  using T = K5Tile<RB>;
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the workgroups of one XCD (linear index mod 8) take a contiguous run of tiles: neighbours share halo rows in its L2
  int t = (blockIdx.x & 7) * (gridDim.x / 8) + (blockIdx.x >> 3);
  if (t >= a.ntiles) return;
  const int w0 = (t % a.tiles_w) * 32; t /= a.tiles_w;
  const int h0 = (t % a.tiles_h) * 8 * RB; t /= a.tiles_h;
  const int p = t % a.out.d, n = t / a.out.d, blk = blockIdx.y;
  const int W = a.in.w, H = a.in.h;
  const bf16_t* is = in + (int64_t)n * a.in.nstride;
  const int cstride = (int)a.in.cstride;

  // ---- staging plan: one (channel group, row, group of 8 columns from w0 - 8 on) a thread; of the first and the last group
  //      two columns each lie in the patch
  const int cg = tid % 6, row = (tid / 6) % T::ROWS, cig = tid / (6 * T::ROWS);
  const int h = h0 + row - 2, col = w0 - 8 + 8 * cg;
  const bool ok = tid < T::ITEMS && h >= 0 && h < H && col >= 0;
  const int off = cig * 8 * cstride + h * W;
  const int unit = cig * T::CIG + row * T::PITCH + 9 * cg - 6;
  uint4 v[8], wv0, wv1, wv2, wv3;
  const uint4* wb = wp + (int64_t)blk * a.nchunk * 125 * 64;
  // Descriptor of the chunk's channels: byte offsets inside 16 channels are 32-bit whatever the sample's size.  A last chunk of fewer than
  // 8 elements begins as far before its own as a 16-byte load needs.
  auto chunk_base = [&](int c, int pp, int& o, int& span) -> int64_t {
    const int64_t own = (int64_t)c * 16 * cstride, base = V16 ? own : min(own, stored_span(a.in) - 8);
    const int before = (int)(own - base);
    span = (int)min(stored_span(a.in) - base, (int64_t)16 * cstride + before);
    o = off + before + (pp + a.in.hlo) * (int)a.in.plane;
    return base;
  };
  auto load_stage = [&](int c, int pp) {
    const int kd = pp - p + 2;
    const uint4* ws = wb + ((int64_t)c * 125 + kd * 25) * 64 + tid;
    wv0 = ws[0];
    wv1 = ws[512];
    wv2 = ws[1024];
    wv3 = ws[min(1536, T::WU - 1 - tid)];
    int o, span;
    const int64_t base = chunk_base(c, pp, o, span);
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(is + base, (uint32_t)span * 2);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = row8<V16>(rs, o + e * cstride, col, W, span, ok && c * 16 + cig * 8 + e < a.cin);
  };
  // no branches: they would cut the schedule of the products these stores are spread over
  auto store_weights = [&](int buf) {
    uint4* wd = lds + buf * T::BUF + 2 * T::CIG + tid;
    wd[0] = wv0;
    wd[512] = wv1;
    wd[1024] = wv2;
    lds[tid + 1536 < T::WU ? buf * T::BUF + 2 * T::CIG + tid + 1536 : T::TRASH + lane] = wv3;
  };
  auto store_rows = [&](int c, int pp, int buf) {
    int o, span;
    chunk_base(c, pp, o, span);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = fix8<V16>(v[e], o + e * cstride, col, W, span);
    const int base = buf * T::BUF + unit;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool in_patch = tid < T::ITEMS && (k >= 6 || cg > 0) && (k < 2 || cg < 5);
      lds[in_patch ? base + k : T::TRASH + lane] = column_unit(v, k);
    }
  };

  f32x16 acc[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[r][i] = 0.f;

  // unit of column w0 - 2 + lane % 32 + kw in its row: eight columns and a gap, so that the 8 units a thread writes and those of its
  // neighbours (9 apart, rows 46 apart) lie on different banks
  int bcol[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) bcol[k] = (lane & 31) + k + ((lane & 31) + k + 6) / 8;
  const int p0 = max(p - 2, a.pmin), p1 = min(p + 3, a.pmax);      // input planes of this output plane
  const int nst = p1 > p0 ? a.nchunk * (p1 - p0) : 0;
  if (nst) {
    load_stage(0, p0);
    store_rows(0, p0, 0);
    store_weights(0);
  }
  int c = 0, pp = p0;
  for (int s = 0; s < nst; ++s) {
    __syncthreads();
    int cn = c, pn = pp + 1;
    if (pn == p1) {
      pn = p0;
      ++cn;
    }
    // (behind the last stage the request and the stores go nowhere that is read: the last rows again, into the other buffer)
    const bool more = s + 1 < nst;
    const int cl = more ? cn : c, pl = more ? pn : pp;
    load_stage(cl, pl);
    const uint4* bl = lds + (s & 1) * T::BUF + (lane >> 5) * T::CIG + wave * RB * T::PITCH;
    const uint4* wl = lds + (s & 1) * T::BUF + 2 * T::CIG + lane;
    // row fragments are refilled for the next kw as soon as their last product has been issued, weight fragments a kw ahead
    uint4 B[RB + 4], A[2][5];
#pragma unroll
    for (int kh = 0; kh < 5; ++kh) A[0][kh] = wl[kh * 5 * 64];
#pragma unroll
    for (int r = 0; r < RB + 4; ++r) B[r] = bl[r * T::PITCH + bcol[0]];
#pragma unroll
    for (int kw = 0; kw < 5; ++kw) {
      if (kw == 3) store_rows(cl, pl, (s + 1) & 1);
      if (kw == 4) store_weights((s + 1) & 1);
#pragma unroll
      for (int r = 0; r < RB + 4; ++r) {
        if (r < 5 && kw + 1 < 5) A[(kw + 1) & 1][r] = wl[(r * 5 + kw + 1) * 64];
#pragma unroll
        for (int kh = 0; kh < 5; ++kh)
          if (r - kh >= 0 && r - kh < RB) acc[r - kh] = mfma32(A[kw & 1][kh], B[r], acc[r - kh]);
        if (kw + 1 < 5) B[r] = bl[r * T::PITCH + bcol[kw + 1]];
      }
#pragma unroll
      for (int i = 0; i < 5 * RB; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x326, 3, 0);      // up to three of: VALU, SALU, memory read, LDS
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    c = cn;
    pp = pn;
  }

  // ---- result: bias, activation; the rows of a block of 32 channels through one descriptor
  const int j = lane & 31, WO = a.out.w;
  const bool odd = lane & 1;
  const int64_t obase = (int64_t)n * a.out.nstride + (int64_t)blk * 32 * a.out.cstride + (int64_t)(p + a.out.hlo) * a.out.plane;
  const __amdgpu_buffer_rsrc_t ro = row_rsrc(out + obase, 0x7fffffffu);
  const int ocs = (int)a.out.cstride;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int hh = h0 + wave * RB + r;
    float f[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int co = blk * 32 + acc_row(q, lane);
      float s = acc[r][q] + ((bias && co < a.cout) ? bias[co] : 0.f);
      if (!(s > 0.f)) s *= a.slope;
      f[q] = s;
    }
    if (a.vec) {        // neighbouring lanes swap one value: a lane stores two neighbouring voxels of one channel
      const int w = w0 + j - (odd ? 1 : 0);
      const bool inside = hh < H && w < WO;
#pragma unroll
      for (int q = 0; q < 16; q += 2) {
        const int cl = acc_row(q, lane) + (odd ? 1 : 0);
        const float give = odd ? f[q] : f[q + 1];
        const float got = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(give), 0xB1, 0xF, 0xF, true));
        const uint32_t pk = odd ? pack_bf16x2(got, f[q + 1]) : pack_bf16x2(f[q], got);
        __builtin_amdgcn_raw_buffer_store_b32(pk, ro, inside && blk * 32 + cl < a.cout ? 2 * (cl * ocs + hh * WO + w) : ROW_OOB, 0, 0);
      }
    } else {
      const int w = w0 + j;
      const bool inside = hh < H && w < WO;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int cl = acc_row(q, lane);
        __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(f[q]), ro, inside && blk * 32 + cl < a.cout ? 2 * (cl * ocs + hh * WO + w) : ROW_OOB, 0, 0);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------------ backward-filter
// Contraction over voxels, both operands in NCDHW: rows = 32 output channels (A = g, 8 consecutive columns a lane), columns = 32 input
// channels (B = x shifted by kw: the 12 columns around a lane's 8 are read once, the odd shifts made with v_alignbit), K = 16 columns.
// The wavefront kh of a group of five holds the five kw blocks of its kh (80 registers) for one kd; a group walks down the rows of a
// 64-column segment, one x row (ring of seven) and one g row (ring of three) a step, copied to LDS two steps ahead, one barrier a
// step.  Needs rows of whole 16-byte pieces in both tensors (other widths come as padded copies).  Five wavefronts do not divide
// over four SIMDs, so a workgroup is THREE such groups (15 wavefronts: 4, 4, 4, 3 of them on a SIMD, at most 128 registers each), each
// with its own run of rows; their sums are added in order through LDS, so that one partial tile leaves a workgroup.
// Partial sums [chunk][125][co][ci] (taps.hip).  32 -> 32 channels on 32 x 128 x 128, call without a mask and with the reduction: 375
// -> 165 us; a mask adds its copy (20); 64 -> 64: 1007 -> 563, 0.95 PFLOP/s.  Without four of the five products 95 us remain: the wavefronts of a
// SIMD leave the barrier together and wait for the LDS together, so reads and products of a step hardly overlap; without the copies
// 129, so they are not it.  Two groups of wavefronts instead of three (10 of them, more registers): 168.
constexpr int KF_SEG = 64, KF_XP = 10, KF_X = 32 * KF_XP, KF_G = 32 * 8, KF_XS = 7, KF_GS = 3, KF_PART = KF_XS * KF_X + KF_GS * KF_G + 64;
constexpr int KF_GROUPS = 3;      // groups of five wavefronts in a workgroup
constexpr size_t KF_LDS = (size_t)KF_GROUPS * KF_PART * 16 > 81 * 320 * 4 ? (size_t)KF_GROUPS * KF_PART * 16 : 81 * 320 * 4;      // (and 100 KB of accumulators at the end)

__global__ void __launch_bounds__(320 * KF_GROUPS) k5_bwf_rows_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ g, float* __restrict__ part,
                                                          float* __restrict__ part_db, K5MArgs a) {
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63, lc = lane & 31, lh = lane >> 5;
  const int grp = __builtin_amdgcn_readfirstlane(tid / 320), t320 = tid % 320, kh = __builtin_amdgcn_readfirstlane(t320 >> 6);
  // an XCD (linear index mod 8) takes an eighth of the list (chunk, channel block, kd): a chunk's kd planes and channel blocks read the
  // same rows
  const int per_chunk = 5 * a.cobs * a.cibs, q = (int)(blockIdx.x & 7) * (int)(gridDim.x / 8) + (int)(blockIdx.x >> 3);
  const int chunk = q / per_chunk, kd = q % per_chunk % 5, blk = q % per_chunk / 5;
  if (chunk >= a.chunks) return;
  const int run = chunk >= a.half ? chunk - a.half : chunk;
  if (chunk >= a.half) g += a.neg;
  const int cob = blk / a.cibs, cib = blk % a.cibs;
  const int H = a.in.h, W = a.in.w;
  uint4* xl = lds + grp * KF_PART;
  uint4* gl = xl + KF_XS * KF_X;
  const uint32_t x_addr = lds_addr_of(xl) + kh * 1024, g_addr = lds_addr_of(gl) + kh * 1024, trash = lds_addr_of(gl + KF_GS * KF_G);

  // ---- this group's run of rows: flat index over (sample, output plane with a valid x plane, segment, row)
  const int q0 = max(0, a.pmin + 2 - kd), q1 = min(a.out.d, a.pmax + 2 - kd);
  const int planes = max(q1 - q0, 0);
  const int total = a.out.n * planes * a.segs * H;
  const int per = (total + KF_GROUPS * a.half - 1) / (KF_GROUPS * a.half);
  // steps of a run: its rows, and four more wherever a column of rows starts (the first x rows of the window)
  auto run_steps = [&](int gi) -> int {
    const int r0 = min(total, (run * KF_GROUPS + gi) * per), r1 = min(total, r0 + per);
    return r1 > r0 ? (r1 - r0) + 4 * ((r1 - 1) / H - r0 / H + 1) : 0;
  };
  int steps = 0;
  for (int k = 0; k < KF_GROUPS; ++k) steps = max(steps, run_steps(k));
  const int r0 = min(total, (run * KF_GROUPS + grp) * per), r1 = min(total, r0 + per);
  const bool db_wave = kd == 2 && cib == 0 && kh == 2;

  // position of the step that is being FETCHED: g row h (from -4 on while the window fills), x row h + 2 of the window's last tap
  int left = r1 - r0;               // rows of the run from h on (all of them while the window fills)
  int colm = r0 / H, h = r0 % H, fill = 0, w0 = 0;
  bool live = r0 < r1;
  // one piece of x and (wavefronts 0..3; the last one copies zeros nowhere, so that all wait for the same count) one of g a lane.
  // g pieces lie permuted within their channel's row, so that neighbouring channels' reads of one piece meet different banks.
  // x pieces of channels 8-15 and 24-31 are rotated by one: rows of ten units repeat their banks after eight channels.
  const int x_c = t320 / KF_XP, x_piece = (t320 % KF_XP + KF_XP - ((t320 / KF_XP) >> 3 & 1)) % KF_XP, g_c = t320 >> 3, g_piece = (t320 & 7) ^ (g_c & 7);
  const bool xc_ok = cib * 32 + x_c < a.cin, gc_ok = kh < 4 && cob * 32 + g_c < a.cout;
  // What depends on the lane is settled when a column opens; a row adds a scalar offset, and a row outside the volume an empty
  // descriptor: the few instructions of a request stand between the barrier and the first product of every wavefront.
  h3d_i32x4 rx = lds_dma_rsrc(x, 0), rg = lds_dma_rsrc(g, 0);
  int xv = ROW_OOB, gv = ROW_OOB, xbytes = 0, gbytes = 0;
  auto open_column = [&]() {
    int t = colm;
    h -= 4;
    fill = 4;
    w0 = (t % a.segs) * KF_SEG; t /= a.segs;
    const int p = q0 + t % planes, n = t / planes;
    const int64_t xb = (int64_t)cib * 32 * a.in.cstride, gb = (int64_t)cob * 32 * a.out.cstride;
    xbytes = (int)((uint32_t)min(a.in.nstride - xb, 32 * a.in.cstride) * 2);
    gbytes = (int)((uint32_t)min(a.out.nstride - gb, 32 * a.out.cstride) * 2);
    rx = lds_dma_rsrc(x + (int64_t)n * a.in.nstride + xb, 0);
    rg = lds_dma_rsrc(g + (int64_t)n * a.out.nstride + gb, 0);
    const int xc = w0 - 8 + 8 * x_piece, gc = w0 + 8 * g_piece;
    xv = xc_ok && xc >= 0 && xc < W ? 2 * (x_c * (int)a.in.cstride + (p + kd - 2 + a.in.hlo) * (int)a.in.plane + xc) : ROW_OOB;
    gv = gc_ok && gc < W ? 2 * (g_c * (int)a.out.cstride + (p + a.out.hlo) * (int)a.out.plane + gc) : ROW_OOB;
  };
  auto fetch = [&](int xs, int gs) {
    const int xr = h + 2;
    const bool x_ok = live && xr >= 0 && xr < H, g_ok = live && fill == 0;
    rx[2] = x_ok ? xbytes : 0;
    rg[2] = g_ok ? gbytes : 0;
    lds_dma16_row(rx, x_addr + xs * KF_X * 16, xv, x_ok ? 2 * xr * W : 0);
    lds_dma16_row(rg, kh < 4 ? g_addr + gs * KF_G * 16 : trash, gv, g_ok ? 2 * h * W : 0);
  };
  auto advance = [&]() {
    ++h;
    if (fill > 0) {
      --fill;
    } else if (--left <= 0) {
      live = false;
    } else if (h == H) {
      ++colm;
      h = 0;
      open_column();
    }
  };

  f32x16 acc[5];
#pragma unroll
  for (int k = 0; k < 5; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
  float dbacc = 0.f;

  // two steps ahead: bit 0 of a step's flags says that it multiplies (not while a window fills, nor behind the run's end), bit 1
  // that the columns behind the segment's first 32 lie outside the volume
  auto flags = [&]() { return (live && fill == 0 ? 1 : 0) | (W - w0 <= 32 ? 2 : 0); };
  if (live) open_column();
  int f0 = flags();
  fetch(0, 0);
  advance();
  int f1 = flags();
  fetch(1, 1);
  int xs = 0, gs = 0;               // ring slots of the step that multiplies
  for (int s = 0; s < steps; ++s) {
    asm volatile("s_waitcnt vmcnt(2)" ::: "memory");      // this step's rows are there, the next one's may be on their way
    __syncthreads();
    const bool mul = f0 & 1, narrow = f0 & 2;
    advance();
    f0 = f1;
    f1 = flags();
    fetch(xs + 2 >= KF_XS ? xs + 2 - KF_XS : xs + 2, gs == 0 ? 2 : gs - 1);
    const int my_slot = xs, my_g = gs;
    xs = xs + 1 == KF_XS ? 0 : xs + 1;
    gs = gs == 2 ? 0 : gs + 1;
    if (mul) {
      // x row of tap kh: the newest row is tap 4's
      int sl = my_slot + 3 + kh;
      sl = sl >= KF_XS ? sl - KF_XS : sl;
      const bf16_t* xrow = reinterpret_cast<const bf16_t*>(xl + sl * KF_X + lc * KF_XP + (lc >> 3 & 1));
      const bf16_t* xlast = xrow + 64 + 8 * lh - (lh && (lc >> 3 & 1) ? 8 * KF_XP : 0);      // piece behind the last K-step's
      const bf16_t* grow = reinterpret_cast<const bf16_t*>(gl + my_g * KF_G + lc * 8);
      auto k_step = [&](int ks) {
        const int e0 = 16 * ks + 8 * lh;
        const uint4 A = *reinterpret_cast<const uint4*>(grow + 8 * ((2 * ks + lh) ^ (lc & 7)));
        u32x4 q = *reinterpret_cast<const u32x4*>(xrow + 8 + e0);
        asm("" : "+v"(q));      // one 16-byte read: taken apart into pairs of dwords it would put four lanes on a bank
        const uint32_t dm = *reinterpret_cast<const uint32_t*>(xrow + 6 + e0);
        const uint32_t dp = *reinterpret_cast<const uint32_t*>(ks == 3 ? xlast : xrow + 16 + e0);
        // dwords dm, q.x .. q.w, dp hold columns -2 .. 9 around the piece; o* start at an odd column
        const uint32_t o0 = __builtin_amdgcn_alignbit(q.x, dm, 16), o1 = __builtin_amdgcn_alignbit(q.y, q.x, 16);
        const uint32_t o2 = __builtin_amdgcn_alignbit(q.z, q.y, 16), o3 = __builtin_amdgcn_alignbit(q.w, q.z, 16);
        const uint32_t o4 = __builtin_amdgcn_alignbit(dp, q.w, 16);
        acc[0] = mfma32(A, uint4{dm, q.x, q.y, q.z}, acc[0]);
        acc[1] = mfma32(A, uint4{o0, o1, o2, o3}, acc[1]);
        acc[2] = mfma32(A, uint4{q.x, q.y, q.z, q.w}, acc[2]);
        acc[3] = mfma32(A, uint4{o1, o2, o3, o4}, acc[3]);
        acc[4] = mfma32(A, uint4{q.y, q.z, q.w, dp}, acc[4]);
      };
      // (two K-steps to a block without branches: the reads of one run beside the products of the other)
      k_step(0);
      k_step(1);
      if (!narrow) {
        k_step(2);
        k_step(3);
      }
      if (db_wave) {
#pragma unroll
        for (int ks = 0; ks < KF_SEG / 16; ++ks) {
          const uint4 A = *reinterpret_cast<const uint4*>(grow + 8 * ((2 * ks + lh) ^ (lc & 7)));
          const uint32_t d[4] = {A.x, A.y, A.z, A.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) dbacc += __uint_as_float(d[e] << 16) + __uint_as_float(d[e] & 0xffff0000u);
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (the copies that were still under way land before the LDS is used again)

  // ---- groups 1 and 2 hand their sums to group 0, in that order
  float* xch = reinterpret_cast<float*>(lds);
  for (int k = 1; k < KF_GROUPS; ++k) {
    __syncthreads();
    if (grp == k) {
#pragma unroll
      for (int q = 0; q < 5; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) xch[(q * 16 + i) * 320 + t320] = acc[q][i];
      xch[80 * 320 + t320] = dbacc;
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int q = 0; q < 5; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] += xch[(q * 16 + i) * 320 + t320];
      dbacc += xch[80 * 320 + t320];
    }
  }
  if (grp == 0) {
    const int cop = a.cobs * 32, cip = a.cibs * 32;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      float* pp = part + (((int64_t)chunk * 125 + kd * 25 + kh * 5 + q) * cop + cob * 32) * cip + cib * 32 + lc;
#pragma unroll
      for (int i = 0; i < 16; ++i) pp[(int64_t)acc_row(i, lane) * cip] = acc[q][i];
    }
    if (db_wave) {
      const float v = dbacc + __shfl_xor(dbacc, 32, 64);
      if (lh == 0) part_db[(int64_t)chunk * cop + cob * 32 + lc] = v;
    }
  }
}

// ----------------------------------------------------------------------------------------------------------------- host
// byte offsets inside a block of 32 channels are 32-bit
bool k5_mfma_supported(const h3d_tensor* x, const h3d_tensor* z) {
  return x->dtype == H3D_BF16 && make_geo(x).cstride < ((int64_t)1 << 25) && make_geo(z).cstride < ((int64_t)1 << 25) &&
         (int64_t)z->n * z->d * z->h * cdiv(z->w, 32) < ((int64_t)1 << 28);
}
size_t k5_mfma_wp_bytes(int rows, int contraction) { return (size_t)cdiv(rows, 32) * cdiv(contraction, 16) * 125 * 1024; }

// One round of workgroups (256 CUs, one each): more chunks only add partial sums; at least 8 rows for a group of wavefronts.  Chunks are
// spread over the XCDs by the list's order, whatever their number (a chunk an XCD, as it was, left five of eight XCDs idle with three
// chunks: masked 128->128 on 16x64x64 759 -> 284 us; 96->96 333 -> 178; with multiples of eight chunks 64->64 on 32x64x64 209 -> 154).
// Where that leaves few and long chains of products two rounds halve them for little time: error of dw against 64 bits, 128->128 on
// 16x64x64 (9 chains of 114 rows), 5.3e-7 -> 3.7e-7, 284 -> 296 us; on 32x96x96 1277 -> 1295 us; 64->64 on 64x128x128 1110 -> 1101.
// A gradient in two parts has its chunks split between them.
static int k5_bf_chunks(const h3d_tensor* x, int cout, int parts) {
  const int64_t groups = 5 * cdiv(cout, 32) * cdiv(x->c, 32);
  const int64_t rows = (int64_t)x->n * x->d * cdiv(x->w, KF_SEG) * x->h;
  int64_t full = std::max<int64_t>(parts, 256 / groups);
  if (KF_GROUPS * full < 64 && rows > 96 * KF_GROUPS * full) full = std::max<int64_t>(full, 512 / groups);
  return parts * (int)std::max<int64_t>(1, std::min<int64_t>(full / parts, cdiv(rows, 24)));
}
size_t k5_mfma_bf_bytes(const h3d_tensor* x, int cout, int parts) {
  return (size_t)k5_bf_chunks(x, cout, parts) * (125 * cdiv(cout, 32) * cdiv(x->c, 32) * 1024 + cdiv(cout, 32) * 32) * sizeof(float);
}

static K5MArgs k5m_args(const Geo& in, const Geo& out, int cin, int cout) {
  K5MArgs a;
  memset(&a, 0, sizeof(a));
  a.in = in; a.out = out; a.cin = cin; a.cout = cout;
  a.pmin = (int)std::max<int64_t>(-in.hlo, -in.doff);
  a.pmax = (int)std::min<int64_t>(in.ds - in.hlo, in.dglob - in.doff);
  a.nchunk = (int)cdiv(cin, 16);
  return a;
}
static bool rows16(const Geo& g, const void* p) { return g.w % 8 == 0 && g.cstride % 8 == 0 && (uintptr_t)p % 16 == 0; }

template <int RB, bool V16>
static h3d_status k5_launch(void* handle, const void* in, const void* wp, const float* bias, void* out, K5MArgs a, int n, hipStream_t s) {
  static bool lds_set = false;
  H3D_TRY(raise_lds_limit(handle, k5_conv_mfma_kernel<RB, V16>, K5Tile<RB>::LDS, &lds_set));
  a.tiles_w = (int)cdiv(a.out.w, 32); a.tiles_h = (int)cdiv(a.out.h, 8 * RB);
  a.ntiles = n * a.out.d * a.tiles_h * a.tiles_w;
  hipLaunchKernelGGL((k5_conv_mfma_kernel<RB, V16>), dim3((unsigned)(cdiv(a.ntiles, 8) * 8), (unsigned)cdiv(a.cout, 32)), dim3(512), K5Tile<RB>::LDS, s,
                     (const bf16_t*)in, (const uint4*)wp, bias, (bf16_t*)out, a);
  note_kernel(handle, "k5_conv_mfma_kernel<%d,%d>", RB, (int)V16);
  return hipGetLastError() == hipSuccess ? H3D_OK : fail(handle, H3D_EHIP, "conv3d_k5: launch failed");
}

TapsPackJob k5_mfma_pack(const void* w, void* wp, int cin, int cout, bool transposed) {
  return taps_pack_job(w, wp, cin, cout, transposed ? TAPS_REVERSED : TAPS_FWD, (int)cdiv(transposed ? cout : cin, 16), 125);
}

// in: the staged tensor (x, or g of backward-data, whose rows may be padded: in.w >= out.w); w null: wp is packed already
h3d_status k5_mfma_conv(void* handle, const Geo& in, const void* in_data, const void* w, int cin, int cout, bool transposed, const float* bias,
                        const h3d_tensor* out, float slope, void* wp, hipStream_t s) {
  const Geo go = make_geo(out);
  const int loopc = transposed ? cout : cin, resc = transposed ? cin : cout;
  K5MArgs a = k5m_args(in, go, loopc, resc);
  a.slope = slope;
  a.vec = go.w % 2 == 0 && go.cstride % 2 == 0 && (uintptr_t)out->data % 4 == 0;
  if (w) taps_pack(k5_mfma_pack(w, wp, cin, cout, transposed), s);
  const bool v16 = rows16(in, in_data);
  // 32-row tiles hold more products per staged row; with fewer than one of them per CU (or low volumes) 16-row tiles occupy more CUs
  const int64_t tall = (int64_t)out->n * go.d * cdiv(go.h, 32) * cdiv(go.w, 32) * cdiv(resc, 32);
  if (tall < 256 || go.h <= 16)
    return v16 ? k5_launch<2, true>(handle, in_data, wp, bias, out->data, a, out->n, s) : k5_launch<2, false>(handle, in_data, wp, bias, out->data, a, out->n, s);
  return v16 ? k5_launch<4, true>(handle, in_data, wp, bias, out->data, a, out->n, s) : k5_launch<4, false>(handle, in_data, wp, bias, out->data, a, out->n, s);
}

// gx, g: x and dz or their copies, rows of the same whole number of 16-byte pieces.  neg != 0: g is the first part of the gradient, the
// second one lies `neg` elements further on and counts `slope` times.
h3d_status k5_mfma_bwd_filter(void* handle, const h3d_tensor* x, const Geo& gx, const void* x_data, const Geo& g, const void* g_data, int64_t neg,
                              float slope, int cout, float* dw, float* db, void* ws, hipStream_t s) {
  K5MArgs a = k5m_args(gx, g, x->c, cout);
  a.segs = (int)cdiv(gx.w, KF_SEG);
  a.chunks = k5_bf_chunks(x, cout, neg ? 2 : 1);
  a.half = neg ? a.chunks / 2 : a.chunks; a.neg = neg;
  a.cobs = (int)cdiv(cout, 32); a.cibs = (int)cdiv(x->c, 32);
  float* part = (float*)ws;
  float* part_db = part + (size_t)a.chunks * 125 * a.cobs * a.cibs * 1024;
  const dim3 grid((unsigned)(cdiv((int64_t)a.chunks * 5 * a.cobs * a.cibs, 8) * 8));
  static bool lds_set = false;
  H3D_TRY(raise_lds_limit(handle, k5_bwf_rows_kernel, KF_LDS, &lds_set));
  hipLaunchKernelGGL(k5_bwf_rows_kernel, grid, dim3(320 * KF_GROUPS), KF_LDS, s, (const bf16_t*)x_data, (const bf16_t*)g_data, part, part_db, a);
  note_kernel(handle, "k5_bwf_rows_kernel");
  taps_reduce(part, part_db, dw, db, 125, x->c, cout, a.cibs * 32, a.cobs * 32, a.chunks, a.half, slope, s);
  return H3D_OK;
}

}  // namespace h3d
