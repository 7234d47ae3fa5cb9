// bf16 MFMA implicit-GEMM kernels for the 3x3x3 convolution passes on gfx950.
//
// Forward / backward-data (one kernel; backward-data is the forward correlation of
// g = dz * act'(z) with the weights transposed and reversed, Sec. III-C "BD"):
//   D[co][voxel] = sum_{tap, ci} Wp[co][tap, ci] * X[tap, ci][voxel]
//   * output channels sit on the MFMA rows (A operand = weights), voxels on the columns
//     (B operand = input patches), so one accumulator register of a wavefront covers 32
//     consecutive W positions of one channel: stores along W are contiguous;
//   * the contraction index is ordered (tap, ci) with ci fastest: the 8 bf16 a lane feeds to
//     v_mfma_f32_32x32x16_bf16 are 8 consecutive input channels of ONE voxel.  NCDHW keeps
//     channels a whole volume apart, so the input tile (with its halo) is transposed on its way
//     into LDS: 16-byte units of 8 channels, laid out [ci-group][d][h][w], read back with
//     conflict-free ds_read_b128 at the 27 shifted offsets;
//   * weights are pre-packed in exact fragment order ([co-block][ci-chunk][tap][lane][8], taps.h) and go
//     global -> registers (fully coalesced 1 KB per fragment, L1/L2 resident), requested several
//     (kd,kw) steps ahead, partly by the chunk before; they never touch LDS;
//   * a workgroup is 8 wavefronts: NCB blocks of 32 output channels x ND depth planes; each
//     wavefront owns 32 channels x 128 voxels (4 MFMA column blocks = 4 groups of h rows).  For a
//     fixed (kd,kw) the 12 (block, kh) products need only 3*RPB+3 distinct row fragments, so LDS
//     read traffic is about half of one fragment per MFMA;
//   * the ci loop runs in chunks of 16 channels with two LDS buffers: the global loads of chunk
//     c+1 are in flight while chunk c is multiplied.
#include <algorithm>
#include <type_traits>

#include "prep.h"

namespace h3d {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int CI_CHUNK = 16;
constexpr int WG_THREADS = 512;

struct MfmaArgs {
  Geo in, mask, out;
  int cin_k, cout_k, nchunks, ncoblk;
  int tiles_w, tiles_h, tiles_d, ntiles;
  float out_slope, mask_slope;
  // split of the input-channel chunks over blockIdx.z (small volumes with many channels would otherwise
  // occupy a handful of CUs): each split writes fp32 partial sums, a second kernel adds them in order
  int csplit, chunks_per_split;
  int pairs;        // output rows can be stored two voxels at a time (false only with a prepared input)
  float* part;      // [csplit][n][cout][stored planes][h][w], used when csplit > 1
  Geo yp;           // max-pooled result (POOL)
  bf16_t* ypool;
};

__device__ __forceinline__ uint32_t mask_pair(uint32_t v, uint32_t m, float slope) {
  // per bf16 half: keep v where the mask value is > 0, else v * slope (rounded to bf16)
  float v0 = __uint_as_float(v << 16), v1 = __uint_as_float(v & 0xffff0000u);
  float m0 = __uint_as_float(m << 16), m1 = __uint_as_float(m & 0xffff0000u);
  if (!(m0 > 0.f)) v0 *= slope;
  if (!(m1 > 0.f)) v1 *= slope;
  return (uint32_t)f32_to_bf16(v0) | ((uint32_t)f32_to_bf16(v1) << 16);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int BUF_OOB = (int)0x80000000;   // byte offset beyond every buffer: such a lane reads zero

// The descriptor must live in scalar registers: the pointer is passed through readfirstlane so the
// compiler knows it is wave-uniform (otherwise every load becomes a waterfall loop).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  void* q = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(q, 0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// VEC: rows start 4-byte aligned and W is even, so a pair of bf16 is one dword load (the normal case);
// otherwise the two elements of a pair are fetched by two 2-byte loads with their own validity.
// FLAT: for outputs of one or two planes (the halo strips of a main / halo split) the ND wavefronts of a
// channel block take ND groups of rows of ONE plane instead of ND planes, so no wavefront runs empty.
// ROW16: volumes of 8 or 16 columns in whole aligned 16-byte pieces: a row is one or two loads a channel instead of ten dword loads (the
// vector-memory instructions of a chunk took as long as its products), and the columns outside the volume, always the same units of
// LDS, are cleared once.  256 -> 256 channels on 8 x 16^3 120 -> 111 us, 64 -> 64 on 32 x 8^3 34 -> 31; same products in the
// same order.
// ROW = 1: from the tensor itself.  ROW = 2: from a prepared copy whose rows are longer than the result's, or onto a result whose rows cannot be
// stored two voxels at a time (told apart at run time this cost the first form 3 to 5 %: 64->8 on 4 x 4x198x16 12.9 -> 13.6 us).
template <int NCB, int ND, int TWC, bool MASKED, bool VEC, bool SPLIT, bool FLAT, int ROW>
__global__ void __launch_bounds__(WG_THREADS) conv3d_mfma_kernel(const bf16_t* __restrict__ in, const bf16_t* __restrict__ mask,
                                                                 const uint4* __restrict__ wp, const float* __restrict__ bias,
                                                                 bf16_t* __restrict__ out, MfmaArgs a) {
  static_assert(NCB * ND == 8, "8 wavefronts per workgroup");
  constexpr int RPB = 32 / TWC;        // h rows per MFMA column block
  constexpr int TH = 4 * RPB, TW = TWC;   // rows per wavefront
  constexpr int TDP = FLAT ? 1 : ND, THT = FLAT ? TH * ND : TH;   // planes and rows of the workgroup's tile
  constexpr int TD2 = TDP + 2, TH2 = THT + 2;
  constexpr int P = TWC == 32 ? 36 : 20;   // LDS row pitch in 16-byte units: w in [w0-2, w0+TW+2)
  constexpr int PAIRS = (TW + 4) / 2;
  constexpr int CIG_UNITS = TD2 * TH2 * P;
  constexpr int BUF_UNITS = 2 * CIG_UNITS;
  constexpr bool ROW16 = ROW != 0;
  static_assert(!ROW16 || (TWC == 16 && VEC && !MASKED), "16-byte staging: one tile across, no mask");
  constexpr int ITEMS_ROW = ROW16 ? 2 : PAIRS;
  constexpr int NITEMS = 2 * TD2 * TH2 * ITEMS_ROW;
  constexpr int ROUNDS = (NITEMS + WG_THREADS - 1) / WG_THREADS;
  constexpr int NFRAG = 3 * RPB + 3;   // distinct start rows b*RPB + kh
  constexpr int RING = 4;              // row fragments in flight
  constexpr int APRE = 5, PRE = MASKED ? 0 : 4;   // steps whose weights are requested before the next stage's input; by the chunk before (a masked form has no registers to spare)
  extern __shared__ uint4 lds[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cbw = wave / ND, wd = wave % ND;
  const int co_blk = blockIdx.y * NCB + cbw;
  const int W = a.in.w, H = a.in.h, WO = ROW == 2 ? a.out.w : W;

  // ---- tile-invariant part of the staging plan: which units this thread fills
  int lds_unit[ROUNDS], item_meta[ROUNDS];   // meta: pair | hy << 8 | dz << 16 | cig << 24 (cig 2: no item)
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    int item = tid + r * WG_THREADS;
    int pair = item % ITEMS_ROW;
    int x = item / ITEMS_ROW;
    int hy = x % TH2; x /= TH2;
    int dz = x % TD2;
    int cig = item < NITEMS ? x / TD2 : 2;
    lds_unit[r] = (cig * TD2 + dz) * (TH2 * P) + hy * P + (ROW16 ? 2 + 8 * pair : 2 * pair);
    item_meta[r] = pair | (hy << 8) | (dz << 16) | (cig << 24);
  }

  // ---- per-tile part: byte offsets of this thread's items inside the sample (ci-group included),
  //      BUF_OOB where the item lies outside the volume: a buffer load then returns zero without
  //      any branch or select.  The channel inside the chunk is added as a scalar offset.
  constexpr int NV = VEC ? 1 : 2;
  int voff[ROUNDS][NV], moffb[MASKED ? ROUNDS : 1][NV];
  int n_plan = 0;   // sample index of the planned tile (wave-uniform)
  const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(wp, (uint32_t)a.ncoblk * a.nchunks * 27 * 1024);
  // (Inlined by force: where the compiler kept one of these as a function, every array and the arguments themselves lay in scratch, 816 to 912 bytes a
  // lane in five masked forms for odd rows or addresses.  us, so and inlined, without room for the copy: masked 8->8 on 9x30x41 72 and 34, 64->64 on
  // 2x32x33 167 and 71, 32->32 on 2 x 12x30x15 58 and 35; an odd result, 16->8 on 4 x 16x64x64 80 and 42.)
  auto plan_tile = [&](int tile) __attribute__((always_inline)) {
    int t = tile;
    const int tw = t % a.tiles_w; t /= a.tiles_w;
    const int th = t % a.tiles_h; t /= a.tiles_h;
    const int td = t % a.tiles_d;
    const int n = t / a.tiles_d;
    const int w0 = tw * TW, h0 = th * THT, ps0 = td * TDP;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int m = item_meta[r];
      const int pair = m & 0xff, hy = (m >> 8) & 0xff, dz = (m >> 16) & 0xff, cig = m >> 24;
      const int p_in = ps0 - a.out.hlo + dz - 1;        // local interior index of the input plane
      const int64_t gq = a.in.doff + p_in;
      const int sp = p_in + a.in.hlo;
      const int h = h0 + hy - 1, w = ROW16 ? 8 * pair : w0 - 2 + 2 * pair;
      const bool ok = cig < 2 && gq >= 0 && gq < a.in.dglob && sp >= 0 && sp < a.in.ds && h >= 0 && h < H;
      const int base = 2 * (cig * 8 * (int)a.in.cstride + sp * (int)a.in.plane + h * W + w);
      const int mbase = MASKED ? 2 * (cig * 8 * (int)a.mask.cstride + (p_in + a.mask.hlo) * (int)a.mask.plane + h * W + w) : 0;
#pragma unroll
      for (int e2 = 0; e2 < NV; ++e2) {
        const bool okw = VEC ? (ok && w >= 0 && w + 1 < W) : (ok && w + e2 >= 0 && w + e2 < W);
        voff[r][e2] = okw ? base + 2 * e2 : BUF_OOB;
        if (MASKED) moffb[r][e2] = okw ? mbase + 2 * e2 : BUF_OOB;
      }
    }
    n_plan = n;
  };

  static_assert(!ROW16 || ROUNDS == 1, "one piece of eight channels a thread");
  u32x4 v16[ROW16 ? 8 : 1];
  uint32_t v[ROUNDS][8];
  uint32_t mv[MASKED ? ROUNDS : 1][8];

  // `live` = false turns every load into an out-of-range (zero, no traffic) one: the last stage of a
  // workgroup has nothing to prefetch, but keeping the load count identical on every path lets the
  // compiler use exact s_waitcnt counts for the weight fragments instead of waiting for everything.
  auto load_chunk = [&](int c, bool live) __attribute__((always_inline)) {
    const bool full = (c + 1) * CI_CHUNK <= a.cin_k;   // uniform: no channel of this chunk is beyond Cin
    const __amdgpu_buffer_rsrc_t rs_in = make_rsrc(in + n_plan * a.in.nstride, (uint32_t)a.in.nstride * 2);
    const __amdgpu_buffer_rsrc_t rs_mask = make_rsrc(MASKED ? mask + n_plan * a.mask.nstride : in, (uint32_t)a.mask.nstride * 2);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int soff = __builtin_amdgcn_readfirstlane(2 * (c * CI_CHUNK + e) * (int)a.in.cstride);
      const int smoff = MASKED ? __builtin_amdgcn_readfirstlane(2 * (c * CI_CHUNK + e) * (int)a.mask.cstride) : 0;
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        int vo[NV], mo[NV];
#pragma unroll
        for (int e2 = 0; e2 < NV; ++e2) {
          vo[e2] = live ? voff[r][e2] : BUF_OOB;
          mo[e2] = MASKED ? (live ? moffb[r][e2] : BUF_OOB) : 0;
          if (!full) {
            const bool chan_ok = c * CI_CHUNK + (item_meta[r] >> 24) * 8 + e < a.cin_k;
            vo[e2] = chan_ok ? vo[e2] : BUF_OOB;
            mo[e2] = chan_ok ? mo[e2] : BUF_OOB;
          }
        }
        if constexpr (ROW16) {
          v16[e] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, vo[0], soff, 0);
        } else if (VEC) {
          v[r][e] = __builtin_amdgcn_raw_buffer_load_b32(rs_in, vo[0], soff, 0);
          if (MASKED) mv[r][e] = __builtin_amdgcn_raw_buffer_load_b32(rs_mask, mo[0], smoff, 0);
        } else {
          const uint32_t lo = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs_in, vo[0], soff, 0);
          const uint32_t hi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs_in, vo[NV - 1], soff, 0);
          v[r][e] = lo | (hi << 16);
          if (MASKED) {
            const uint32_t ml = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs_mask, mo[0], smoff, 0);
            const uint32_t mh = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs_mask, mo[NV - 1], smoff, 0);
            mv[r][e] = ml | (mh << 16);
          }
        }
      }
    }
  };

  auto store_chunk = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      if ((item_meta[r] >> 24) >= 2) continue;
      if constexpr (ROW16) {
        uint4* dst = lds + buf * BUF_UNITS + lds_unit[0];
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // dword k of each channel = columns 2k, 2k + 1
          uint4 u0, u1;
          u0.x = __builtin_amdgcn_perm(v16[1][k], v16[0][k], 0x05040100); u1.x = __builtin_amdgcn_perm(v16[1][k], v16[0][k], 0x07060302);
          u0.y = __builtin_amdgcn_perm(v16[3][k], v16[2][k], 0x05040100); u1.y = __builtin_amdgcn_perm(v16[3][k], v16[2][k], 0x07060302);
          u0.z = __builtin_amdgcn_perm(v16[5][k], v16[4][k], 0x05040100); u1.z = __builtin_amdgcn_perm(v16[5][k], v16[4][k], 0x07060302);
          u0.w = __builtin_amdgcn_perm(v16[7][k], v16[6][k], 0x05040100); u1.w = __builtin_amdgcn_perm(v16[7][k], v16[6][k], 0x07060302);
          dst[2 * k] = u0;
          dst[2 * k + 1] = u1;
        }
        continue;
      }
      uint32_t g[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) g[e] = MASKED ? mask_pair(v[r][e], mv[r][e], a.mask_slope) : v[r][e];
      uint4 u0, u1;   // unit of w (low halves) and of w+1 (high halves): 8 channels each
      u0.x = __builtin_amdgcn_perm(g[1], g[0], 0x05040100); u1.x = __builtin_amdgcn_perm(g[1], g[0], 0x07060302);
      u0.y = __builtin_amdgcn_perm(g[3], g[2], 0x05040100); u1.y = __builtin_amdgcn_perm(g[3], g[2], 0x07060302);
      u0.z = __builtin_amdgcn_perm(g[5], g[4], 0x05040100); u1.z = __builtin_amdgcn_perm(g[5], g[4], 0x07060302);
      u0.w = __builtin_amdgcn_perm(g[7], g[6], 0x05040100); u1.w = __builtin_amdgcn_perm(g[7], g[6], 0x07060302);
      uint4* dst = lds + buf * BUF_UNITS + lds_unit[r];
      dst[0] = u0;
      dst[1] = u1;
    }
  };

  const bool wave_active = co_blk < a.ncoblk;
  const int j = lane & 31;
  // accumulators start from the bias of their output channel (row 8*(r/4) + 4*(lane/32) + r%4 of the block)
  f32x16 acc[4];
  auto init_acc = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int co = co_blk * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
      const float bv = (bias && co < a.cout_k) ? bias[co] : 0.f;
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[b][r] = bv;
    }
  };
  init_acc();

  const int lane_unit = (lane >> 5) * CIG_UNITS + ((FLAT ? 0 : wd) * TH2 + (FLAT ? wd * TH : 0) + j / TWC) * P + (j % TWC) + 1;

  const int a_voff = ((wave_active ? co_blk : 0) * a.nchunks * 27 * 64 + lane) * 16;
  auto load_a = [&](int c, int step, uint4 (&dst)[3]) {
    const int kd = step / 3, kw = step % 3;
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
      const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs_w, a_voff, __builtin_amdgcn_readfirstlane((c * 27 + kd * 9 + kh * 3 + kw) * 1024), 0);
      dst[kh] = uint4{t.x, t.y, t.z, t.w};
    }
  };

  // One chunk = 9 (kd,kw) steps of 12 MFMAs.  Vector-memory loads return in order, so a wait for a weight fragment also waits for every
  // load issued before it.  The weights of the first APRE steps are therefore requested before the (long-latency) input loads of the next
  // stage (`issue_next`), PRE of them by the chunk before (c_next: the chunk after this one), and the others once the input has had some
  // steps to land.  Row fragments come through a ring of four, read as the products go (two whole steps of them in registers, read
  // in one go, left the matrix pipes to wait for LDS and no registers for weights of the next chunk), one memory or LDS
  // instruction or two behind each product.  us, before and after: 256->256 on 8 x 16^3 106 and 98, 64->128 on 4 x 16^3 30.9 and 26.4, 128->96 on
  // 53x48x8 52 and 43, 64->64 on 2x256x256 37.7 and 34.3, 256->256 on 8^3 28.2 and 27.6, masked 16->8 on 4 x 16x64x64 28.2 and 27.1.
  uint4 afr[9][3];
  auto compute_chunk = [&](int c, int c_next, int buf, auto&& issue_next) {
    const uint4* base = lds + buf * BUF_UNITS + lane_unit;
    uint4 bfr[RING];
    auto row = [&](int i) { return base[(i / NFRAG / 3 * TH2 + i % NFRAG) * P + i / NFRAG % 3]; };      // row fragment i of the chunk's 9 * NFRAG
#pragma unroll
    for (int step = PRE; step < APRE; ++step) load_a(c, step, afr[step]);
#pragma unroll
    for (int i = 0; i < RING; ++i) bfr[i] = row(i);
    __builtin_amdgcn_sched_barrier(0);   // keep the weight requests ahead of the input loads ...
    issue_next();
    __builtin_amdgcn_sched_barrier(0);   // ... and the input loads ahead of the MFMA steps (not sunk below them)
#pragma unroll
    for (int step = 0; step < 9; ++step) {
      if (step == APRE - 1) {
#pragma unroll
        for (int s2 = APRE; s2 < 9; ++s2) load_a(c, s2, afr[s2]);
      }
      if (step >= 9 - PRE) load_a(c_next, step - (9 - PRE), afr[step - (9 - PRE)]);
#pragma unroll
      for (int s = 0; s < NFRAG; ++s) {
        const int i = step * NFRAG + s;
        const bf16x8 B = __builtin_bit_cast(bf16x8, bfr[i % RING]);
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
          // the block whose start row b*RPB + kh equals s
          if (s - kh >= 0 && (s - kh) % RPB == 0 && (s - kh) / RPB < 4) {
            const int b = (s - kh) / RPB;
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, afr[step][kh]), B, acc[b], 0, 0, 0);
          }
        }
        if (i + RING < 9 * NFRAG) bfr[i % RING] = row(i + RING);
      }
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x326, 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // activation, bf16 store (the bias is already in the accumulators); output planes outside the global
  // volume are zero.  Buffer stores: the lane's voxel offset (BUF_OOB where the voxel is beyond H or W:
  // such a store is dropped) plus a scalar channel offset — no branches, no 64-bit address arithmetic.
  auto epilogue = [&](int tile) {
    int t = tile;
    const int tw = t % a.tiles_w; t /= a.tiles_w;
    const int th = t % a.tiles_h; t /= a.tiles_h;
    const int td = t % a.tiles_d;
    const int n = t / a.tiles_d;
    const int w0 = tw * TW, h0 = th * THT + (FLAT ? wd * TH : 0), ps = td * TDP + (FLAT ? 0 : wd);
    if (!wave_active || ps >= a.out.ds) return;
    const int64_t gp = a.out.doff + ps - a.out.hlo;
    const bool inside = gp >= 0 && gp < a.out.dglob;
    const int row_ch = 4 * (lane >> 5);   // this lane's accumulator rows are channels 8*(r/4) + row_ch + r%4 of the block
    if (SPLIT) {
      // the accumulators go out as they are, [split][tile][channel block][plane of the tile][b*16 + r][lane]: every
      // store instruction writes 256 contiguous bytes; the reduction kernel undoes the mapping
      float* pp = a.part + (((((int64_t)blockIdx.z * a.ntiles + tile) * a.ncoblk + co_blk) * ND + wd) * 64) * 64 + lane;
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) pp[(b * 16 + r) * 64] = acc[b][r];
      return;
    }
    const __amdgpu_buffer_rsrc_t rs_out = make_rsrc(out + n * a.out.nstride, (uint32_t)a.out.nstride * 2);
    if (VEC && (ROW != 2 || a.pairs)) {
      // Two adjacent voxels live in adjacent lanes.  Lane pairs swap one value (DPP quad_perm [1,0,3,2])
      // so that the even lane holds both voxels of channel row r and the odd lane both voxels of row
      // r+1: every lane then stores ONE dword (two bf16) instead of two shorts.
      const bool odd = lane & 1;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int h = h0 + b * RPB + j / TWC, w = w0 + (j % TWC) - (odd ? 1 : 0);
        const int vo = (h < H && w < WO)
                           ? 2 * ((row_ch + (odd ? 1 : 0)) * (int)a.out.cstride + ps * (int)a.out.plane + h * WO + w) : BUF_OOB;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int co_u = co_blk * 32 + 8 * (r / 4) + (r % 4);          // wave-uniform part of the even lane's channel
          const bool ch_ok = co_u + row_ch + (odd ? 1 : 0) < a.cout_k;
          float v0 = acc[b][r], v1 = acc[b][r + 1];
          if (!(v0 > 0.f)) v0 *= a.out_slope;
          if (!(v1 > 0.f)) v1 *= a.out_slope;
          const float give = odd ? v0 : v1;
          const float got = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(give), 0xB1, 0xF, 0xF, true));
          const uint32_t pk = odd ? pack_bf16x2(got, v1) : pack_bf16x2(v0, got);
          __builtin_amdgcn_raw_buffer_store_b32(inside ? pk : 0u, rs_out, ch_ok ? vo : BUF_OOB,
                                                __builtin_amdgcn_readfirstlane(2 * co_u * (int)a.out.cstride), 0);
        }
      }
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int h = h0 + b * RPB + j / TWC, w = w0 + j % TWC;
        const int vo = (h < H && w < WO) ? 2 * (row_ch * (int)a.out.cstride + ps * (int)a.out.plane + h * WO + w) : BUF_OOB;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int co_u = co_blk * 32 + 8 * (r / 4) + (r % 4);            // wave-uniform part of the channel
          const bool ch_ok = co_u + row_ch < a.cout_k;
          float val = acc[b][r];
          if (!(val > 0.f)) val *= a.out_slope;
          __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(inside ? val : 0.f), rs_out, ch_ok ? vo : BUF_OOB,
                                                __builtin_amdgcn_readfirstlane(2 * co_u * (int)a.out.cstride), 0);
        }
      }
    }
  };

  // ---- persistent loop: this workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ...; the
  //      (tile, ci-chunk) stages alternate between two LDS buffers, and the global loads of the next
  //      stage — the next chunk, or chunk 0 of the NEXT TILE — are in flight while this one is multiplied
  // consecutive workgroup ids land on different XCDs (each with its own L2): remap so that the
  // workgroups of one XCD work on neighbouring tiles and share the halo lines in that L2
  const int G = gridDim.x;
  int tile = (G % 8 == 0) ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  if (tile >= a.ntiles) return;
  const int c_begin = SPLIT ? blockIdx.z * a.chunks_per_split : 0;
  const int c_end = SPLIT ? min(a.nchunks, c_begin + a.chunks_per_split) : a.nchunks;
  plan_tile(tile);
  load_chunk(c_begin, true);
  if (wave_active) {
#pragma unroll
    for (int step = 0; step < PRE; ++step) load_a(c_begin, step, afr[step]);
  }
  if constexpr (ROW16) {      // the units of columns -2, -1 and 16, 17 (no piece covers them) of every row, both buffers
    for (int i = tid; i < 2 * 2 * TD2 * TH2 * 4; i += WG_THREADS) lds[(i >> 2) * P + (i & 1) + ((i & 2) ? 18 : 0)] = uint4{0, 0, 0, 0};
  }
  store_chunk(0);
  __syncthreads();
  int buf = 0;
  while (true) {
    for (int c = c_begin; c < c_end; ++c) {
      const bool last_chunk = c + 1 == c_end;
      const int next_tile = tile + G;
      const bool more = !last_chunk || next_tile < a.ntiles;
      auto issue_next = [&]() __attribute__((always_inline)) {
        if (last_chunk && more) plan_tile(next_tile);
        load_chunk(last_chunk ? c_begin : c + 1, more);
      };
      if (wave_active) compute_chunk(c, last_chunk ? c_begin : c + 1, buf, issue_next);
      else issue_next();
      if (more) store_chunk(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
    epilogue(tile);
    init_acc();
    tile += G;
    if (tile >= a.ntiles) break;
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Wide-blocked form of the same implicit GEMM for the large layers (more than 16 columns, at least 3 stored output
// planes, no fused mask): FOUR wavefronts per workgroup, one per SIMD, each owning CB blocks of 32 output channels x
// 8 MFMA column blocks (8 rows x 32 columns of one plane = 256 voxels): CB * 8 accumulator tiles = up to 256
// registers, which the compiler keeps in the accumulation registers.  Per (kd,kw) step a wavefront then needs 3 * CB
// weight fragments and 10 row fragments for 24 * CB products: one weight fragment feeds 8 products and one row
// fragment up to 3 * CB, against 4 and 2-3 in the kernel above, so the weight stream from L2 and the LDS reads per
// product are both halved, and a chunk of 16 input channels is 216 * CB products per wavefront between two barriers.
// Nothing else hides a wavefront's stall, so everything is requested ahead: weight fragments two steps ahead (three
// register sets; they do not depend on the tile, so the stream runs on across chunk and tile borders, and nine steps a
// chunk let the sets take turns without a copy), row fragments RING products' worth ahead (a register is refilled as soon
// as its last product has been issued), and the input of the next stage in two groups of 8 channels that are requested in
// thirds at steps 0-2 and 4-6 and written to the other LDS buffer at step 4 and after step 8.  Vector-memory operations
// return in issue order and share one counter, so a wait for the weight fragments of step s + 2 also waits for the input
// requests issued before them, i.e. up to step s - 1: with one step between request and use (ten row fragments in flight,
// which left no registers for a third set) the products waited for HBM.  Five row fragments are enough beside three sets:
// 64 -> 64 on 32x128x128 98.9 -> 94.8 us, 32 -> 64 on 66x256x256 474 -> 457, 128 -> 64 on 64x256x256 1409 -> 1380, its
// backward-data 1498 -> 1465, 64 -> 8 on 8 x 21x118x160 373 -> 357; layers of one or two chunks a tile as before; four fragments 1 % slower.
// Measured by switching parts off (128 -> 64 channels on 64 x 256 x 256, one box): with the output stores redirected
// into a 64 KB window that stays in the L2 the kernel takes 1.19 instead of 1.44 ms although it issues the same
// instructions - 5 % fewer cycles and a shader clock of 2.14 instead of 1.85 GHz; cache-policy bits on the stores and a
// staggered start of the workgroups change nothing.  The 537 MB of output cost about 0.25 ms that nothing in the kernel
// hides.
// The sums are taken in the order of the kernel above (chunk, kd, kw, kh), so the two give identical bits.
// WCB = 2 (the form that runs for more than 32 output channels, with CB = 1): EIGHT wavefronts per workgroup, two per
// SIMD and plane, each with its own channel block of the same tile: a wavefront holds 128 accumulators and 256
// registers in all, the staged input serves the same 64 channels as with CB = 2, and while one wavefront of a SIMD waits
// (request, LDS, barrier, epilogue stores) the other multiplies.  Measured against the four-wavefront CB = 2 form on one
// box, seven layers of the U-Net level: 4 to 9 % faster on every one (128->64: 1.48 -> 1.43 ms, 32->64: 0.505 -> 0.46).
// Instantiated: <1, 1> and <1, 1, 2> (at most 32 output channels, or small volumes) and <1, 2>.
// RSP = 2 (for layers with a single block of output channels): eight wavefronts as well, the two of a plane taking
// four rows of the tile each (64 accumulators, 6 row fragments per step).
// RAGGED: output rows of odd length (the input is then a prepared copy): a row's last voxel is stored on its own.
// SPLIT: the input chunks are dealt to blockIdx.z; the accumulators leave as they are, [split][tile][channel block][plane][row * 16 + r][lane].
// POOL: the 2x2x2 max pooling of the result is written beside it.  A wavefront takes half of the rows of two planes, so that a window's eight voxels are
// in one pair of lanes (12 row fragments a step instead of 10; with whole planes and an exchange through LDS the wavefronts meet between tiles: 512 us).
// The form of two blocks a workgroup keeps 13 registers of its epilogue's addresses and tests in scratch, and waits for its stores where it reads them back.  us,
// two calls and one: 32 -> 64 on 64x256x256 544 and 486, on 16x128x128 41.6 and 38.1, 16 -> 32 on 4 x 64^3 54.7 and 46.4, 32 -> 64 on 4 x 32^3 31.3 and 24.8.
template <int CB, int WCB, int RSP = 1, bool RAGGED = false, bool SPLIT = false, bool POOL = false>
__global__ void __launch_bounds__(256 * WCB * RSP) conv3d_mfma_wide_kernel(const bf16_t* __restrict__ in, const uint4* __restrict__ wp,
                                                                     const float* __restrict__ bias, bf16_t* __restrict__ out, MfmaArgs a) {
  static_assert(WCB * RSP <= 2, "at most eight wavefronts");
  constexpr int NT = 256 * WCB * RSP;
  constexpr int TD = 4, TH = 8, TW = 32, VB = TH / RSP;      // VB: row blocks (of 32 voxels) per wavefront
  constexpr int TD2 = TD + 2, TH2 = TH + 2;
  constexpr int P = 36, PAIRS = 18;            // LDS row: w in [w0-2, w0+34), 16-byte units of 8 channels
  constexpr int CIG_UNITS = TD2 * TH2 * P;
  constexpr int BUF_UNITS = 2 * CIG_UNITS;
  constexpr int NITEMS = TD2 * TH2 * PAIRS;   // (plane, row, pair of columns) items of one channel group
  constexpr int ROUNDS = (NITEMS + NT - 1) / NT;
  constexpr int PL = POOL ? 2 : 1, VR = VB / PL;             // planes, and rows of each, of a wavefront
  constexpr int NFRAG = PL * (VR + 2);
  constexpr int RING = WCB == 2 ? (POOL ? 4 : 5) : NFRAG;   // row fragments in flight: as many as fit beside three sets of weights (pooling, 5: 498 us)
  extern __shared__ uint4 lds[];

  const int tid = threadIdx.x, lane = tid & 63, wd = POOL ? (tid >> 6) & 2 : (tid >> 6) & 3;      // (first) plane of the tile
  const int wcb = WCB == 2 ? tid >> 8 : 0, rh = RSP == 2 ? tid >> 8 : 0;   // channel-block group, row half
  const int row0 = POOL ? ((tid >> 6) & 1) * (TH / 2) + rh * VR : rh * VB;                  // first row of the tile
  const int co_blk0 = (blockIdx.y * WCB + wcb) * CB;
  const int W = a.in.w, H = a.in.h, WO = a.out.w;     // a prepared input has padded rows: W = WO rounded up

  int lds_unit[ROUNDS], item_meta[ROUNDS];     // meta: pair | hy << 8 | dz << 16 | valid << 24
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int item = tid + r * NT;
    const int pair = item % PAIRS;
    int x = item / PAIRS;
    const int hy = x % TH2; x /= TH2;
    const int dz = x % TD2;
    const int valid = item < NITEMS ? 1 : 0;
    lds_unit[r] = (dz * TH2 + hy) * P + 2 * pair;
    item_meta[r] = pair | (hy << 8) | (dz << 16) | (valid << 24);
  }

  int voff[ROUNDS];
  int n_plan = 0;
  const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(wp, (uint32_t)a.ncoblk * a.nchunks * 27 * 1024);
  auto plan_tile = [&](int tile) {
    int t = tile;
    const int tw = t % a.tiles_w; t /= a.tiles_w;
    const int th = t % a.tiles_h; t /= a.tiles_h;
    const int td = t % a.tiles_d;
    const int n = t / a.tiles_d;
    const int w0 = tw * TW, h0 = th * TH, ps0 = td * TD;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int m = item_meta[r];
      const int pair = m & 0xff, hy = (m >> 8) & 0xff, dz = (m >> 16) & 0xff;
      const int p_in = ps0 - a.out.hlo + dz - 1;
      const int64_t gq = a.in.doff + p_in;
      const int sp = p_in + a.in.hlo;
      const int h = h0 + hy - 1, w = w0 - 2 + 2 * pair;
      const bool ok = (m >> 24) && gq >= 0 && gq < a.in.dglob && sp >= 0 && sp < a.in.ds && h >= 0 && h < H && w >= 0 && w + 1 < W;
      voff[r] = ok ? 2 * (sp * (int)a.in.plane + h * W + w) : BUF_OOB;
    }
    n_plan = n;
  };

  uint32_t v[ROUNDS][8];
  // part `q` of 3 of one group of 8 input channels of chunk c for the planned tile (`live` false: nothing to fetch, all
  // loads out of range).  A group is requested over three steps so that no request queue ever holds a long batch in
  // front of the weight fragments (vector loads return in order).
  auto load_part = [&](int c, int cig, int q, bool live) {
    const __amdgpu_buffer_rsrc_t rs_in = make_rsrc(in + n_plan * a.in.nstride, (uint32_t)a.in.nstride * 2);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e / 3 != q) continue;                      // channels 0-2, 3-5, 6-7
      const int ch = c * CI_CHUNK + cig * 8 + e;
      const bool chan_ok = live && ch < a.cin_k;     // wave-uniform
      const int soff = __builtin_amdgcn_readfirstlane(chan_ok ? 2 * ch * (int)a.in.cstride : 0);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) v[r][e] = __builtin_amdgcn_raw_buffer_load_b32(rs_in, chan_ok ? voff[r] : BUF_OOB, soff, 0);
    }
  };
  auto load_half = [&](int c, int cig, bool live) {
    load_part(c, cig, 0, live);
    load_part(c, cig, 1, live);
    load_part(c, cig, 2, live);
  };
  auto store_half = [&](int buf, int cig) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      if (!(item_meta[r] >> 24)) continue;
      uint4 u0, u1;
      u0.x = __builtin_amdgcn_perm(v[r][1], v[r][0], 0x05040100); u1.x = __builtin_amdgcn_perm(v[r][1], v[r][0], 0x07060302);
      u0.y = __builtin_amdgcn_perm(v[r][3], v[r][2], 0x05040100); u1.y = __builtin_amdgcn_perm(v[r][3], v[r][2], 0x07060302);
      u0.z = __builtin_amdgcn_perm(v[r][5], v[r][4], 0x05040100); u1.z = __builtin_amdgcn_perm(v[r][5], v[r][4], 0x07060302);
      u0.w = __builtin_amdgcn_perm(v[r][7], v[r][6], 0x05040100); u1.w = __builtin_amdgcn_perm(v[r][7], v[r][6], 0x07060302);
      uint4* dst = lds + buf * BUF_UNITS + cig * CIG_UNITS + lds_unit[r];
      dst[0] = u0;
      dst[1] = u1;
    }
  };

  const int j = lane & 31;
  // The accumulators of a tile start from the bias (the sums are then taken in the order of the kernel above: same
  // bits).  Writing 256 accumulation registers one by one from the vector ALU costs a wavefront about 5000 cycles
  // per tile (measured); instead the bias enters as a product: a weight-shaped fragment that holds, for each channel
  // of the block, the three bfloat16 pieces of its fp32 bias (upper, middle and lower 8 mantissa bits, cut by
  // truncation: their sum is the bias exactly) in the first three of the 16 contraction slots and zeros in the others,
  // multiplied by a fragment of ones: sixteen extra MFMAs per tile, D = hi + mid + lo + 0 ... = bias in every column.
  uint4* biasf_l = lds + 2 * BUF_UNITS + wcb * CB * 64;       // [WCB][CB][64 lanes] fragments behind the two stage buffers
  if ((tid & 255) < CB * 64) {
    const int cb = (tid & 255) >> 6, l = tid & 63;
    uint4 f = {0u, 0u, 0u, 0u};
    const int co = (co_blk0 + cb) * 32 + l;
    if (l < 32 && bias && co < a.cout_k) {
      const float bv = bias[co];
      const uint32_t hi = __float_as_uint(bv) & 0xffff0000u;
      const float r1 = bv - __uint_as_float(hi);
      const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
      const float r2 = r1 - __uint_as_float(mid);
      const uint32_t lo = __float_as_uint(r2) & 0xffff0000u;
      f.x = (hi >> 16) | mid;
      f.y = lo >> 16;
    }
    biasf_l[tid & 255] = f;
  }
  __syncthreads();
  f32x16 acc[CB][VB];
  auto init_acc = [&]() {
    const uint4 ones_u = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_u);
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const bf16x8 bf = __builtin_bit_cast(bf16x8, biasf_l[cb * 64 + lane]);
#pragma unroll
      for (int b = 0; b < VB; ++b) acc[cb][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf, ones, zero, 0, 0, 0);
    }
  };
  init_acc();

  const int lane_unit = (lane >> 5) * CIG_UNITS + (wd * TH2 + row0) * P + j + 1;
  const int a_voff = lane * 16;
  // weight fragments of one (kd,kw) step: [kh][channel block]; a channel block beyond Cout re-reads the last valid one
  auto load_a = [&](int c, int step, uint4 (&dst)[3][CB]) {
    const int kd = step / 3, kw = step % 3;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int blk = min(co_blk0 + cb, a.ncoblk - 1);
#pragma unroll
      for (int kh = 0; kh < 3; ++kh) {
        const int soff = __builtin_amdgcn_readfirstlane(((blk * a.nchunks + c) * 27 + kd * 9 + kh * 3 + kw) * 1024);
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs_w, a_voff, soff, 0);
        dst[kh][cb] = uint4{t.x, t.y, t.z, t.w};
      }
    }
  };

  uint4 afr[3][3][CB];        // weight fragments of the current and of the next two steps (nine steps a chunk: the sets take turns across chunks)
  const int G = gridDim.x;
  int tile = (G % 8 == 0) ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  if (tile >= a.ntiles) return;
  const int c_begin = SPLIT ? blockIdx.z * a.chunks_per_split : 0, c_end = SPLIT ? min(a.nchunks, c_begin + a.chunks_per_split) : a.nchunks;

  // One chunk: 9 steps of 24 * CB products.  c_next: the chunk whose weight stream follows this one's.  The step order
  // is: request the weight fragments of the step after next, then this step's share of the next stage's input, then
  // multiply; a row fragment register is refilled as soon as its last product has been issued.
  auto compute_chunk = [&](int c, int c_next, int buf, bool more, int next_tile, bool last_chunk) {
    const uint4* base = lds + buf * BUF_UNITS + lane_unit;
    uint4 bfr[RING];
    auto row = [&](int i) { return base[((i / NFRAG / 3 + i % NFRAG / (VR + 2)) * TH2 + i % NFRAG % (VR + 2)) * P + i / NFRAG % 3]; };      // row fragment i of the chunk's 9 * NFRAG
#pragma unroll
    for (int i = 0; i < RING; ++i) bfr[i] = row(i);
    const int cn = last_chunk ? c_begin : c + 1;
#pragma unroll
    for (int step = 0; step < 9; ++step) {
      if (step + 2 < 9) load_a(c, step + 2, afr[(step + 2) % 3]);
      else load_a(c_next, step + 2 - 9, afr[(step + 2) % 3]);
      if (step == 0 && last_chunk && more) plan_tile(next_tile);
      if (step < 3) load_part(cn, 0, step, more);
      if (step == 4 && more) store_half(buf ^ 1, 0);
      if (step >= 4 && step < 7) load_part(cn, 1, step - 4, more);
#pragma unroll
      for (int s = 0; s < NFRAG; ++s) {
        const int i = step * NFRAG + s;
        const bf16x8 B = __builtin_bit_cast(bf16x8, bfr[i % RING]);
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
          const int b = s % (VR + 2) - kh, o = s / (VR + 2) * VR + b;
          if (b >= 0 && b < VR) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
              acc[cb][o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, afr[step % 3][kh][cb]), B, acc[cb][o], 0, 0, 0);
          }
        }
        if (i + RING < 9 * NFRAG) bfr[i % RING] = row(i + RING);
      }
      // the requests, address arithmetic and LDS traffic of the step must be issued in the
      // shadow of its products (a product occupies the matrix pipe for 32 cycles, the wavefront can issue about seven
      // other instructions meanwhile), not in a block in front of them
#pragma unroll
      for (int i = 0; i < 3 * VB * CB; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x326, 3, 0);      // up to three of: VALU, SALU, vector-memory read, LDS read / write
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) store_half(buf ^ 1, 1);
  };

  // Epilogue of a tile (CB * 128 values per lane): everything that does not depend on the value is taken out of the
  // per-value path.  The activation is skipped when there is none, and max(v, slope * v) where that has the bits of
  // "v > 0 ? v : slope * v": 0 < slope <= 1.  Any other slope compares: above 1 the larger one is the wrong one, below 0 a zero gets the other
  // sign, and with slope 0 the maximum loses the NaN of -inf * 0.
  auto epilogue = [&](int tile_) {
    int t = tile_;
    const int tw = t % a.tiles_w; t /= a.tiles_w;
    const int th = t % a.tiles_h; t /= a.tiles_h;
    const int td = t % a.tiles_d;
    const int n = t / a.tiles_d;
    const int w0 = tw * TW, h0 = th * TH + row0, ps = td * TD + wd;      // this wavefront's first row
    if (ps >= a.out.ds) return;
    if constexpr (SPLIT) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        float* pp = a.part + ((((int64_t)blockIdx.z * a.ntiles + tile_) * a.ncoblk + co_blk0 + cb) * TD + wd) * (TH * 1024) + rh * VB * 1024 + lane;
        if (co_blk0 + cb < a.ncoblk)
#pragma unroll
          for (int b = 0; b < VB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) pp[(b * 16 + r) * 64] = acc[cb][b][r];
      }
      return;
    }
    const int64_t gp = a.out.doff + ps - a.out.hlo;
    const bool inside = gp >= 0 && gp < a.out.dglob;
    const int row_ch = 4 * (lane >> 5);
    const __amdgpu_buffer_rsrc_t rs_out = make_rsrc(out + n * a.out.nstride, (uint32_t)a.out.nstride * 2);
    // A lane holds one voxel of 16 channels; a store wants two neighbouring voxels of one channel.  Each lane packs
    // its channel pair (r, r+1) to bf16, fetches its neighbour's packed pair (lanes 2k and 2k+1 hold voxels 2k and
    // 2k+1) and picks, with a per-lane byte selector, channel r of both voxels (even lane) or channel r+1 of both
    // (odd lane): one conversion, one lane exchange and one byte permute per stored dword, no selects.
    const bool odd = lane & 1;
    const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
    const int cs2 = 2 * (int)a.out.cstride;
    const int vbase = (row_ch + (odd ? 1 : 0)) * cs2 + 2 * (ps * (int)a.out.plane + h0 * WO + w0 + j - (odd ? 1 : 0));
    const bool w_ok = w0 + j - (odd ? 1 : 0) < WO;
    using T_ = std::true_type;
    using F_ = std::false_type;
    const float slope = a.out_slope;
    const bool act = slope != 1.f, by_max = slope > 0.f && slope <= 1.f;        // wave-uniform
    auto activate = [&](float v, auto max_c) {
      const float s = v * slope;
      if (decltype(max_c)::value) asm("v_max_f32 %0, %1, %2" : "=v"(v) : "v"(v), "v"(s));
      else v = v > 0.f ? v : s;
      return v;
    };
    // ACT / BY_MAX / WHOLE are wave-uniform facts: one branch per channel block, not one select per value
    auto block = [&](int cb, auto act_c, auto max_c, auto whole_c) {
      constexpr bool ACT = decltype(act_c)::value, WHOLE = decltype(whole_c)::value;
      const int cblk = co_blk0 + cb;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const int co_u = cblk * 32 + 8 * (r / 4) + (r % 4);
        const int soff = __builtin_amdgcn_readfirstlane(co_u * cs2);
        const bool ch_ok = WHOLE || co_u + row_ch + (odd ? 1 : 0) < a.cout_k;
#pragma unroll
        for (int b = 0; b < VB; ++b) {
          float v0 = acc[cb][b][r], v1 = acc[cb][b][r + 1];
          if (ACT) { v0 = activate(v0, max_c); v1 = activate(v1, max_c); }
          const uint32_t own = pack_bf16x2(v0, v1);
          const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);
          uint32_t pk = __builtin_amdgcn_perm(nb, own, sel);
          int o = (w_ok && h0 + b < H) ? vbase + 2 * b * WO : BUF_OOB;
          if (!WHOLE) {
            pk = inside ? pk : 0u;
            o = ch_ok ? o : BUF_OOB;
          }
          if (RAGGED) {
            const bool second = w0 + j + (odd ? 0 : 1) < WO;
            __builtin_amdgcn_raw_buffer_store_b16((short)(pk & 0xffffu), rs_out, o, soff, 0);
            __builtin_amdgcn_raw_buffer_store_b16((short)(pk >> 16), rs_out, second && o != BUF_OOB ? o + 2 : BUF_OOB, soff, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b32(pk, rs_out, o, soff, 0);
          }
        }
      }
    };
    if constexpr (POOL) {
      static_assert(CB == 1 && !RAGGED && !SPLIT, "one channel block a wavefront, whole rows");
      if (co_blk0 >= a.ncoblk) return;
      // two lanes that hold neighbouring voxels of a channel store both of one of two pooled rows (or, of one row, of one of two channels)
      const __amdgpu_buffer_rsrc_t rs_y = make_rsrc(a.ypool + n * a.yp.nstride, (uint32_t)a.yp.nstride * 2);
      const bool second = lane & 2;
      const uint32_t sel2 = second ? 0x03020706u : 0x05040100u;
      const int wy = w0 / 2 + (j >> 1) - (second ? 1 : 0), qy = ps / 2 + a.yp.hlo, hy = h0 / 2 + (VR == 4 && second ? 1 : 0);
      const bool y_ok = wy < a.yp.w && hy < a.yp.h;
      const int ybase = 2 * ((row_ch + (odd ? 1 : 0) + (VR == 2 && second ? 2 : 0)) * (int)a.yp.cstride + qy * (int)a.yp.plane + hy * a.yp.w + wy);
      auto block = [&](auto max_c, auto whole_c) {
        constexpr bool WHOLE = decltype(whole_c)::value;
        uint32_t before = 0;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int co_u = co_blk0 * 32 + 8 * (r / 4) + (r % 4), co = co_u + row_ch + (odd ? 1 : 0);
          const int soff = __builtin_amdgcn_readfirstlane(co_u * cs2);
          uint32_t pk[VB];
#pragma unroll
          for (int b = 0; b < VB; ++b) {
            const uint32_t own = pack_bf16x2(activate(acc[0][b][r], max_c), activate(acc[0][b][r + 1], max_c));
            const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);
            pk[b] = __builtin_amdgcn_perm(nb, own, sel);
            const int o = w_ok && h0 + b % VR < H ? vbase + 2 * (b / VR * (int)a.out.plane + b % VR * WO) : BUF_OOB;
            __builtin_amdgcn_raw_buffer_store_b32(pk[b], rs_out, WHOLE || co < a.cout_k ? o : BUF_OOB, soff, 0);
          }
          uint32_t best[VR / 2];
#pragma unroll
          for (int k = 0; k < VR / 2; ++k) {
            const uint32_t w4[4] = {pk[2 * k], pk[2 * k + 1], pk[VR + 2 * k], pk[VR + 2 * k + 1]};
            float e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = __uint_as_float((i & 1) ? w4[i / 2] & 0xffff0000u : w4[i / 2] << 16);
            // The pooling kernel goes through a window with "if e > m": m stays where the first element is NaN or equals the maximum.  A maximum of
            // the others does for that unless zeros of both signs follow a negative element.
            float m;
            asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(e[1]), "v"(e[2]), "v"(e[3]));
            asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(m), "v"(e[4]), "v"(e[5]));
            asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(m), "v"(e[6]), "v"(e[7]));
            m = m > e[0] ? m : e[0];
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(m == 0.f && e[0] < 0.f) != 0, 0)) {
              m = e[0];
#pragma unroll
              for (int i = 1; i < 8; ++i) m = e[i] > m ? e[i] : m;
            }
            best[k] = __float_as_uint(m);
          }
          uint32_t own;
          if (VR == 4) {
            own = __builtin_amdgcn_perm(best[VR / 2 - 1], best[0], 0x07060302u);
          } else if (r % 4 == 0) {
            before = best[0];
            continue;
          } else {
            own = __builtin_amdgcn_perm(best[0], before, 0x07060302u);
          }
          const uint32_t nb = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0x4E, 0xF, 0xF, true);
          const int co_y = VR == 4 ? co_u : co_u - 2;
          const bool ok = y_ok && (WHOLE || co_y + row_ch + (odd ? 1 : 0) + (VR == 2 && second ? 2 : 0) < a.cout_k);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(nb, own, sel2), rs_y, ok ? ybase : BUF_OOB,
                                                __builtin_amdgcn_readfirstlane(2 * co_y * (int)a.yp.cstride), 0);
        }
      };
      const bool whole = co_blk0 * 32 + 32 <= a.cout_k;
      if (whole && by_max) block(T_{}, T_{});
      else if (whole) block(F_{}, T_{});
      else if (by_max) block(T_{}, F_{});
      else block(F_{}, F_{});
      return;
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int cblk = co_blk0 + cb;
      if (cblk >= a.ncoblk) continue;
      const bool whole = cblk * 32 + 32 <= a.cout_k && inside;     // the common case
      if (whole) {
        if (!act) block(cb, F_{}, F_{}, T_{});
        else if (by_max) block(cb, T_{}, T_{}, T_{});
        else block(cb, T_{}, F_{}, T_{});
      } else {       // (slope 1 leaves the values as they are)
        if (by_max) block(cb, T_{}, T_{}, F_{});
        else block(cb, T_{}, F_{}, F_{});
      }
    }
  };

  // prologue: first stage into buffer 0, first two steps of the weight stream
  plan_tile(tile);
  load_half(c_begin, 0, true);
  store_half(0, 0);
  load_half(c_begin, 1, true);
  store_half(0, 1);
  load_a(c_begin, 0, afr[0]);
  load_a(c_begin, 1, afr[1]);
  __syncthreads();
  int buf = 0;
  while (true) {
    const int next_tile = tile + G;
    for (int c = c_begin; c < c_end; ++c) {
      const bool last_chunk = c + 1 == c_end;
      const bool more = !last_chunk || next_tile < a.ntiles;
      compute_chunk(c, last_chunk ? c_begin : c + 1, buf, more, next_tile, last_chunk);
      __syncthreads();
      buf ^= 1;
    }
    epilogue(tile);
    init_acc();
    tile = next_tile;
    if (tile >= a.ntiles) break;
  }
}

// out = act(bias + sum over splits of part[split]) in split order; planes outside the global volume are zero.
// part holds raw accumulator tiles (see the SPLIT epilogue): an output element (n, co, ps, h, w) is register
// b*16 + r of lane `lane` of the wavefront (channel block co/32, plane ps % ND) of tile (n, ps/ND, h/TH, w/TW).
struct SplitGeo {
  int nd, twc, rpb, ncoblk, tiles_w, tiles_h, tiles_d, ntiles;
};
__global__ void __launch_bounds__(256) conv_split_reduce_kernel(const float* __restrict__ part, const float* __restrict__ bias,
                                                                bf16_t* __restrict__ out, Geo g, SplitGeo q, int splits, float slope) {
  const int64_t total = (int64_t)g.n * g.nstride;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  int64_t t = i;
  const int w = (int)(t % g.w); t /= g.w;
  const int h = (int)(t % g.h); t /= g.h;
  const int ps = (int)(t % g.ds); t /= g.ds;
  const int co = (int)(t % g.c);
  const int n = (int)(t / g.c);
  const int th_rows = 4 * q.rpb;
  const int tile = ((n * q.tiles_d + ps / q.nd) * q.tiles_h + h / th_rows) * q.tiles_w + w / q.twc;
  const int hl = h % th_rows, wl = w % q.twc, c32 = co % 32;
  const int b = hl / q.rpb, j = (hl % q.rpb) * q.twc + wl;
  const int r = 4 * (c32 / 8) + c32 % 4, lane = ((c32 / 4) % 2) * 32 + j;
  const int64_t slot = ((((int64_t)tile * q.ncoblk + co / 32) * q.nd + ps % q.nd) * 64 + (b * 16 + r)) * 64 + lane;
  const int64_t per_split = (int64_t)q.ntiles * q.ncoblk * q.nd * 4096;
  float s = 0.f;
  for (int sp = 0; sp < splits; ++sp) s += part[sp * per_split + slot];
  const int64_t gp = g.doff + ps - g.hlo;
  float v = s + (bias ? bias[co] : 0.f);
  if (!(v > 0.f)) v *= slope;
  out[i] = f32_to_bf16((gp >= 0 && gp < g.dglob) ? v : 0.f);
}

// The same for the wide kernel's tiles (4 planes x 8 rows x 32 columns, a block of 32 channels 128 KB a split), four columns a thread.
__global__ void __launch_bounds__(256) conv_wide_split_reduce_kernel(const float* __restrict__ part, const float* __restrict__ bias, bf16_t* __restrict__ out,
                                                                     MfmaArgs a, uint32_t total, int vec) {
  uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t >= total) return;
  const Geo& g = a.out;
  const uint32_t w4 = (g.w + 3) / 4;
  const int w = 4 * (int)(t % w4); t /= w4;
  const int h = (int)(t % g.h); t /= g.h;
  const int ps = (int)(t % g.ds); t /= g.ds;
  const int co = (int)(t % a.cout_k), n = (int)(t / a.cout_k);
  const int tile = ((n * a.tiles_d + ps / 4) * a.tiles_h + h / 8) * a.tiles_w + w / 32, c32 = co % 32;
  const int r = 4 * (c32 / 8) + c32 % 4, lane = ((c32 / 4) % 2) * 32 + w % 32;
  const int64_t slot = (((int64_t)tile * a.ncoblk + co / 32) * 4 + ps % 4) * 8192 + ((h % 8) * 16 + r) * 64 + lane;
  const int64_t per_split = (int64_t)a.ntiles * a.ncoblk * 32768;
  const float b = bias ? bias[co] : 0.f;
  float4 s = {0.f, 0.f, 0.f, 0.f};
  for (int sp = 0; sp < a.csplit; ++sp) {
    const float4 v = *reinterpret_cast<const float4*>(part + sp * per_split + slot);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  const int64_t gp = g.doff + ps - g.hlo;
  const bool inside = gp >= 0 && gp < g.dglob;
  auto finish = [&](float v) {
    v += b;
    if (!(v > 0.f)) v *= a.out_slope;
    return inside ? v : 0.f;
  };
  bf16_t* o = out + (int64_t)n * g.nstride + (int64_t)co * g.cstride + (int64_t)ps * g.plane + h * g.w + w;
  const uint2 pk = {pack_bf16x2(finish(s.x), finish(s.y)), pack_bf16x2(finish(s.z), finish(s.w))};
  if (vec) {
    *reinterpret_cast<uint2*>(o) = pk;
  } else {
    const bf16_t e[4] = {(bf16_t)pk.x, (bf16_t)(pk.x >> 16), (bf16_t)pk.y, (bf16_t)(pk.y >> 16)};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (w + k < g.w) o[k] = e[k];
  }
}

// How many ways the input-channel chunks of a narrow volume are split: 1 unless the tiles alone would leave most CUs idle.
// (room: of a workspace for the sums of every split; without it those of at least 64 workgroups are not split)
static int mfma_splits(const h3d_tensor* in, const h3d_tensor* out, int num_cu, bool room) {
  const int nchunks = (int)cdiv(in->c, CI_CHUNK), ncoblk = (int)cdiv(out->c, 32);
  const bool wide = out->w > 16, two_cb = out->c > 32;
  const int twc = wide ? 32 : 16, ncb = two_cb ? 2 : 1, nd = 8 / ncb, th = 4 * (32 / twc);
  const int64_t ds = out->halo_lo + out->d + out->halo_hi;
  const int64_t wgs = (int64_t)out->n * cdiv(ds, nd) * cdiv(out->h, th) * cdiv(out->w, twc) * cdiv(ncoblk, ncb);
  if (wide || wgs == 0 || nchunks < 2 || !is_packed(out)) return 1;    // (only the narrow-volume variants come in a split form)
  // bytes of one split's sums: they cost a write and a read
  const int64_t part = (int64_t)out->n * cdiv(ds, nd) * cdiv(out->h, 8) * cdiv(out->w, 16) * ncoblk * nd * 4096 * 4;
  // from 64 workgroups on whole samples only: a shard's sums are those of the views that tile it
  if (wgs >= 64 && (!room || out->d != out->d_global || out->halo_lo || out->halo_hi)) return 1;
  int s = (int)std::min<int64_t>(nchunks, wgs < 64 ? cdiv(256, wgs) : std::max<int64_t>(1, num_cu / wgs));
  while (s > 1 && s * part > ((int64_t)(wgs < 64 ? 24 : 40) << 20)) --s;
  // from 64 workgroups on a split has to save more of a tile's 6 us a chunk than its sums and the launch that adds them take: 256->256 on
  // 8 x 8^3 101 -> 52 us, on 2 x 16^3 100 -> 58, 128->128 on 8 x 8x16x16 53 -> 45
  if (wgs >= 64 && s > 1 && 6.0 * (nchunks - (double)cdiv(nchunks, s)) < 8.0 + 4e-7 * (double)(s * part)) return 1;
  const int cps = (int)cdiv(nchunks, s);
  return (int)cdiv(nchunks, cps);
}

bool mfma_fwd_supported(const h3d_tensor* in, const h3d_tensor* out) {
  if (in->dtype != H3D_BF16) return false;
  if (in->c < 1 || out->c < 1) return false;
  // 32-bit in-sample offsets inside the kernel
  // buffer loads address a whole sample (all channels) with 31-bit byte offsets
  return sample_span(in) < ((int64_t)1 << 30) && sample_span(out) < ((int64_t)1 << 30);
}

static void wp_dims(int cin_k, int cout_k, int* nchunks, int* ncoblk) {
  *nchunks = (int)cdiv(cin_k, CI_CHUNK);
  *ncoblk = (int)cdiv(cout_k, 32);
}

// floats of ONE split's partial tiles: the split kernels are the narrow-volume instances (16-column blocks, 8 rows)
static size_t split_part_floats(const h3d_tensor* out) {
  const int ncoblk = (int)cdiv(out->c, 32), nd = out->c > 32 ? 4 : 8;
  const int64_t ds = out->halo_lo + out->d + out->halo_hi;
  return (size_t)((int64_t)out->n * cdiv(ds, nd) * cdiv(out->h, 8) * cdiv(out->w, 16)) * ncoblk * nd * 4096;
}

static size_t mfma_wp_bytes(const h3d_tensor* in, const h3d_tensor* out) {
  int nchunks, ncoblk;
  wp_dims(in->c, out->c, &nchunks, &ncoblk);
  return ((size_t)ncoblk * nchunks * 27 * 512 * sizeof(bf16_t) + 255) & ~(size_t)255;
}

template <typename T>
h3d_status conv3d_direct(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const void* w, const float* bias, h3d_tensor* out, bool transpose,
                         float out_slope, float mask_slope, void* ws, size_t ws_bytes, hipStream_t stream);
bool conv3d_thin_supported(const h3d_tensor* in, const h3d_tensor* out);
h3d_status conv3d_thin(void* handle, const h3d_tensor* in, const void* w, const float* bias, h3d_tensor* out, bool transpose,
                       float out_slope, void* ws, hipStream_t stream);

// Backward-data onto at most 4 channels from 17 to 32 (the first layer of the U-Net-shaped level: 32 -> 1): the
// row-streaming thin kernel holds 16 input channels in its LDS ring, so the sum over the channels is taken in two
// passes, channels 0-15 into dx and the rest into a buffer of dx's size in the workspace, and the two are added:
// dx = bf16(bf16(sum over the first 16) + bf16(sum over the others)), one rounding more than a single pass.
// `in` is split into two channel-range views; both must be shapes of the row-streaming variant.
constexpr size_t THIN2_WP_BYTES = 16384;
static bool thin_two_pass_shape(const h3d_tensor* in, const h3d_tensor* out, h3d_tensor* ia, h3d_tensor* ib) {
  if (in->dtype != H3D_BF16 || in->c <= 16 || in->c > 32 || out->c < 1 || out->c > 4 || !is_packed(out)) return false;
  if (in->w % 8 || out->h < 8 || (uintptr_t)in->data % 16 || (out->data && (uintptr_t)out->data % 16)) return false;
  const Geo g = make_geo(in);
  if (g.cstride % 8) return false;
  h3d_tensor a = *in, b = *in;
  a.c = 16; a.c_stride = g.cstride; a.n_stride = g.nstride;
  b.c = in->c - 16; b.c_stride = g.cstride; b.n_stride = g.nstride;
  b.data = in->data ? (void*)((bf16_t*)in->data + 16 * g.cstride) : nullptr;
  if (!conv3d_thin_supported(&a, out) || !conv3d_thin_supported(&b, out)) return false;
  if (ia) *ia = a;
  if (ib) *ib = b;
  return true;
}
static size_t thin_two_pass_ws_bytes(const h3d_tensor* out) {
  return THIN2_WP_BYTES + (size_t)out->n * out->c * (out->halo_lo + out->d + out->halo_hi) * out->h * out->w * sizeof(bf16_t);
}
// dst[i] = bf16(dst[i] + src[i]), 8 elements per thread (n8 groups), then the tail one by one
__global__ void __launch_bounds__(256) add_bf16_kernel(bf16_t* __restrict__ dst, const bf16_t* __restrict__ src, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i + 8 <= n) {
    uint4 a = *reinterpret_cast<const uint4*>(dst + i);
    const uint4 b = *reinterpret_cast<const uint4*>(src + i);
    auto add2 = [](uint32_t x, uint32_t y) {
      return pack_bf16x2(__uint_as_float(x << 16) + __uint_as_float(y << 16),
                         __uint_as_float(x & 0xffff0000u) + __uint_as_float(y & 0xffff0000u));
    };
    a.x = add2(a.x, b.x); a.y = add2(a.y, b.y); a.z = add2(a.z, b.z); a.w = add2(a.w, b.w);
    *reinterpret_cast<uint4*>(dst + i) = a;
  } else {
    for (int64_t j = i; j < n; ++j) dst[j] = f32_to_bf16(bf16_to_f32(dst[j]) + bf16_to_f32(src[j]));
  }
}

// Wide volumes of few tiles: a tile takes 4.4 us a chunk of 16 input channels however many others run (measured for 1 to 256 of them), so the
// chunks of one are split over workgroups as long as these fit the CUs and the partial sums (128 KB a tile, block of 32 channels and split, written
// and read at about 6 TB/s) and the launch that adds them cost less than is saved.  Whole samples only: on a shard the sum of a voxel does not
// depend on the tiles of the call, so that a main part and halo strips have the bits of one call.  us, whole and split: 256->64 on 16x32x32 81 and
// 33, 256->256 on 8x32x32 85 and 46, 128->96 on 16x16x32 46 and 25, 192->64 on 6x16x34 60 and 28, 64->32 on 8x16x24 25 and 18, 64->64 on 16x32x32
// 28 and 25.
static bool wide_dims(const h3d_tensor* in, const h3d_tensor* out) {
  return out->w > 16 && out->halo_lo + out->d + out->halo_hi >= 3 && out->h >= 4;
}
static int64_t wide_units(const h3d_tensor* out) {
  return (int64_t)out->n * cdiv(out->halo_lo + out->d + out->halo_hi, 4) * cdiv(out->h, 8) * cdiv(out->w, 32) * cdiv(out->c, 32);
}
static int wide_splits(const h3d_tensor* in, const h3d_tensor* out, int num_cu) {
  const int nchunks = (int)cdiv(in->c, CI_CHUNK);
  if (nchunks < 2 || !wide_dims(in, out) || !is_packed(out) || out->d != out->d_global || out->halo_lo || out->halo_hi) return 1;
  const int64_t units = wide_units(out);
  int best = 1;
  double cost = 4.4 * nchunks;
  for (int s = 2; s <= nchunks && s * units <= num_cu; ++s) {
    const double c = 4.4 * cdiv(nchunks, s) + 4.0 + 0.045 * (double)(s * units);
    if (cdiv(nchunks, cdiv(nchunks, s)) == s && c < cost) { cost = c; best = s; }
  }
  return best;
}
static size_t wide_split_bytes(const h3d_tensor* in, const h3d_tensor* out, int num_cu) {
  const int s = wide_splits(in, out, num_cu);
  return s > 1 ? (size_t)(s * wide_units(out)) * 131072 : 0;
}

// what a call needs without copies; less room, down to what is left without the splits that can be left out, is taken too (the sums are then one
// chain): a workspace that is large enough for a larger volume, which is not split, does for this one
static size_t mfma_base_ws_bytes(const h3d_tensor* in, const h3d_tensor* out, int num_cu, bool room) {
  size_t b = mfma_wp_bytes(in, out) + (room ? wide_split_bytes(in, out, num_cu) : 0);
  if (thin_two_pass_shape(in, out, nullptr, nullptr)) b = std::max(b, thin_two_pass_ws_bytes(out));
  const int s = mfma_splits(in, out, num_cu, room);
  if (s > 1) b += (size_t)s * split_part_floats(out) * sizeof(float);
  return b;
}

template <int NCB, int ND, int TWC, bool MASKED, bool VEC, bool SPLIT, bool FLAT, int ROW>
static h3d_status launch_variant_as(void* handle, const bf16_t* in, const bf16_t* mask, const uint4* wp, const float* bias,
                                 bf16_t* out, MfmaArgs a, int n, hipStream_t stream) {
  constexpr int RPB = 32 / TWC, TH = 4 * RPB;
  constexpr int P = TWC == 32 ? 36 : 20;
  constexpr int TDP = FLAT ? 1 : ND, THT = FLAT ? TH * ND : TH;
  constexpr size_t lds_bytes = (size_t)2 * 2 * (TDP + 2) * (THT + 2) * P * 16;
  a.tiles_w = (int)cdiv(a.out.w, TWC);
  a.tiles_h = (int)cdiv(a.out.h, THT);
  a.tiles_d = (int)cdiv(a.out.ds, TDP);
  int64_t ntiles = (int64_t)n * a.tiles_d * a.tiles_h * a.tiles_w;
  int64_t gy = cdiv(a.ncoblk, NCB);
  if (ntiles >= ((int64_t)1 << 31) || gy > 65535) return fail(handle, H3D_EINVAL, "conv3d: too many workgroups");
  a.ntiles = (int)ntiles;
  // one resident workgroup per CU (LDS-limited), spread over the output-channel groups
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  int64_t gx = std::min<int64_t>(ntiles, std::max<int64_t>(1, num_cu / (gy * a.csplit)));
  auto kern = conv3d_mfma_kernel<NCB, ND, TWC, MASKED, VEC, SPLIT, FLAT, ROW>;
  static bool attr_set = false;   // per instantiation
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess)
      return fail(handle, H3D_EHIP, "conv3d: cannot raise the dynamic LDS limit to %zu bytes", lds_bytes);
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)gy, (unsigned)a.csplit), dim3(WG_THREADS), lds_bytes, stream, in, mask, wp,
                     a.csplit > 1 ? nullptr : bias, out, a);
  note_kernel(handle, "conv3d_mfma_kernel<%d,%d,%d,%d,%d,%d,%d,%d>", NCB, ND, TWC, (int)MASKED, (int)VEC, (int)SPLIT, (int)FLAT, ROW);
  if (a.csplit > 1) return hipGetLastError() == hipSuccess ? H3D_OK : fail(handle, H3D_EHIP, "conv3d_mfma: launch failed");
  return launch_status(handle, "conv3d_mfma");
}

template <int NCB, int ND, int TWC, bool MASKED, bool VEC, bool SPLIT = false, bool FLAT = false>
static h3d_status launch_variant(void* handle, const bf16_t* in, const bf16_t* mask, const uint4* wp, const float* bias,
                                 bf16_t* out, const MfmaArgs& a, int n, hipStream_t stream) {
  if constexpr (TWC == 16 && VEC && !MASKED) {
    if (a.in.w % 8 == 0 && (uintptr_t)in % 16 == 0 && a.in.cstride % 8 == 0 && a.in.nstride % 8 == 0)
      return a.pairs && a.in.w == a.out.w ? launch_variant_as<NCB, ND, TWC, MASKED, VEC, SPLIT, FLAT, 1>(handle, in, mask, wp, bias, out, a, n, stream)
                                          : launch_variant_as<NCB, ND, TWC, MASKED, VEC, SPLIT, FLAT, 2>(handle, in, mask, wp, bias, out, a, n, stream);
  }
  return launch_variant_as<NCB, ND, TWC, MASKED, VEC, SPLIT, FLAT, 0>(handle, in, mask, wp, bias, out, a, n, stream);
}

static bool wide_shape(const MfmaArgs& a) {
  return a.out.w > 16 && a.out.ds >= 3 && a.out.h >= 4;
}

template <int CB, int WCB = 1, int RSP = 1, bool RAGGED = false, bool SPLIT = false, bool POOL = false>
static h3d_status launch_wide(void* handle, const bf16_t* in, const uint4* wp, const float* bias, bf16_t* out, MfmaArgs a, int n,
                              hipStream_t stream) {
  if constexpr (!RAGGED && !SPLIT && !POOL)
    if (a.out.w & 1) return launch_wide<CB, WCB, RSP, true>(handle, in, wp, bias, out, a, n, stream);
  constexpr size_t lds_bytes = (size_t)2 * 2 * 6 * 10 * 36 * 16 + WCB * CB * 64 * 16;     // two stage buffers + the bias fragments
  a.tiles_w = (int)cdiv(a.out.w, 32);
  a.tiles_h = (int)cdiv(a.out.h, 8);
  a.tiles_d = (int)cdiv(a.out.ds, 4);
  const int64_t ntiles = (int64_t)n * a.tiles_d * a.tiles_h * a.tiles_w;
  const int64_t gy = cdiv(a.ncoblk, CB * WCB);
  if (ntiles >= ((int64_t)1 << 31) || gy > 65535) return fail(handle, H3D_EINVAL, "conv3d: too many workgroups");
  a.ntiles = (int)ntiles;
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  const int64_t gx = std::min<int64_t>(ntiles, std::max<int64_t>(1, num_cu / (gy * a.csplit)));
  auto kern = conv3d_mfma_wide_kernel<CB, WCB, RSP, RAGGED, SPLIT, POOL>;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess)
      return fail(handle, H3D_EHIP, "conv3d: cannot raise the dynamic LDS limit to %zu bytes", lds_bytes);
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)gy, (unsigned)a.csplit), dim3(256 * WCB * RSP), lds_bytes, stream, in, wp, SPLIT ? nullptr : bias, out, a);
  note_kernel(handle, "conv3d_mfma_wide_kernel<%d,%d,%d,%d>%s", CB, WCB, RSP, (int)RAGGED, SPLIT ? " (split)" : POOL ? " (max-pooled)" : "");
  if constexpr (SPLIT) {
    const int64_t total = (int64_t)n * a.cout_k * a.out.ds * a.out.h * cdiv(a.out.w, 4);
    const int vec = a.out.w % 4 == 0 && a.out.cstride % 4 == 0 && a.out.nstride % 4 == 0 && (uintptr_t)out % 8 == 0;
    hipLaunchKernelGGL(conv_wide_split_reduce_kernel, dim3((unsigned)cdiv(total, 256)), dim3(256), 0, stream, (const float*)a.part, bias, out, a, (uint32_t)total, vec);
  }
  return launch_status(handle, "conv3d_mfma_wide");
}

// ---- prepared input (prep.h): the wide kernel takes neither a fused mask nor rows of odd length.  Where it takes the shape
// otherwise, the input is copied, masked and padded, slab by slab, and the wide kernel runs on the copy: same products, same order,
// same bits as the general kernel.  The copy is bounded; without the workspace for it the general kernel runs.
// Backward-data of masked layers, before -> after: 64->64 on 4 x 64^3 345 -> 265 us, 128->128 on 2 x 40x100x100 1140 -> 830,
// 24->48 on 2 x 22x50x54 52 -> 36, and down to a few tiles and channels: 16->32 on 4x8x20 30 -> 19, 4->16 on 16x32x32 23 -> 16, 1->32 on
// 32x64x64 36 -> 26; rows of odd length, 64->64 on 64x128x127: forward 402 -> 267, backward-data 416 -> 261.
// The budget: 64 MiB leaves slabs too small for the two-block form at 64 channels (267 -> 308 us on the last one).
constexpr int64_t PREP_FWD_BUDGET = (int64_t)160 << 20;

static int64_t prep_plane_bytes(const h3d_tensor* in) { return (int64_t)in->c * in->h * prep_w(in->w) * 2; }
// workspace for the copies behind the packed weights; 0: no prepared form
static size_t prep_fwd_bytes(const h3d_tensor* in, const h3d_tensor* out) {
  if (in->n < 1 || !wide_dims(in, out)) return 0;
  PrepTiling t;
  if (!prep_tiling(in->n, out->halo_lo + out->d + out->halo_hi, prep_plane_bytes(in), 2, PREP_FWD_BUDGET, &t)) return 0;
  return up256((size_t)t.nn * (t.np + 2) * prep_plane_bytes(in));
}

// Volumes of at most 16 columns: rows of odd length are staged element by element, masked ones with the mask's loads beside their own.  A
// masked, padded copy of the whole tensor goes through the 16-byte staging instead.  us, before and on the copy: masked backward-data 256->32
// on 53x48x11 240 and 56, 128->96 on 8 x 5x80x16 130 and 104, 256->256 on 8 x 8^3 132 and 104, 16->2 on 2 x 8x32x15 56 and 20, 16->16 on 4x8x8 22
// and 17; odd rows without a mask, 128->128 on 8 x 9x48x9 162 and 110, 16->24 on 9x32x13 25 and 21.  Unmasked rows of even length gain nothing
// (11->96 on 8 x 64x10x10 26 and 27, 96->11 there 45 and 53): pairs of elements from the tensor itself.
static size_t prep_narrow_bytes(const h3d_tensor* in, const h3d_tensor* out) {
  if (in->n < 1 || out->w > 16 || in->c < 1) return 0;
  const int64_t bytes = ((int64_t)in->halo_lo + in->d + in->halo_hi) * in->n * prep_plane_bytes(in);
  return bytes <= PREP_FWD_BUDGET ? up256((size_t)bytes) : 0;
}

// backward-data may come with a mask, which is not known here; forward needs the copy for rows of odd length only
size_t mfma_fwd_ws_bytes(void* handle, const h3d_tensor* in, const h3d_tensor* out, bool backward_data) {
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  size_t b = mfma_base_ws_bytes(in, out, num_cu, true);
  if (backward_data || in->w % 2)
    b = std::max(mfma_wp_bytes(in, out) + wide_split_bytes(in, out, num_cu) + prep_fwd_bytes(in, out), b + prep_narrow_bytes(in, out));
  return b;
}

// Two channel blocks a workgroup, or one with the rows of a plane over two wavefronts (same sums in the same order): a tile takes 0.58 to 0.64 times
// as long with one, so it pays where the tiles, or an odd number of blocks, divide badly over the CUs.  us, two blocks and one: 64->64
// on 4 x 8x134x54 (272 tiles) 81 and 75, 128->96 on 16x112x160 231 and 197, 256->96 446 and 375, 32->51 on 58x96x64 52 and 47, 64->64 on 24x48x48 41
// and 29; but on 32x128x128 (512 tiles) 97 and 113, 24->48 on 2 x 22x50x54 31 and 36, 22->96 on 8 x 24x64x53 170 and 172
static bool one_block(void* handle, int64_t ntiles, int64_t ncoblk) {
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  auto rounds = [&](int64_t gy) { return cdiv(ntiles, std::max<int64_t>(1, num_cu / gy)); };
  return 62 * rounds(ncoblk) < 100 * rounds(cdiv(ncoblk, 2));
}

static h3d_status wide_conv(void* handle, const bf16_t* ip, const uint4* wq, const float* bias, bf16_t* op, const MfmaArgs& a, int n,
                            hipStream_t stream) {
  const int64_t ntiles = (int64_t)n * cdiv(a.out.ds, 4) * cdiv(a.out.h, 8) * cdiv(a.out.w, 32);
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  if (a.csplit > 1) return launch_wide<1, 1, 2, false, true>(handle, ip, wq, bias, op, a, n, stream);
  if (a.cout_k > 32) {
    if (one_block(handle, ntiles, a.ncoblk)) return launch_wide<1, 1, 2>(handle, ip, wq, bias, op, a, n, stream);
    return launch_wide<1, 2>(handle, ip, wq, bias, op, a, n, stream);
  }
  // one block of output channels: with short channel loops (at most 32 input channels) or few tiles the eight-wavefront
  // form that splits the rows of a plane measured faster (32->16 on 4 x 64^3 0.068 -> 0.062 ms, 32->1 on the U-Net
  // shard 0.239 -> 0.222), with four chunks and many tiles slower (64->32 on the U-Net shard 0.480 -> 0.490)
  if (a.nchunks <= 2 || ntiles < 2 * num_cu) return launch_wide<1, 1, 2>(handle, ip, wq, bias, op, a, n, stream);
  return launch_wide<1, 1>(handle, ip, wq, bias, op, a, n, stream);
}

// pack: the weights, to the start of the workspace, beside the first copy
static h3d_status prep_conv(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const float* bias, h3d_tensor* out, MfmaArgs a,
                            float mask_slope, void* ws, size_t split_bytes, const TapsPackJob& pack, hipStream_t stream) {
  const int planes = out->halo_lo + out->d + out->halo_hi, w8 = prep_w(in->w);
  PrepTiling t;
  if (!prep_tiling(in->n, planes, prep_plane_bytes(in), 2, PREP_FWD_BUDGET, &t)) return H3D_OK;     // (nothing to compute)
  bf16_t* copy = reinterpret_cast<bf16_t*>(static_cast<char*>(ws) + mfma_wp_bytes(in, out) + split_bytes);
  const Geo gi = make_geo(in), go = make_geo(out);
  for (int i = 0; i < t.count(); ++i) {
    const PrepSlab b = t.at(i);
    const int a0 = b.p0 - out->halo_lo, a1 = a0 + b.np;             // output planes, interior-relative
    // input planes of the slab that lie inside the volume (all of them are stored)
    const int lo = (int)std::max<int64_t>(a0 - 1, -gi.doff), hi = (int)std::min<int64_t>(a1 + 1, gi.dglob - gi.doff);
    const int np = std::max(hi - lo, 0);
    const PrepJob j = prep_job(in, mask, mask_slope, b.n0, b.nn, lo, np, copy);
    H3D_TRY(prep_launch(handle, j, nullptr, stream, i ? nullptr : &pack));
    MfmaArgs s = a;
    s.in.n = b.nn; s.in.d = b.np; s.in.w = w8; s.in.doff = gi.doff + a0; s.in.hlo = a0 - lo; s.in.ds = np; s.in.hhi = np - b.np - s.in.hlo;
    s.in.plane = (int64_t)in->h * w8; s.in.cstride = s.in.plane * np; s.in.nstride = s.in.cstride * in->c;
    s.out.n = b.nn; s.out.d = s.out.ds = b.np; s.out.hlo = s.out.hhi = 0; s.out.doff = go.doff + a0;
    H3D_TRY(wide_conv(handle, copy, (const uint4*)ws, bias, (bf16_t*)out->data + b.n0 * go.nstride + (int64_t)b.p0 * go.plane, s, b.nn, stream));
  }
  return H3D_OK;
}

template <bool MASKED, bool VEC>
static h3d_status pick_variant(void* handle, const bf16_t* in, const bf16_t* mask, const uint4* wp, const float* bias,
                               bf16_t* out, const MfmaArgs& a, int n, hipStream_t s) {
  const bool wide = a.out.w > 16;
  const bool two_cb = a.cout_k > 32;
  // one- or two-plane outputs with more than 32 channels and enough rows: the row-group layout
  const bool flat = two_cb && a.out.ds <= 2 && a.csplit == 1;
  if (flat && wide && a.out.h >= 16) return launch_variant<2, 4, 32, MASKED, VEC, false, true>(handle, in, mask, wp, bias, out, a, n, s);
  if (flat && !wide && a.out.h >= 32) return launch_variant<2, 4, 16, MASKED, VEC, false, true>(handle, in, mask, wp, bias, out, a, n, s);
  // a wide volume whose channels are split, without a copy of its masked or odd rows: the wide kernel's splits and sums (its partial tiles of 8 rows
  // hold these of 4), one block of output channels in half of the wavefronts
  if (wide && a.csplit > 1) return launch_variant<2, 4, 32, MASKED, VEC, true>(handle, in, mask, wp, bias, out, a, n, s);
  if (wide) {
    return two_cb ? launch_variant<2, 4, 32, MASKED, VEC>(handle, in, mask, wp, bias, out, a, n, s)
                  : launch_variant<1, 8, 32, MASKED, VEC>(handle, in, mask, wp, bias, out, a, n, s);
  }
  if (a.csplit > 1)
    return two_cb ? launch_variant<2, 4, 16, MASKED, VEC, true>(handle, in, mask, wp, bias, out, a, n, s)
                  : launch_variant<1, 8, 16, MASKED, VEC, true>(handle, in, mask, wp, bias, out, a, n, s);
  return two_cb ? launch_variant<2, 4, 16, MASKED, VEC>(handle, in, mask, wp, bias, out, a, n, s)
                : launch_variant<1, 8, 16, MASKED, VEC>(handle, in, mask, wp, bias, out, a, n, s);
}

h3d_status conv3d_mfma(void* handle, const h3d_tensor* in, const h3d_tensor* mask, const void* w, const float* bias,
                       h3d_tensor* out, bool transpose, float out_slope, float mask_slope, void* ws, size_t ws_bytes,
                       hipStream_t stream) {
  MfmaArgs a;
  a.in = make_geo(in);
  a.mask = mask ? make_geo(mask) : a.in;
  a.out = make_geo(out);
  a.cin_k = in->c; a.cout_k = out->c;
  wp_dims(a.cin_k, a.cout_k, &a.nchunks, &a.ncoblk);
  a.out_slope = out_slope; a.mask_slope = mask_slope;
  if ((int64_t)out->n * a.out.ds * out->h * out->w == 0) return H3D_OK;
  const int num_cu = static_cast<Handle*>(handle)->num_cu;
  const bool room = ws_bytes >= mfma_base_ws_bytes(in, out, num_cu, true);
  if (!ws || ws_bytes < mfma_base_ws_bytes(in, out, num_cu, false)) return fail(handle, H3D_EWORKSPACE, "conv3d: workspace too small");
  if ((uintptr_t)ws % 16) return fail(handle, H3D_EWORKSPACE, "conv3d: workspace must be 16-byte aligned");
  // a handful of output channels from at most 16 input channels: the tap-row-folding kernel
  if (!mask && conv3d_thin_supported(in, out)) return conv3d_thin(handle, in, w, bias, out, transpose, out_slope, ws, stream);
  // .. from 17 to 32 channels, backward-data without bias and activation: two passes of it
  h3d_tensor ia, ib;
  if (!mask && transpose && !bias && out_slope == 1.f && thin_two_pass_shape(in, out, &ia, &ib)) {
    h3d_tensor tmp = *out;
    tmp.data = static_cast<char*>(ws) + THIN2_WP_BYTES;
    H3D_TRY(conv3d_thin(handle, &ia, w, nullptr, out, true, 1.f, ws, stream));
    // transposed packing reads w[c][m][tap] with c the channel of `in`: the second half starts 16 rows further on
    H3D_TRY(conv3d_thin(handle, &ib, (const bf16_t*)w + (size_t)16 * out->c * 27, nullptr, &tmp, true, 1.f, ws, stream));
    const int64_t n = (int64_t)out->n * a.out.nstride;
    hipLaunchKernelGGL(add_bf16_kernel, dim3((unsigned)cdiv(cdiv(n, 8), 256)), dim3(256), 0, stream, (bf16_t*)out->data,
                       (const bf16_t*)tmp.data, n);
    note_kernel(handle, "conv3d_thin_roll (two passes)");
    return launch_status(handle, "conv3d_thin_two_pass");
  }
  const bool vec = (in->w % 2 == 0) && ((uintptr_t)in->data % 4 == 0) && ((uintptr_t)out->data % 4 == 0) &&
                   (!mask || (uintptr_t)mask->data % 4 == 0);
  const int cin = transpose ? a.cout_k : a.cin_k, cout = transpose ? a.cin_k : a.cout_k;
  const TapsPackJob pack = taps_pack_job(w, ws, cin, cout, transpose ? TAPS_REVERSED : TAPS_FWD, a.nchunks, 27);
  const bf16_t* ip = (const bf16_t*)in->data;
  const bf16_t* mp = mask ? (const bf16_t*)mask->data : nullptr;
  bf16_t* op = (bf16_t*)out->data;
  const uint4* wq = (const uint4*)ws;
  a.csplit = mfma_splits(in, out, num_cu, room);
  a.chunks_per_split = (int)cdiv(a.nchunks, a.csplit);
  a.part = a.csplit > 1 ? reinterpret_cast<float*>(static_cast<char*>(ws) + mfma_wp_bytes(in, out)) : nullptr;
  h3d_status st;
  const size_t split_bytes = room ? wide_split_bytes(in, out, num_cu) : 0;
  if (split_bytes) {      // (wide volumes: mfma_splits is 1)
    a.csplit = wide_splits(in, out, num_cu);
    a.chunks_per_split = (int)cdiv(a.nchunks, a.csplit);
    a.part = reinterpret_cast<float*>(static_cast<char*>(ws) + mfma_wp_bytes(in, out));
  }
  // Also where half of the only chunk is padding (at most 8 input and 32 output channels).  us, general kernel and here: 8->32 on 32x64x64 18.5 and 14.1,
  // 8->16 on 64x128x128 47 and 37, on copies masked backward-data of 16->8 on 4 x 16x64x64 29.6 and 17.9, 8->8 on 9x30x41 71 and 15.6
  if (!mask && vec && wide_shape(a)) {
    taps_pack(pack, stream);
    return wide_conv(handle, ip, wq, bias, op, a, out->n, stream);
  }
  if (const size_t copies = prep_fwd_bytes(in, out); copies && (uintptr_t)out->data % 4 == 0 && ws_bytes >= mfma_wp_bytes(in, out) + split_bytes + copies)
    return prep_conv(handle, in, mask, bias, out, a, mask_slope, ws, split_bytes, pack, stream);
  a.pairs = vec;
  if (const size_t copy = mask || in->w % 2 ? prep_narrow_bytes(in, out) : 0; copy && ws_bytes >= mfma_base_ws_bytes(in, out, num_cu, room) + copy) {
    // the planes that the output's window reaches inside the volume (all of them are stored), behind whatever else the workspace holds
    bf16_t* dst = reinterpret_cast<bf16_t*>(static_cast<char*>(ws) + mfma_base_ws_bytes(in, out, num_cu, room));
    const int lo = (int)std::max<int64_t>(-out->halo_lo - 1, -a.in.doff), hi = (int)std::min<int64_t>(out->d + out->halo_hi + 1, a.in.dglob - a.in.doff);
    H3D_TRY(prep_launch(handle, prep_job(in, mask, mask_slope, 0, in->n, lo, hi - lo, dst), nullptr, stream, &pack));
    a.in.w = prep_w(in->w); a.in.ds = hi - lo; a.in.hlo = -lo; a.in.hhi = hi - in->d;
    a.in.plane = (int64_t)in->h * a.in.w; a.in.cstride = a.in.plane * a.in.ds; a.in.nstride = a.in.cstride * in->c;
    a.pairs = out->w % 2 == 0 && (uintptr_t)out->data % 4 == 0 && a.out.cstride % 2 == 0 && a.out.nstride % 2 == 0;
    st = pick_variant<false, true>(handle, dst, nullptr, wq, bias, op, a, out->n, stream);
  } else if (mask && sample_span(mask) >= ((int64_t)1 << 30)) {      // (the copies above address it in 64 bits)
    return conv3d_direct<bf16_t>(handle, in, mask, w, bias, out, transpose, out_slope, mask_slope, ws, ws_bytes, stream);
  } else {
    taps_pack(pack, stream);
    if (mask) st = vec ? pick_variant<true, true>(handle, ip, mp, wq, bias, op, a, out->n, stream)
                       : pick_variant<true, false>(handle, ip, mp, wq, bias, op, a, out->n, stream);
    else st = vec ? pick_variant<false, true>(handle, ip, mp, wq, bias, op, a, out->n, stream)
                  : pick_variant<false, false>(handle, ip, mp, wq, bias, op, a, out->n, stream);
  }
  if (st != H3D_OK || a.csplit == 1) return st;
  const int64_t out_total = (int64_t)out->n * a.out.nstride;
  SplitGeo q;
  const bool wide = a.out.w > 16;
  q.nd = wide || a.cout_k > 32 ? 4 : 8; q.twc = wide ? 32 : 16; q.rpb = wide ? 1 : 2; q.ncoblk = a.ncoblk;
  q.tiles_w = (int)cdiv(a.out.w, q.twc); q.tiles_h = (int)cdiv(a.out.h, 4 * q.rpb); q.tiles_d = (int)cdiv(a.out.ds, q.nd);
  q.ntiles = out->n * q.tiles_d * q.tiles_h * q.tiles_w;
  hipLaunchKernelGGL(conv_split_reduce_kernel, dim3((unsigned)cdiv(out_total, 256)), dim3(256), 0, stream, (const float*)a.part, bias, op,
                     a.out, q, a.csplit, out_slope);
  return launch_status(handle, "conv3d_split_reduce");
}

// Forward and 2x2x2 max pooling in one launch, for what h3d_conv3d_fwd gives to the wide kernel unsplit and without a copy: pairs of planes, rows and
// columns that begin with the tensor, and whole pairs of pooled voxels in a row.  The pooled tensor is written through 31-bit byte offsets too, and its
// halos, which nothing here bounds, can make it larger than z.
bool wide_pool_supported(void* handle, const h3d_tensor* in, const h3d_tensor* z, const h3d_tensor* y) {
  if (!mfma_fwd_supported(in, z) || y->dtype != H3D_BF16 || conv3d_thin_supported(in, z) || !wide_dims(in, z)) return false;
  if (z->halo_lo || z->halo_hi || z->d % 2 || z->h % 2 || z->w % 4 || !is_packed(y) || sample_span(y) >= ((int64_t)1 << 30)) return false;
  if ((uintptr_t)in->data % 4 || (uintptr_t)z->data % 4 || (uintptr_t)y->data % 4) return false;
  return z->n > 0 && wide_splits(in, z, static_cast<Handle*>(handle)->num_cu) == 1;
}
h3d_status conv3d_wide_pool(void* handle, const h3d_tensor* in, const void* w, const float* bias, h3d_tensor* z, h3d_tensor* y, float out_slope, void* ws,
                            size_t ws_bytes, hipStream_t stream) {
  MfmaArgs a;
  a.in = a.mask = make_geo(in); a.out = make_geo(z); a.yp = make_geo(y);
  a.cin_k = in->c; a.cout_k = z->c;
  wp_dims(a.cin_k, a.cout_k, &a.nchunks, &a.ncoblk);
  a.out_slope = out_slope; a.mask_slope = 1.f;
  a.csplit = 1; a.chunks_per_split = a.nchunks; a.pairs = 1; a.part = nullptr;
  a.ypool = (bf16_t*)y->data;
  if (!ws || ws_bytes < mfma_base_ws_bytes(in, z, static_cast<Handle*>(handle)->num_cu, false)) return fail(handle, H3D_EWORKSPACE, "conv3d: workspace too small");
  if ((uintptr_t)ws % 16) return fail(handle, H3D_EWORKSPACE, "conv3d: workspace must be 16-byte aligned");
  taps_pack(taps_pack_job(w, ws, a.cin_k, a.cout_k, TAPS_FWD, a.nchunks, 27), stream);
  const int64_t ntiles = (int64_t)z->n * cdiv(a.out.ds, 4) * cdiv(a.out.h, 8) * cdiv(a.out.w, 32);
  const bf16_t* ip = (const bf16_t*)in->data;
  const uint4* wq = (const uint4*)ws;
  bf16_t* op = (bf16_t*)z->data;
  return one_block(handle, ntiles, a.ncoblk) || a.cout_k <= 32 ? launch_wide<1, 1, 2, false, false, true>(handle, ip, wq, bias, op, a, z->n, stream)
                                                               : launch_wide<1, 2, 1, false, false, true>(handle, ip, wq, bias, op, a, z->n, stream);
}

}  // namespace h3d
