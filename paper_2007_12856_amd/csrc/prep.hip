// The copy kernel behind prepared operands (prep.h).
#include "prep.h"
#include "rowload.h"

#include <algorithm>

namespace h3d {

// HBM: 2 B read (4 with a mask) and 2 B written per element.  A thread owns one 16-byte unit of the copy.  Source rows may start
// at any 2-byte address (unaligned 16-byte loads); the last unit of a ragged row is loaded so that it ends with the row, and
// shifted.
__device__ __forceinline__ uint4 prep_load(const bf16_t* row, int col, int w) {
  if (w < 8) {                                   // (col is 0)
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = i < w ? (uint32_t)row[i] : 0u;
    return uint4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
  }
  const int back = max(col + 8 - w, 0);          // 0 except in the last unit of a ragged row
  uint4 v;
  __builtin_memcpy(&v, row + col - back, 16);
  return shift8(v, back);
}
// the elements whose saved output is positive (or those whose isn't), as they are
__device__ __forceinline__ uint32_t prep_part2(uint32_t v, uint32_t m, bool positive) {
  const bool k0 = (__uint_as_float(m << 16) > 0.f) == positive, k1 = (__uint_as_float(m & 0xffff0000u) > 0.f) == positive;
  return v & ((k0 ? 0xffffu : 0u) | (k1 ? 0xffff0000u : 0u));
}
__device__ __forceinline__ void prep_unit(const PrepJob& a, int64_t i) {
  if (i >= a.units) return;
  const int wu = a.w8 / 8;
  int64_t t = i;
  const int u = (int)(t % wu); t /= wu;
  const int h = (int)(t % a.s.h); t /= a.s.h;
  const int p = (int)(t % a.np); t /= a.np;
  const int c = (int)(t % a.s.c);
  const int n = (int)(t / a.s.c) + a.n0;
  const int col = 8 * u;
  uint4 v = prep_load(a.src + n * a.s.nstride + c * a.s.cstride + (int64_t)(a.p0 + p + a.s.hlo) * a.s.plane + (int64_t)h * a.s.w, col, a.s.w);
  if (a.msk) {
    const uint4 m = prep_load(a.msk + n * a.m.nstride + c * a.m.cstride + (int64_t)(a.p0 + p + a.m.hlo) * a.m.plane + (int64_t)h * a.m.w, col, a.m.w);
    if (a.part) {      // a branch, not a choice of values: every thread would compute both (24->48 on 2 x 22x50x54, three passes: 121 and 119 us)
      const bool pos = a.part == 1;
      v = uint4{prep_part2(v.x, m.x, pos), prep_part2(v.y, m.y, pos), prep_part2(v.z, m.z, pos), prep_part2(v.w, m.w, pos)};
    } else {
      v = mask8(v, m, a.slope);
    }
  }
  reinterpret_cast<uint4*>(a.dst)[i] = v;
}

// PACK: the first workgroups pack a filter.  A launch of its own holds up a queue of small ones for 4.7 us, here most of it hides behind the copy:
// masked backward-data of 24->48 on 2 x 22x50x54 32.9 -> 30.4 us, 64->64 on 16x32x32 29.2 -> 27.0, on 4 x 64^3 264 -> 254, odd rows forward 64->64 on
// 16x32x33 32.0 -> 30.2.
template <bool PACK>
__global__ void __launch_bounds__(256) prep_kernel(PrepJob a, PrepJob b, int64_t blocks_a, TapsPackJob pack, int blocks_p) {
  if (PACK && (int)blockIdx.x < blocks_p) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (pack.taps == 27) taps_pack_element(pack, i, 27);
    else taps_pack_element(pack, i, 125);
    return;
  }
  const int64_t blk = (int64_t)blockIdx.x - (PACK ? blocks_p : 0);
  if (blk < blocks_a) prep_unit(a, blk * 256 + threadIdx.x);
  else prep_unit(b, (blk - blocks_a) * 256 + threadIdx.x);
}

PrepJob prep_job(const h3d_tensor* t, const h3d_tensor* mask, float slope, int n0, int nn, int p0, int np, void* dst, int part) {
  PrepJob j;
  j.src = (const bf16_t*)t->data; j.msk = mask ? (const bf16_t*)mask->data : nullptr; j.dst = (bf16_t*)dst;
  j.s = make_geo(t); j.m = mask ? make_geo(mask) : j.s;
  j.n0 = n0; j.nn = nn; j.p0 = p0; j.np = np; j.w8 = prep_w(t->w); j.slope = slope; j.part = part;
  j.units = (int64_t)nn * t->c * np * t->h * (j.w8 / 8);
  return j;
}

h3d_status prep_launch(void* handle, const PrepJob& a, const PrepJob* b, hipStream_t stream, const TapsPackJob* pack) {
  const int64_t ba = cdiv(a.units, 256), bb = b ? cdiv(b->units, 256) : 0, bp = pack ? cdiv(pack->total, 256) : 0;
  if (ba + bb + bp == 0) return H3D_OK;
  if (ba + bb + bp >= ((int64_t)1 << 31)) return fail(handle, H3D_EINVAL, "operand copy: too many blocks");
  const dim3 grid((unsigned)(ba + bb + bp));
  if (pack) hipLaunchKernelGGL(prep_kernel<true>, grid, dim3(256), 0, stream, a, b ? *b : a, ba, *pack, (int)bp);
  else hipLaunchKernelGGL(prep_kernel<false>, grid, dim3(256), 0, stream, a, b ? *b : a, ba, TapsPackJob{}, 0);
  return hipGetLastError() == hipSuccess ? H3D_OK : fail(handle, H3D_EHIP, "operand copy: launch failed");
}

bool prep_tiling(int n, int planes, int64_t plane_bytes, int extra, int64_t budget, PrepTiling* t) {
  if (n < 1 || planes < 1 || plane_bytes < 1) return false;
  const int64_t sample = (int64_t)(planes + extra) * plane_bytes;
  if (sample <= budget) {
    *t = {n, planes, (int)std::min<int64_t>(n, budget / sample), planes};
    return true;
  }
  int64_t np = budget / plane_bytes - extra;
  if (np < 1) return false;
  np = std::min<int64_t>(np, planes);
  const int64_t even = cdiv(planes, cdiv(planes, np));       // slabs of one size, and whole tiles of the kernels that own four planes
  np = cdiv(even, 4) * 4 <= np ? cdiv(even, 4) * 4 : even;
  *t = {n, planes, 1, (int)np};
  return true;
}

}  // namespace h3d
