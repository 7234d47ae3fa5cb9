// Packed filters, and the second stage of the filter gradients whose partial sums are stored [chunk][tap][co][ci] (rows of input channels, padded to the
// kernels' channel blocks: a wavefront's accumulator registers leave as whole lines).
#include "taps.h"

namespace h3d {

// dw[co][ci][tap] and db[co] = the partial sums in a fixed order (eight loads in flight), those of the chunks from `half` on times `slope`
__global__ void __launch_bounds__(256) taps_reduce_kernel(const float* __restrict__ part, const float* __restrict__ part_db, float* __restrict__ dw,
                                                        float* __restrict__ db, int taps, int cin, int cout, int cip, int cop, int nchunks, int half, float slope) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nw = (int64_t)taps * cout * cin;
  const float* src;
  float* dst;
  int64_t stride;
  if (i < nw) {
    const int ci = (int)(i % cin), co = (int)(i / cin % cout), tap = (int)(i / cin / cout);
    src = part + ((int64_t)tap * cop + co) * cip + ci;
    dst = dw + ((int64_t)co * cin + ci) * taps + tap;
    stride = (int64_t)taps * cop * cip;
  } else if (db && i < nw + cout) {
    src = part_db + (i - nw);
    dst = db + (i - nw);
    stride = cop;
  } else {
    return;
  }
  auto sum = [&](int c, int end) {
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};      // (of every eighth chunk: a chain of 170 chunks would show in db)
    for (; c + 8 <= end; c += 8)
#pragma unroll
      for (int k = 0; k < 8; ++k) s[k] += src[(c + k) * stride];
#pragma unroll
    for (int k = 0; k < 7; ++k)
      if (c + k < end) s[k] += src[(c + k) * stride];
    return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  };
  const float s = sum(0, half);
  *dst = half < nchunks ? fmaf(slope, sum(half, nchunks), s) : s;
}

void taps_reduce(const float* part, const float* part_db, float* dw, float* db, int taps, int cin, int cout, int cip, int cop, int nchunks,
                 int half, float slope, hipStream_t s) {
  const int64_t total = (int64_t)taps * cout * cin + cout;
  hipLaunchKernelGGL(taps_reduce_kernel, dim3((unsigned)cdiv(total, 256)), dim3(256), 0, s, part, part_db, dw, db, taps, cin, cout, cip, cop, nchunks, half, slope);
}

template <int TAPS>
__global__ void __launch_bounds__(256) taps_pack_kernel(TapsPackJob j) {
  taps_pack_element(j, (int64_t)blockIdx.x * 256 + threadIdx.x, TAPS);
}

void taps_pack(const TapsPackJob& j, hipStream_t s) {
  const dim3 grid((unsigned)cdiv(j.total, 256));
  if (j.taps == 27) hipLaunchKernelGGL(taps_pack_kernel<27>, grid, dim3(256), 0, s, j);
  else hipLaunchKernelGGL(taps_pack_kernel<125>, grid, dim3(256), 0, s, j);
}

}  // namespace h3d
