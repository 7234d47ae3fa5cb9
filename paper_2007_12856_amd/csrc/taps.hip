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
__global__ void __launch_bounds__(256) taps_pack_kernel(const bf16_t* __restrict__ w, bf16_t* __restrict__ wp, int cin, int cout, int form,
                                                      int nchunk, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int e = (int)(i & 7), lane = (int)((i >> 3) & 63);
  int64_t r = i >> 9;
  const int tap = (int)(r % TAPS); r /= TAPS;
  const int chunk = (int)(r % nchunk), blk = (int)(r / nchunk);
  const int row = blk * 32 + (lane & 31), k = chunk * 16 + (lane >> 5) * 8 + e;
  const int co = form == TAPS_FWD ? row : k, ci = form == TAPS_FWD ? k : row;
  wp[i] = (co < cout && ci < cin) ? w[((int64_t)co * cin + ci) * TAPS + (form == TAPS_REVERSED ? TAPS - 1 - tap : tap)] : (bf16_t)0;
}

template <int TAPS>
void taps_pack(const void* w, void* wp, int cin, int cout, int form, int nchunk, hipStream_t s) {
  const int64_t total = cdiv(form == TAPS_FWD ? cout : cin, 32) * (int64_t)nchunk * TAPS * 512;
  hipLaunchKernelGGL(taps_pack_kernel<TAPS>, dim3((unsigned)cdiv(total, 256)), dim3(256), 0, s, (const bf16_t*)w, (bf16_t*)wp, cin, cout, form, nchunk,
                     total);
}
template void taps_pack<27>(const void*, void*, int, int, int, int, hipStream_t);
template void taps_pack<125>(const void*, void*, int, int, int, int, hipStream_t);

}  // namespace h3d
