// Filters in the order the matrix-core kernels read them, and the second stage of their filter gradients (taps.hip).
#pragma once
#include "common.h"

namespace h3d {

// wp [block of 32 result channels][16-channel chunk][tap][lane][8] from w [cout][cin][taps]: lane l holds channels 8 (l / 32) .. + 7 of the
// chunk for result channel l % 32.  Channels beyond the tensor's are zero.
enum { TAPS_FWD, TAPS_TRANSPOSED, TAPS_REVERSED };      // results are output channels; input channels; input channels, taps from the last on
struct TapsPackJob {
  const bf16_t* w;
  bf16_t* wp;
  int cin, cout, form, nchunk, taps;
  int64_t total;      // elements of wp
};
inline TapsPackJob taps_pack_job(const void* w, void* wp, int cin, int cout, int form, int nchunk, int taps) {
  return {(const bf16_t*)w, (bf16_t*)wp, cin, cout, form, nchunk, taps, cdiv(form == TAPS_FWD ? cout : cin, 32) * (int64_t)nchunk * taps * 512};
}
// element i of wp (also from the launch that copies a call's operand: prep.h)
__device__ __forceinline__ void taps_pack_element(const TapsPackJob& j, int64_t i, uint32_t taps) {
  if (i >= j.total) return;
  const int e = (int)(i & 7), lane = (int)((i >> 3) & 63);
  uint32_t r = (uint32_t)(i >> 9);
  const int tap = r % taps; r /= taps;
  const int chunk = r % (uint32_t)j.nchunk, blk = r / (uint32_t)j.nchunk;
  const int row = blk * 32 + (lane & 31), k = chunk * 16 + (lane >> 5) * 8 + e;
  const int co = j.form == TAPS_FWD ? row : k, ci = j.form == TAPS_FWD ? k : row;
  j.wp[i] = (co < j.cout && ci < j.cin) ? j.w[((int64_t)co * j.cin + ci) * taps + (j.form == TAPS_REVERSED ? taps - 1 - tap : tap)] : (bf16_t)0;
}
void taps_pack(const TapsPackJob& j, hipStream_t s);

// dw [co][ci][tap] and db [co] (or null) from partial sums [chunk][tap][cop][cip] and [chunk][cop]; those of the chunks from `half` on count
// `slope` times
void taps_reduce(const float* part, const float* part_db, float* dw, float* db, int taps, int cin, int cout, int cip, int cop, int nchunks,
                 int half, float slope, hipStream_t s);

}  // namespace h3d
