// Filters in the order the matrix-core kernels read them, and the second stage of their filter gradients (taps.hip).
#pragma once
#include "common.h"

namespace h3d {

// wp [block of 32 result channels][16-channel chunk][tap][lane][8] from w [cout][cin][taps]: lane l holds channels 8 (l / 32) .. + 7 of the
// chunk for result channel l % 32.  Channels beyond the tensor's are zero.
enum { TAPS_FWD, TAPS_TRANSPOSED, TAPS_REVERSED };      // results are output channels; input channels; input channels, taps from the last on
template <int TAPS>
void taps_pack(const void* w, void* wp, int cin, int cout, int form, int nchunk, hipStream_t s);

// dw [co][ci][tap] and db [co] (or null) from partial sums [chunk][tap][cop][cip] and [chunk][cop]; those of the chunks from `half` on count
// `slope` times
void taps_reduce(const float* part, const float* part_db, float* dw, float* db, int taps, int cin, int cout, int cip, int cop, int nchunks,
                 int half, float slope, hipStream_t s);

}  // namespace h3d
