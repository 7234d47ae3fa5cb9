// Prepared operands: a copy of a tensor's planes in the workspace with rows padded to a multiple of 8 columns (zeros), and
// with the activation's derivative multiplied in where the tensor is a gradient.  The fast matrix-core kernels want aligned
// rows and no mask; a pass over the operand at streaming rate buys them for every other width and for fused masks.
#pragma once
#include "common.h"
#include "taps.h"

namespace h3d {

inline int prep_w(int w) { return (w + 7) & ~7; }

// One copy: samples [n0, n0 + nn) and interior-relative planes [p0, p0 + np) of `s` (and of the mask `m`) -> dst
// [nn][c][np][h][prep_w(w)].  The planes must be stored.
struct PrepJob {
  const bf16_t* src;
  const bf16_t* msk;      // saved output, or null
  bf16_t* dst;
  Geo s, m;
  int n0, nn, p0, np, w8;
  int part;               // of a masked tensor: 0 all of it, times the slope where the saved output is not positive; 1 / 2 what lies where it is
                          // positive / where it is not, as it is, and zeros elsewhere
  float slope;
  int64_t units;          // 16-byte units of dst
};
PrepJob prep_job(const h3d_tensor* t, const h3d_tensor* mask, float slope, int n0, int nn, int p0, int np, void* dst, int part = 0);
// one launch for up to two copies (b may be null) and the packed filter of the kernel behind them (or null: 27 or 125 taps)
h3d_status prep_launch(void* handle, const PrepJob& a, const PrepJob* b, hipStream_t stream, const TapsPackJob* pack = nullptr);

// Work is done in slabs whose copies fit a budget: runs of whole samples, or of planes of one sample.
struct PrepSlab { int n0, nn, p0, np; };      // p0: index of the first output plane, counted from the caller's first one
struct PrepTiling {
  int n, planes, nn, np;                      // tensor, and samples / planes of a full slab (np < planes only with nn = 1)
  int count() const { return (int)(cdiv(n, nn) * cdiv(planes, np)); }
  PrepSlab at(int i) const {
    const int per = (int)cdiv(planes, np), n0 = i / per * nn, p0 = i % per * np;
    return {n0, n - n0 < nn ? n - n0 : nn, p0, planes - p0 < np ? planes - p0 : np};
  }
};
// plane_bytes: of one output plane's copies in one sample; extra: planes (halo) a slab copies beyond its own.  False if not
// even one plane fits the budget.
bool prep_tiling(int n, int planes, int64_t plane_bytes, int extra, int64_t budget, PrepTiling* t);

}  // namespace h3d
