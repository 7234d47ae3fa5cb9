// Local parts of distributed batch normalisation (Sec. II-B: partial statistics per shard, allreduce, per-channel
// affine map; Sec. III-C: its cost = this computation + the allreduce of the per-channel sum and squared sum).
// All four passes are HBM-bound streams over the interior planes of a slab (a contiguous run per sample and
// channel): 16-byte loads, fp32 arithmetic.  The reductions are deterministic: every (sample, channel) run is cut
// into segments by shape alone, a block sums one segment in a fixed order, and a second kernel adds the
// segments of a channel in order (in fp64) — no atomics.
#include <algorithm>

#include "common.h"

namespace h3d {
namespace {

constexpr int64_t BN_SEG_MIN = 16384, BN_SEG_MAX = 131072;       // elements of one (sample, channel) run summed by one block
constexpr int BN_BLOCKS = 4096;
constexpr int BN_FEW = 8;             // partial sums a channel that one thread adds
// elements in one 16-byte piece a thread.  Runs of at most UN of them (no LONG form) load all their pieces at once, runs of at most one take
// forms with few registers: bf16, statistics call, element by element (as the rest behind whole steps was) -> so: 64 channels of 20^3
// 7.8 -> 4.7 us, 256 of 16^3 6.2 -> 4.4, 8 x 256 of 8^3 6.0 -> 5.1; with a single step and a rest, 16 of 33x35x37, 9.8 -> 6.7.
template <typename T> constexpr int64_t BN_STEP = 256 * 16 / sizeof(T);

struct BnArgs {
  Geo x, y;            // y: second tensor of the pass (dy, or the output)
  int segs;            // segments per (sample, channel) run
  int64_t seg;         // elements of one
  int64_t run;         // d * h * w
};

// 16 bytes of a run, at any element's address
template <typename T> struct BnPack { T v[16 / sizeof(T)]; };
template <typename T> __device__ __forceinline__ BnPack<T> bn_load(const T* p) {
  BnPack<T> r;
  __builtin_memcpy(&r, p, 16);
  return r;
}

// block-wide sum of two values in a fixed order: lanes by butterfly, wavefronts in index order
__device__ __forceinline__ void bn_block_sum2(float& a, float& b) {
  __shared__ float red[2][4];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) { a += __shfl_xor(a, off, 64); b += __shfl_xor(b, off, 64); }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) { red[0][wave] = a; red[1][wave] = b; }
  __syncthreads();
  a = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
  b = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
}

// MODE 0: (sum x, sum x^2).  MODE 1: (sum dy, sum dy * (x - mean) * invstd) with y = dy.
// part: [c][n * segs][2]
template <typename T, int MODE, int UN, bool LONG>
__global__ void __launch_bounds__(256) bn_partial_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                         const float* __restrict__ mean, const float* __restrict__ invstd,
                                                         float* __restrict__ part, BnArgs a) {
  constexpr int V = 16 / sizeof(T);
  const int seg = blockIdx.x, c = blockIdx.y, n = blockIdx.z;
  const int64_t e0 = seg * a.seg, e1 = min(e0 + a.seg, a.run);
  const T* xp = x + n * a.x.nstride + c * a.x.cstride + (int64_t)a.x.hlo * a.x.plane;
  const T* gp = MODE == 1 ? dy + n * a.y.nstride + c * a.y.cstride + (int64_t)a.y.hlo * a.y.plane : nullptr;
  const float mu = MODE == 1 ? mean[c] : 0.f, is = MODE == 1 ? invstd[c] : 0.f;
  // UN 16-byte loads in flight per thread and tensor, none behind a branch, each with a pair of accumulators of its own.  Bound by
  // memory: 4 x 16 x 128^3 bf16, statistics 57 us (4.7 TB/s; 63 before), backward sums 109 (4.9; 113 before), each behind a pass that
  // leaves 268 MB of results on their way to memory.
  constexpr int64_t STEP = (int64_t)256 * V * UN;
  float s0 = 0.f, s1 = 0.f, t0[UN], t1[UN];
#pragma unroll
  for (int u = 0; u < UN; ++u) t0[u] = t1[u] = 0.f;
  int64_t eb = e0;
  for (; LONG && eb + STEP <= e1; eb += STEP) {
    BnPack<T> px[UN], pg[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t e = eb + ((int64_t)u * 256 + threadIdx.x) * V;
      px[u] = bn_load(xp + e);
      if (MODE == 1) pg[u] = bn_load(gp + e);
    }
    __builtin_amdgcn_sched_barrier(0);      // (a use moved between the loads would wait for the first of them alone)
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const float v = ld(&px[u].v[i]);
        if (MODE == 0) { t0[u] += v; t1[u] = fmaf(v, v, t1[u]); }
        else { const float g = ld(&pg[u].v[i]); t0[u] += g; t1[u] = fmaf(g, (v - mu) * is, t1[u]); }
      }
  }
  auto piece = [&](const BnPack<T>& x0, const BnPack<T>& g0, float& a0, float& a1) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float v = ld(&x0.v[i]);
      if (MODE == 0) { a0 += v; a1 = fmaf(v, v, a1); }
      else { const float g = ld(&g0.v[i]); a0 += g; a1 = fmaf(g, (v - mu) * is, a1); }
    }
  };
  int64_t tail = e1 - (e1 - eb) % V;
  if (LONG) {
    // the rest of the segment: single pieces (few registers: the loop above wants its wavefronts)
    for (int64_t e = eb + (int64_t)threadIdx.x * V; e + V <= e1; e += (int64_t)256 * V) {
      const BnPack<T> px = bn_load(xp + e);
      piece(px, MODE == 1 ? bn_load(gp + e) : px, s0, s1);
    }
  } else if (UN == 1 && a.run <= 256) {
    tail = eb;      // one element a thread
  } else {
    BnPack<T> px[UN], pg[UN];
    bool in[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t e = eb + ((int64_t)u * 256 + threadIdx.x) * V;
      in[u] = e + V <= e1;
      if (in[u]) {
        px[u] = bn_load(xp + e);
        if (MODE == 1) pg[u] = bn_load(gp + e);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (in[u]) piece(px[u], pg[u], t0[u], t1[u]);
  }
  const int64_t e = tail + threadIdx.x;
  if (e < e1) {
    const float v = ld(xp + e);
    if (MODE == 0) { s0 += v; s1 = fmaf(v, v, s1); }
    else { const float g = ld(gp + e); s0 += g; s1 = fmaf(g, (v - mu) * is, s1); }
  }
#pragma unroll
  for (int u = 0; u < UN; ++u) { s0 += t0[u]; s1 += t1[u]; }
  bn_block_sum2(s0, s1);
  if (threadIdx.x == 0) {
    float* o = part + (((int64_t)c * gridDim.z + n) * a.segs + seg) * 2;
    o[0] = s0; o[1] = s1;
  }
}

// LANES threads a channel (fp64): lane l adds the partial sums l, l + LANES, ... in order, then the lanes by butterfly
template <int LANES>
__global__ void __launch_bounds__(256) bn_reduce_kernel(const float* __restrict__ part, float* __restrict__ out0, float* __restrict__ out1, int c, int per) {
  const int ch = blockIdx.x * (256 / LANES) + threadIdx.x / LANES, lane = threadIdx.x % LANES;
  if (ch >= c) return;
  double s0 = 0.0, s1 = 0.0;
  const float* p = part + (int64_t)ch * per * 2;
  for (int i = lane; i < per; i += LANES) { s0 += p[2 * i]; s1 += p[2 * i + 1]; }
#pragma unroll
  for (int off = LANES / 2; off >= 1; off >>= 1) { s0 += __shfl_xor(s0, off, 64); s1 += __shfl_xor(s1, off, 64); }
  if (lane == 0) { out0[ch] = (float)s0; out1[ch] = (float)s1; }
}
// One thread a channel for a few partial sums, a wavefront from there on (256 channels of 8^3 bf16, whole statistics call: one sample 4.4 us
// and 5.0, four samples 4.9 and 5.2, eight 6.5 and 6.6, sixteen 10.6 and 9.1)
void bn_reduce(const void* part, float* out0, float* out1, int c, int per, hipStream_t s) {
  if (per > BN_FEW) hipLaunchKernelGGL(bn_reduce_kernel<64>, dim3((unsigned)cdiv(c, 4)), dim3(256), 0, s, (const float*)part, out0, out1, c, per);
  else hipLaunchKernelGGL(bn_reduce_kernel<1>, dim3((unsigned)cdiv(c, 256)), dim3(256), 0, s, (const float*)part, out0, out1, c, per);
}

// per-channel parameters of the affine passes (the arrays hold one value a channel; gamma / beta may be null)
struct BnCoef {
  const float *mean, *invstd, *gamma, *beta, *sum_dy, *sum_dy_xhat;
  float inv_count;
};
// out = in0 * ka + kc (forward: y = gamma (x - mean) invstd + beta), or in0 * ka + in1 * kb + kc (backward:
// dx = k1 (dy - m1 - (x - mean) invstd m2), in0 = dy, in1 = x).  Every block works its channel's factors out itself (two launches
// of 5 us less a layer).  The blocks walk the tensor backwards: the reduction in front of an affine pass walked it forwards, and
// the planes it read last are still in the last-level cache (394 -> 387 us for the five passes on 4 x 16 x 128^3 bf16; with the
// results written past the cache as well, 346; 406 before).
template <typename T, bool TWO, int UN, bool LONG>
__global__ void __launch_bounds__(256) bn_apply_kernel(const T* __restrict__ in0, const T* __restrict__ in1, T* __restrict__ out,
                                                       BnCoef q, Geo g0, Geo g1, Geo go, int64_t run, bool past_cache) {
  constexpr int V = 16 / sizeof(T);
  const int c = gridDim.y - 1 - blockIdx.y, n = gridDim.z - 1 - blockIdx.z, bx = gridDim.x - 1 - blockIdx.x;
  const float k1 = (q.gamma ? q.gamma[c] : 1.f) * q.invstd[c];
  float ka = k1, kb = 0.f, kc;
  if (TWO) {
    const float m1 = q.sum_dy[c] * q.inv_count, m2 = q.sum_dy_xhat[c] * q.inv_count;
    kb = -k1 * q.invstd[c] * m2;
    kc = k1 * (q.mean[c] * q.invstd[c] * m2 - m1);
  } else {
    kc = (q.beta ? q.beta[c] : 0.f) - q.mean[c] * k1;
  }
  const T* p0 = in0 + n * g0.nstride + c * g0.cstride + (int64_t)g0.hlo * g0.plane;
  const T* p1 = TWO ? in1 + n * g1.nstride + c * g1.cstride + (int64_t)g1.hlo * g1.plane : nullptr;
  T* po = out + n * go.nstride + c * go.cstride + (int64_t)go.hlo * go.plane;
  constexpr int64_t STEP = (int64_t)256 * V * UN;
  const int64_t stride = (int64_t)gridDim.x * STEP;
  int64_t eb = (int64_t)bx * STEP;
  for (; LONG && eb + STEP <= run; eb += stride) {
    BnPack<T> a[UN], b[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t e = eb + ((int64_t)u * 256 + threadIdx.x) * V;
      a[u] = bn_load(p0 + e);
      if (TWO) b[u] = bn_load(p1 + e);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      BnPack<T> o;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        float r = fmaf(ld(&a[u].v[i]), ka, kc);
        if (TWO) r = fmaf(ld(&b[u].v[i]), kb, r);
        st(&o.v[i], r);
      }
      store16(po + eb + ((int64_t)u * 256 + threadIdx.x) * V, &o, past_cache);
    }
  }
  // the last, partial step of the run (at most one block has one): its 16-byte pieces, and fewer than V elements behind them
  if (eb >= run) return;
  auto piece = [&](int64_t e, const BnPack<T>& a0, const BnPack<T>& b0) {
    BnPack<T> o;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float r = fmaf(ld(&a0.v[i]), ka, kc);
      if (TWO) r = fmaf(ld(&b0.v[i]), kb, r);
      st(&o.v[i], r);
    }
    store16(po + e, &o, past_cache);
  };
  int64_t tail = run - (run - eb) % V;
  if (LONG) {
    for (int64_t e = eb + (int64_t)threadIdx.x * V; e + V <= run; e += (int64_t)256 * V) {
      const BnPack<T> a0 = bn_load(p0 + e);
      piece(e, a0, TWO ? bn_load(p1 + e) : a0);
    }
  } else if (UN == 1 && run <= 256) {
    tail = eb;
  } else {
    BnPack<T> a[UN], b[UN];
    bool in[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t e = eb + ((int64_t)u * 256 + threadIdx.x) * V;
      in[u] = e + V <= run;
      if (in[u]) {
        a[u] = bn_load(p0 + e);
        if (TWO) b[u] = bn_load(p1 + e);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (in[u]) piece(eb + ((int64_t)u * 256 + threadIdx.x) * V, a[u], b[u]);
  }
  const int64_t e = tail + threadIdx.x;
  if (e < run) {
    float r = fmaf(ld(p0 + e), ka, kc);
    if (TWO) r = fmaf(ld(p1 + e), kb, r);
    st(po + e, r);
  }
}

__global__ void bn_finalize_kernel(const float* s, const float* sq, double inv_count, float eps, float* mean, float* invstd, int c) {
  const int ch = blockIdx.x * blockDim.x + threadIdx.x;
  if (ch >= c) return;
  const double m = (double)s[ch] * inv_count;
  double var = (double)sq[ch] * inv_count - m * m;
  if (var < 0.0) var = 0.0;
  mean[ch] = (float)m;
  invstd[ch] = (float)(1.0 / sqrt(var + (double)eps));
}

h3d_status bn_check(void* handle, const h3d_tensor* x, const char* what) {
  H3D_TRY(check_tensor_packed(handle, x, what));
  if (x->c > 65535 || x->n > 65535) return fail(handle, H3D_EINVAL, "%s: more than 65535 channels or samples", what);
  return H3D_OK;
}

// Whole steps of the bf16 statistics, as many blocks as keep every CU's memory pipes full to the end.  us, segments of 131072 each -> 1024, 2048 and
// 4096 blocks: statistics of 64 x 64^3 bf16 14.0 -> 9.8, 9.5, 8.6, of 4 x 96 of 32x144x34 (a second segment of 25600) 24.7 -> 21.0, 21.6, 21.0;
// backward sums there 46.2 -> 38.4, 37.7, 37.2, of 4 x 16 x 128^3 94.0 -> 94.2, 95.3, 91.4, fp32 2 x 64 of 32x64x66 30.7 -> 23.9, 23.4, 23.5
int64_t bn_seg(const h3d_tensor* x) {
  const int64_t run = (int64_t)x->d * x->h * x->w, rows = std::max<int64_t>(1, (int64_t)x->n * x->c);
  return std::min(BN_SEG_MAX, std::max<int64_t>(1, cdiv(cdiv(run, cdiv(BN_BLOCKS, rows)), BN_SEG_MIN)) * BN_SEG_MIN);
}

BnArgs bn_args(const h3d_tensor* x, const h3d_tensor* y, int64_t seg) {
  BnArgs a;
  a.x = make_geo(x);
  a.y = y ? make_geo(y) : a.x;
  a.run = (int64_t)x->d * x->h * x->w;
  a.seg = seg;
  a.segs = (int)std::max<int64_t>(1, cdiv(a.run, a.seg));
  return a;
}

// partial sums of segments of `seg` elements.  The longest ones are what a call is refused below: what a larger tensor asks for does for a smaller one.
size_t bn_ws(const h3d_tensor* x, int64_t seg) {
  const int64_t run = (int64_t)x->d * x->h * x->w;
  const int64_t segs = std::max<int64_t>(1, cdiv(run, seg));
  return (size_t)((int64_t)x->c * x->n * segs * 2 * sizeof(float) + 255) & ~(size_t)255;      // partial sums [c][n * segs][2]
}

template <typename T, int MODE>
h3d_status bn_sums(void* handle, const h3d_tensor* x, const h3d_tensor* dy, const float* mean, const float* invstd, float* o0,
                   float* o1, void* ws, size_t ws_bytes, hipStream_t s) {
  if (x->c == 0) return H3D_OK;
  if (!o0 || !o1) return fail(handle, H3D_EINVAL, "bn: NULL output");
  if (!ws || ws_bytes < bn_ws(x, BN_SEG_MAX)) return fail(handle, H3D_EWORKSPACE, "bn: workspace too small");
  const int64_t seg = bn_seg(x);
  const BnArgs a = bn_args(x, dy, ws_bytes < bn_ws(x, seg) ? BN_SEG_MAX : seg);
  if ((int64_t)x->n * a.run == 0) {
    bn_reduce(ws, o0, o1, x->c, 0, s);
    return launch_status(handle, "bn_sums");
  }
  constexpr int UN = MODE == 0 ? 8 : 4;
  auto kern = a.run <= BN_STEP<T> ? bn_partial_kernel<T, MODE, 1, false> : a.run < UN * BN_STEP<T> ? bn_partial_kernel<T, MODE, UN, false> : bn_partial_kernel<T, MODE, UN, true>;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.segs, (unsigned)x->c, (unsigned)x->n), dim3(256), 0, s,
                     (const T*)x->data, dy ? (const T*)dy->data : nullptr, mean, invstd, (float*)ws, a);
  bn_reduce(ws, o0, o1, x->c, x->n * a.segs, s);
  return launch_status(handle, "bn_sums");
}

template <typename T, bool TWO>
h3d_status bn_apply(void* handle, const h3d_tensor* in0, const h3d_tensor* in1, h3d_tensor* out, const BnCoef& q, hipStream_t s) {
  const int64_t run = (int64_t)in0->d * in0->h * in0->w;
  if ((int64_t)in0->n * in0->c * run == 0) return H3D_OK;
  const Geo g0 = make_geo(in0), g1 = in1 ? make_geo(in1) : g0, go = make_geo(out);
  const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(run, 256 * (16 / (int64_t)sizeof(T)) * 4), 1024));
  auto kern = run <= BN_STEP<T> ? bn_apply_kernel<T, TWO, 1, false> : run < 4 * BN_STEP<T> ? bn_apply_kernel<T, TWO, 4, false> : bn_apply_kernel<T, TWO, 4, true>;
  hipLaunchKernelGGL(kern, dim3(gx, (unsigned)in0->c, (unsigned)in0->n), dim3(256), 0, s, (const T*)in0->data,
                     in1 ? (const T*)in1->data : nullptr, (T*)out->data, q, g0, g1, go, run,
                     (int64_t)in0->n * in0->c * run * (int64_t)sizeof(T) >= STREAM_PAST_CACHE_BYTES && run % (16 / sizeof(T)) == 0 && (uintptr_t)out->data % 16 == 0 &&
                         go.plane * go.hlo % (16 / sizeof(T)) == 0 && go.cstride % (16 / sizeof(T)) == 0);
  return launch_status(handle, "bn_apply");
}

}  // namespace
}  // namespace h3d

using namespace h3d;

extern "C" size_t h3d_bn_workspace_bytes(void* handle, const h3d_tensor* x) {
  if (!handle || !x) return 0;
  return bn_ws(x, bn_seg(x));
}

extern "C" h3d_status h3d_bn_stats(void* handle, const h3d_tensor* x, float* sum, float* sqsum, void* ws, size_t ws_bytes,
                                   void* stream) {
  if (!handle) return H3D_EINVAL;
  H3D_TRY(bn_check(handle, x, "bn_stats: x"));
  return x->dtype == H3D_F32 ? bn_sums<float, 0>(handle, x, nullptr, nullptr, nullptr, sum, sqsum, ws, ws_bytes, (hipStream_t)stream)
                             : bn_sums<bf16_t, 0>(handle, x, nullptr, nullptr, nullptr, sum, sqsum, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" h3d_status h3d_bn_finalize(void* handle, const float* sum, const float* sqsum, int channels, int64_t count, float eps,
                                      float* mean, float* invstd, void* stream) {
  if (!handle) return H3D_EINVAL;
  if (channels < 0 || count <= 0 || eps < 0.f) return fail(handle, H3D_EINVAL, "bn_finalize: bad channels, count or eps");
  if (channels == 0) return H3D_OK;
  if (!sum || !sqsum || !mean || !invstd) return fail(handle, H3D_EINVAL, "bn_finalize: NULL pointer");
  hipLaunchKernelGGL(bn_finalize_kernel, dim3((unsigned)cdiv(channels, 64)), dim3(64), 0, (hipStream_t)stream, sum, sqsum,
                     1.0 / (double)count, eps, mean, invstd, channels);
  return launch_status(handle, "bn_finalize");
}

extern "C" h3d_status h3d_bn_fwd(void* handle, const h3d_tensor* x, const float* mean, const float* invstd, const float* gamma,
                                 const float* beta, h3d_tensor* y, void* ws, size_t ws_bytes, void* stream) {
  if (!handle) return H3D_EINVAL;
  H3D_TRY(bn_check(handle, x, "bn_fwd: x"));
  H3D_TRY(bn_check(handle, y, "bn_fwd: y"));
  if (!same_shard(x, y) || x->c != y->c) return fail(handle, H3D_EINVAL, "bn_fwd: x and y must agree in shape, shard and dtype");
  if (x->c == 0) return H3D_OK;
  if (!mean || !invstd) return fail(handle, H3D_EINVAL, "bn_fwd: NULL statistics");
  if (!ws || ws_bytes < bn_ws(x, BN_SEG_MAX)) return fail(handle, H3D_EWORKSPACE, "bn_fwd: workspace too small");
  const BnCoef q{mean, invstd, gamma, beta, nullptr, nullptr, 0.f};
  hipStream_t s = (hipStream_t)stream;
  return x->dtype == H3D_F32 ? bn_apply<float, false>(handle, x, nullptr, y, q, s) : bn_apply<bf16_t, false>(handle, x, nullptr, y, q, s);
}

extern "C" h3d_status h3d_bn_bwd_stats(void* handle, const h3d_tensor* dy, const h3d_tensor* x, const float* mean,
                                       const float* invstd, float* sum_dy, float* sum_dy_xhat, void* ws, size_t ws_bytes,
                                       void* stream) {
  if (!handle) return H3D_EINVAL;
  H3D_TRY(bn_check(handle, x, "bn_bwd_stats: x"));
  H3D_TRY(bn_check(handle, dy, "bn_bwd_stats: dy"));
  if (!same_shard(x, dy) || x->c != dy->c) return fail(handle, H3D_EINVAL, "bn_bwd_stats: x and dy must agree in shape, shard and dtype");
  if (x->c > 0 && (!mean || !invstd)) return fail(handle, H3D_EINVAL, "bn_bwd_stats: NULL statistics");
  return x->dtype == H3D_F32 ? bn_sums<float, 1>(handle, x, dy, mean, invstd, sum_dy, sum_dy_xhat, ws, ws_bytes, (hipStream_t)stream)
                             : bn_sums<bf16_t, 1>(handle, x, dy, mean, invstd, sum_dy, sum_dy_xhat, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" h3d_status h3d_bn_bwd(void* handle, const h3d_tensor* dy, const h3d_tensor* x, const float* mean, const float* invstd,
                                 const float* gamma, const float* sum_dy, const float* sum_dy_xhat, int64_t count, h3d_tensor* dx,
                                 void* ws, size_t ws_bytes, void* stream) {
  if (!handle) return H3D_EINVAL;
  H3D_TRY(bn_check(handle, x, "bn_bwd: x"));
  H3D_TRY(bn_check(handle, dy, "bn_bwd: dy"));
  H3D_TRY(bn_check(handle, dx, "bn_bwd: dx"));
  if (!same_shard(x, dy) || !same_shard(x, dx) || x->c != dy->c || x->c != dx->c)
    return fail(handle, H3D_EINVAL, "bn_bwd: x, dy and dx must agree in shape, shard and dtype");
  if (count <= 0) return fail(handle, H3D_EINVAL, "bn_bwd: count must be positive");
  if (x->c == 0) return H3D_OK;
  if (!mean || !invstd || !sum_dy || !sum_dy_xhat) return fail(handle, H3D_EINVAL, "bn_bwd: NULL pointer");
  if (!ws || ws_bytes < bn_ws(x, BN_SEG_MAX)) return fail(handle, H3D_EWORKSPACE, "bn_bwd: workspace too small");
  const BnCoef q{mean, invstd, gamma, nullptr, sum_dy, sum_dy_xhat, (float)(1.0 / (double)count)};
  hipStream_t s = (hipStream_t)stream;
  return x->dtype == H3D_F32 ? bn_apply<float, true>(handle, dy, x, dx, q, s) : bn_apply<bf16_t, true>(handle, dy, x, dx, q, s);
}
