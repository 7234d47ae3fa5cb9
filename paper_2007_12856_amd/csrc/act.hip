// Activation backward as its own streaming pass: g = (dz [+ dz2]) * (z > 0 ? 1 : slope) on the
// shard interior.  The product g is what the halo exchange of the backward pass carries (one
// tensor instead of dz and z), and both backward convolutions then run without a mask.  The
// optional second gradient merges the two branches that meet at a U-Net skip connection.
#include "common.h"

namespace h3d {

struct ActArgs {
  Geo dz, dz2, z, g;
  int64_t run;     // d*h*w: a channel's interior is one run of elements in every tensor
  int64_t units;   // pieces of 16 bytes (the last one may be shorter) in a run
  int64_t total;   // n*c*units
  float slope;
};

// HBM-bound: three or four streams.  A thread takes 16 bytes of each, wherever they start: runs are cut without regard to rows, so a
// width that is no multiple of 8 costs nothing (unaligned 16-byte accesses; one voxel a thread took 91 us for 64 channels of
// 32x100x90 bf16, this takes 19; aligned rows of 32 x 64x256x256 137 and 137).  The last piece of a run goes element by
// element: g may be one of the inputs, so no piece overlaps another.
template <typename T, bool TWO>
__global__ void __launch_bounds__(256) act_bwd_kernel(const T* dz, const T* dz2, const T* z, T* g, ActArgs a) {
  constexpr int V = 16 / sizeof(T);
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= a.total) return;
  int64_t nc;
  int n;
  if (a.total >> 32) {
    nc = t / a.units;
    n = (int)(nc / a.g.c);
  } else {
    nc = (uint32_t)t / (uint32_t)a.units;
    n = (int)((uint32_t)nc / (uint32_t)a.g.c);
  }
  const int c = (int)(nc - (int64_t)n * a.g.c);
  const int64_t e0 = (t - nc * a.units) * V;
  auto off = [&](const Geo& q) { return n * q.nstride + c * q.cstride + q.hlo * q.plane + e0; };
  const T *pd = dz + off(a.dz), *pz = z + off(a.z), *p2 = TWO ? dz2 + off(a.dz2) : nullptr;
  T* po = g + off(a.g);
  T d[V], d2[V], m[V], o[V];
  auto product = [&](int i) {
    float v = ld(&d[i]);
    if (TWO) v += ld(&d2[i]);
    if (!(ld(&m[i]) > 0.f)) v *= a.slope;
    st(&o[i], v);
  };
  if (e0 + V <= a.run) {
    __builtin_memcpy(d, pd, 16);
    __builtin_memcpy(m, pz, 16);
    if (TWO) __builtin_memcpy(d2, p2, 16);
#pragma unroll
    for (int i = 0; i < V; ++i) product(i);
    h3d_u32x4 q;
    __builtin_memcpy(&q, o, 16);
    asm volatile("" : "+v"(q));      // one store: the compiler would share the last element's with the branch below
    __builtin_memcpy(po, &q, 16);
  } else {
    // (loads behind a branch each would wait for one another: 16 channels of 7x9x11 bf16 3.0 -> 2.75 us; a thread an element 2.4, but the
    // arithmetic for it costs large tensors 4 %)
    const int last = (int)(a.run - 1 - e0);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int k = min(i, last);
      d[i] = pd[k];
      m[i] = pz[k];
      if (TWO) d2[i] = p2[k];
    }
#pragma unroll
    for (int i = 0; i < V; ++i) product(i);
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i <= last) po[i] = o[i];
  }
}

template <typename T>
static h3d_status act_bwd_t(void* handle, const h3d_tensor* dz, const h3d_tensor* dz2, const h3d_tensor* z, h3d_tensor* g,
                            float slope, hipStream_t s) {
  ActArgs a;
  a.dz = make_geo(dz); a.dz2 = dz2 ? make_geo(dz2) : a.dz; a.z = make_geo(z); a.g = make_geo(g);
  a.slope = slope;
  a.run = (int64_t)g->d * g->h * g->w;
  a.units = cdiv(a.run, 16 / (int64_t)sizeof(T));
  a.total = (int64_t)g->n * g->c * a.units;
  if (a.total == 0) return H3D_OK;
  int64_t grid = cdiv(a.total, 256);
  if (grid >= ((int64_t)1 << 31)) return fail(handle, H3D_EINVAL, "act_bwd: too many blocks");
  const T *pd = (const T*)dz->data, *p2 = dz2 ? (const T*)dz2->data : nullptr, *pz = (const T*)z->data;
  T* pg = (T*)g->data;
  if (dz2) hipLaunchKernelGGL((act_bwd_kernel<T, true>), dim3((unsigned)grid), dim3(256), 0, s, pd, p2, pz, pg, a);
  else hipLaunchKernelGGL((act_bwd_kernel<T, false>), dim3((unsigned)grid), dim3(256), 0, s, pd, p2, pz, pg, a);
  return launch_status(handle, "act_bwd");
}

}  // namespace h3d

using namespace h3d;

extern "C" h3d_status h3d_act_bwd(void* handle, const h3d_tensor* dz, const h3d_tensor* dz2, const h3d_tensor* z, h3d_tensor* g,
                                  int act, float alpha, void* stream) {
  if (!handle) return H3D_EINVAL;
  H3D_TRY(check_tensor(handle, dz, "dz"));
  H3D_TRY(check_tensor(handle, z, "z"));
  H3D_TRY(check_tensor(handle, g, "g"));
  if (dz2) H3D_TRY(check_tensor(handle, dz2, "dz2"));
  if (act != H3D_ACT_NONE && act != H3D_ACT_RELU && act != H3D_ACT_LEAKY) return fail(handle, H3D_EINVAL, "act_bwd: bad activation");
  if (!same_shard(dz, g) || !same_shard(z, g) || dz->c != g->c || z->c != g->c || (dz2 && (!same_shard(dz2, g) || dz2->c != g->c)))
    return fail(handle, H3D_EINVAL, "act_bwd: all tensors must agree in n,c,d,h,w,d_offset,d_global,dtype");
  const float slope = act_slope(act, alpha);
  return g->dtype == H3D_F32 ? act_bwd_t<float>(handle, dz, dz2, z, g, slope, (hipStream_t)stream)
                             : act_bwd_t<bf16_t>(handle, dz, dz2, z, g, slope, (hipStream_t)stream);
}
