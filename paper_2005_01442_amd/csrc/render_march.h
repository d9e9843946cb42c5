// render_march.h -- the whole-image forward kernel (gfx950), instantiated by
// render_fwd.hip (unlit, the cubic B-spline) and render_filters.hip (local
// lighting, the other filters).
//
// Per pixel (Section 2 of the paper): cast a ray from the camera, clip it to
// the volume box, march the midpoint lattice with the fixed step, reconstruct
// the scalar with the tricubic B-spline, classify through the TF
// (post-classification), composite front to back, stop once the opacity
// reaches the threshold, and leap over blocks that cannot be visible.
#pragma once

#include <algorithm>

#include "vr_internal.h"

namespace vr {

// One sample's classified colour and extinction at (px, py, pz): the value (or,
// lit, value and gradient) reconstructed from the LDS box when the step's
// stencils lie in it, else from global memory, then classified through the TF
// (post-classification; pre-classification for F == 2).  SHADE lights the
// classified colour with the gradient of the same 64 taps (the value, hence
// opacity and termination, is unchanged).
template <int DT, bool SHADE, int F>
__device__ inline Classified eval_sample(const VolConst &v, const TfShared &s, const TfConst &tf, float tf_v0,
                                         float tf_scale, const ShadeConst &sc, const RayLight &rl,
                                         __amdgpu_buffer_rsrc_t rs, const ValBox &box, float px, float py, float pz,
                                         uint32_t &unstaged) {
  Classified q;
  if constexpr (SHADE) {
    StencilG sg = make_stencil_grad(px, py, pz);
    float4 vg;
    if (box.valid) {
      float t[4][4][4];
      load_taps_box<false>(box, sg.s, t);
      vg = combine_grad(sg, t);
    } else {
      vg = reconstruct_grad<DT>(rs, v, sg);
      ++unstaged;
    }
    q = classify(s, tf.K, tf.v0, tf.scale, vg.x);
    light_colour(sc, rl, vg, q.c);
  } else if constexpr (F == 2) {
    Stencil st = make_stencil(px, py, pz);
    float t[4][4][4];
    if (box.valid) {
      load_taps_box<true>(box, st, t);
    } else {
      load_taps<DT>(rs, v, st, t);
      ++unstaged;
    }
    q = preclassify(s, tf.K, tf.v0, tf.scale, st, t);
  } else {
    Stencil st = make_stencil_f<F>(px, py, pz);
    float val;
    if (box.valid) {
      val = reconstruct_box(box, st);
    } else {
      val = reconstruct<DT>(rs, v, st);
      ++unstaged;
    }
    q = classify(s, tf.K, tf_v0, tf_scale, val);
  }
  return q;
}

// March each ray with a group of G lanes (see walk_group).  Skipped samples are
// exactly those whose block is empty under the TF; such a sample would
// contribute a = 0 exactly, so the result is bit-identical to marching every
// sample, whatever G.  Lighting and pre-classification hold more registers: two
// box rows in flight per lane.
template <int G, int DT, bool SHADE, int F, int ZD = VR_VBOX_Z>
__device__ inline float4 march_group(const VolConst &v, const TfShared &s, const TfConst &tf, const MarchConst &mc,
                                     const ShadeConst &sc, const Ray &r, __amdgpu_buffer_rsrc_t rs, ValBox &box,
                                     uint32_t &evaluated, uint32_t &unstaged) {
  const float sl2 = mc.step * 1.4426950408889634f;
  float tf_v0 = tf.v0, tf_scale = tf.scale;
  asm volatile("" : "+v"(tf_v0), "+v"(tf_scale));
  RayLight rl;
  if constexpr (SHADE) rl = ray_light(sc, r.d);
  constexpr int kFillBatch = SHADE || F == 2 ? 2 : 4;
  auto prep = [&](bool want, float px, float py, float pz) {
    if (box.cells) vbox_prepare<DT, kFillBatch, ZD>(box, rs, v, r, want, px, py, pz);
  };
  auto eval = [&](int, float px, float py, float pz) -> ChainSample {
    const Classified q = eval_sample<DT, SHADE, F>(v, s, tf, tf_v0, tf_scale, sc, rl, rs, box, px, py, pz, unstaged);
    return ChainSample{q.c.x, q.c.y, q.c.z, transmit(q.c.w, sl2)};
  };
  auto take = [&](bool mine, const ChainState &) { evaluated += mine ? 1u : 0u; };
  NoFlat flat;
  NoPost post;
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 1.0f);
  walk_group<G>(v, s, tf, mc, r, eval, prep, take, flat, post, acc);
  return make_float4(acc.x, acc.y, acc.z, 1.0f - acc.w);
}

// The LDS value boxes bound the workgroups per CU (14^3 boxes: three, i.e.
// three wavefronts per SIMD); the register budget is set to match.
#ifndef VR_FWD_MAX_WAVES
#define VR_FWD_MAX_WAVES 3
#endif
// Unlit 16-bit volumes: registers budgeted for three wavefronts per SIMD (C1:
// leaving the compiler free measured 1 % slower); fp32 volumes keep the free
// budget (the C3 forward measured 2 % slower with the limit).
#ifndef VR_FWD_MIN_WAVES
#define VR_FWD_MIN_WAVES 3
#endif

#ifdef VR_TIMELINE
// (the forward's kernels lie in several files, each with records of its own)
static __device__ unsigned long long g_timeline_fwd[kTimelineWaves * 4];
static hipError_t timeline_copy_here(unsigned long long *host, size_t bytes) {
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(g_timeline_fwd), bytes);
}
#endif

// One wavefront item: wavefront w of workgroup item i (a part of a
// super-tile); the counts of its samples are added to the caller's.
template <int G, int DT, bool SHADE, int F, int ZD>
__device__ inline void render_wave_item(const RenderArgs &a, const TfShared &s, bool tf_ok, ValBox &box,
                                        __amdgpu_buffer_rsrc_t rs, int64_t i, int w, uint32_t &evaluated,
                                        uint32_t &unstaged, uint32_t &lattice, uint32_t &hits) {
#ifdef VR_TIMELINE
  const unsigned long long tl0 = __builtin_amdgcn_s_memrealtime();
#endif
  int part;
  const SuperTile st = group_tile_of<G>(a.order, i, a.W, a.H, a.n_views, a.chunk_edge, part);
  if (!st.valid) return;  // uniform over the wavefront
  int col, row;
  group_pixel_of<G>(st.sx, st.sy, part, w * kWaveSize + (int)(threadIdx.x % kWaveSize), col, row);
  const bool inside = col < a.W && row < a.H;
  const bool lead = (threadIdx.x % G) == 0;  // the lane that stores its group's pixel
  if (!tf_ok) {  // uniform: an invalid TF gives NaN pixels
    if (inside && lead) reinterpret_cast<float4 *>(a.out)[((size_t)st.view * a.H + row) * a.W + col] = nan_rgba();
    return;
  }
  const CamConst &cam = a.cams[st.view];
  // every lane enters the march (it steps the wavefront in unison); pixels
  // outside the image carry an empty ray
  Ray r;
  r.hit = false;
  r.ns = 0;
  r.k0 = 0;
  if (inside) r = setup_ray(cam, col, row, a.vol.nx, a.vol.ny, a.vol.nz, a.mc.step);
#ifdef VR_TIMELINE
  const uint32_t before = evaluated;
#endif
  const float4 rgba = march_group<G, DT, SHADE, F, ZD>(a.vol, s, a.tf, a.mc, a.shade, r, rs, box, evaluated, unstaged);
  if (inside && lead) {
    float4 *o = reinterpret_cast<float4 *>(a.out);
    o[((size_t)st.view * a.H + row) * a.W + col] = rgba;
  }
  lattice += lead ? (uint32_t)r.ns : 0u;
  hits += lead && r.hit ? 1u : 0u;
#ifdef VR_TIMELINE
  const int tx = (a.W + kSuperEdge - 1) / kSuperEdge, ty = (a.H + kSuperEdge - 1) / kSuperEdge;
  timeline_record(g_timeline_fwd, (size_t)i * kWavesPerWg + w, tl0, st.view * tx * ty + st.sy * tx + st.sx,
                  evaluated - before);
#endif
}

// ZD: depth of the LDS value boxes (see ValBox).
template <int G, int DT, bool SHADE, int F, int ZD>
__global__ __launch_bounds__(kWgSize) __attribute__((amdgpu_waves_per_eu(SHADE ? VR_FWD_MAX_WAVES : (DT == kF32 ? 1 : VR_FWD_MIN_WAVES), VR_FWD_MAX_WAVES)))
void k_render(const RenderArgs args) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const RenderArgs &a = kernarg<RenderArgs>();
  if (!a.queue) {  // one workgroup item per workgroup
    int part;
    if (!group_tile_of<G>(a.order, blockIdx.x, a.W, a.H, a.n_views, a.chunk_edge, part).valid)
      return;  // uniform over the workgroup
  }
  TfShared s = carve_tf(lds, a.tf.K);
  if (a.occ_lds_words > 0)
    stage_occupancy(s, a.vol, lds + vbox_lds_offset(a.tf.K) + vbox_lds_bytes(), a.occ_lds_words);
  const bool tf_ok = load_tf(s, a.tf);
  __amdgpu_buffer_rsrc_t rs = make_rsrc(a.vol.data, a.vol.bytes);
  // the wavefront's LDS value box (its contents stay valid from one item to
  // the next: the volume is the launch's)
  ValBox box;
  box.valid = false;
  box.ox = box.oy = box.oz = 0;
  box.cells = a.use_box ? reinterpret_cast<float *>(lds + vbox_lds_offset(a.tf.K)) +
                              (threadIdx.x / kWaveSize) * kVBoxCells
                        : nullptr;
  uint32_t evaluated = 0, unstaged = 0, lattice = 0, hits = 0;
  if (!a.queue) {
    render_wave_item<G, DT, SHADE, F, ZD>(a, s, tf_ok, box, rs, blockIdx.x, (int)(threadIdx.x / kWaveSize), evaluated,
                                   unstaged, lattice, hits);
  } else {
    const int x = (int)(blockIdx.x % kXcds);
    int w = 0;
    int64_t i = 0;
    while (next_wave_item(a.queue, (uint32_t)a.queue_items, x, i, w))
      render_wave_item<G, DT, SHADE, F, ZD>(a, s, tf_ok, box, rs, i, w, evaluated, unstaged, lattice, hits);
  }
  if (a.counters) {
    wave_count(a.counters + 0, evaluated);
    wave_count(a.counters + 1, lattice);
    wave_count(a.counters + 2, hits);
    wave_count(a.counters + 3, unstaged);
  }
}

template <int G, bool SHADE, int F, int ZD>
static hipError_t launch_render_as(const RenderArgs &a0, uint32_t lds, hipStream_t s) {
  RenderArgs a = a0;
  int64_t grid = group_grid(render_grid(a), G);
#ifdef VR_TIMELINE
  g_timeline_forward = {grid * kWavesPerWg, &timeline_copy_here};
#endif
  auto *k = a.vol.dtype == kU16   ? &k_render<G, kU16, SHADE, F, ZD>
            : a.vol.dtype == kI16 ? &k_render<G, kI16, SHADE, F, ZD>
                                  : &k_render<G, kF32, SHADE, F, ZD>;
  const void *fn = reinterpret_cast<const void *>(k);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // with an order (and its queue counters) the launch is queued: as many
  // workgroups as the device holds, fed wavefront items
  a.queue = nullptr;
  a.queue_items = 0;
  if (a.order) {
    const int64_t resident = resident_workgroups(fn, lds);
    if (resident >= kXcds && resident < grid) {
      a.queue = reinterpret_cast<uint32_t *>(const_cast<int32_t *>(a.order) + tile_order_count(a));
      a.queue_items = (int32_t)(grid / kXcds * kWavesPerWg);
      grid = resident;
    }
  }
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kWgSize), lds, s, a);
  return hipGetLastError();
}

// The launch with the ray group of the launch rule (ray_group).
template <bool SHADE, int F>
static hipError_t launch_render_grouped(const RenderArgs &a, int group, uint32_t lds, hipStream_t s) {
  switch (group) {
  case 16: return launch_render_as<16, SHADE, F, VR_VBOX_Z>(a, lds, s);
  case 4: return launch_render_as<4, SHADE, F, VR_VBOX_Z>(a, lds, s);
  default: return launch_render_as<2, SHADE, F, VR_VBOX_Z>(a, lds, s);
  }
}

}  // namespace vr
