// render_fwd.hip -- forward ray casting (gfx950): the unlit whole-image kernel,
// launch rules, and the serving kernel.
#include "render_march.h"

namespace vr {

constexpr uint32_t kLdsPerCu = 160u * 1024u;  // gfx950
constexpr uint64_t kMallBytes = 256ull << 20;   // MI355X: 256 MB of Infinity Cache (MALL)
constexpr uint32_t kFwdWgPerCu = VR_FWD_MAX_WAVES;  // four wavefronts per workgroup, one per SIMD

// The occupancy bits join the LDS state (after the boxes) when three
// workgroups still fit on a compute unit; else the kernels read them from
// global memory.
int32_t occupancy_lds_words(const VolConst &v, uint32_t lds) {
  if (!v.occ) return 0;
  const int64_t words = ((int64_t)v.nbx * v.nby * v.nbz + 31) / 32;
  return (int64_t)lds + words * 4 <= (int64_t)(kLdsPerCu / kFwdWgPerCu) ? (int32_t)words : 0;
}
// Workgroups of `fn` the current device holds at once with `lds` bytes of
// LDS each (0 when it cannot be found out).
int64_t resident_workgroups(const void *fn, uint32_t lds) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kWgSize, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return (int64_t)cus * per;
}

int64_t render_grid(const RenderArgs &a) {
  if (a.order)
    return (int64_t)a.n_views * ((a.W + kSuperEdge - 1) / kSuperEdge) * ((a.H + kSuperEdge - 1) / kSuperEdge);
  return grid_size_for(a.W, a.H, a.n_views, a.chunk_edge);
}

hipError_t launch_render(const RenderArgs &a0, hipStream_t s) {
  RenderArgs a = a0;
  if (a.vol.dtype != kU16 && a.vol.dtype != kI16 && a.vol.dtype != kF32) return hipErrorInvalidValue;
  uint32_t lds = tf_lds_bytes(a.tf.K);
  const uint32_t with_box = vbox_lds_offset(a.tf.K) + vbox_lds_bytes();
  a.use_box = with_box <= max_lds_per_workgroup() ? 1 : 0;
  if (a.use_box) lds = with_box;
  a.occ_lds_words = a.use_box ? occupancy_lds_words(a.vol, lds) : 0;
  lds += (uint32_t)a.occ_lds_words * 4u;
  const int lanes = ray_group(ray_field(a), a.mc.step, a.filter == 2 ? kFullHeavy : kFullRays, a.filter == 2);
  const int group = lanes_within(lanes, render_grid(a));
  if (a.shaded || a.filter != 0) return launch_render_variant(a, group, lds, s);
  // the shallow value box for volumes the MALL holds (their refills are
  // cheap, its fill passes fewer), the deep one above
  if (group == 2 && a.use_box && a.vol.bytes <= kMallBytes) return launch_render_as<2, false, 0, kVBoxShallow>(a, lds, s);
  return launch_render_grouped<false, 0>(a, group, lds, s);
}

// Serving: `parts` workgroups per work item, a 16x16 super-tile of one admitted
// request, its rays marched by groups of the slot's lanes per ray as in the
// whole-image kernel (the super-tile's `group` parts of 256 / group rays go
// round its workgroups); the items of a launch may come from many requests of
// different volumes, sizes and TFs.  The per-ray arithmetic is the whole-image
// kernel's, so a request's pixels do not depend on what it is batched with.  One
// kernel holds the marches of three lane counts and three voxel types (a launch mixes
// them) and spills 38 of its 168 registers for it.
template <class T>
__device__ inline const T *constant_ref(const T *p) {
  typedef const __attribute__((address_space(4))) T constant_T;
  return (const T *)(constant_T *)(uintptr_t)p;
}

template <int G, int DT>
__device__ inline void serve_part(const ServeSlot &sl, const ServeItem &it, const TfShared &s, bool tf_ok, ValBox &box,
                                  __amdgpu_buffer_rsrc_t rs, int part, uint32_t &evaluated) {
  int col, row;
  group_pixel_of<G>(it.sx, it.sy, part, col, row);
  const bool inside = col < sl.cam.W && row < sl.cam.H;
  const bool lead = (threadIdx.x % G) == 0;
  float4 rgba = nan_rgba();
  if (tf_ok) {  // (uniform; the server validates every table at submit)
    Ray r;
    r.hit = false;
    r.ns = 0;
    r.k0 = 0;
    if (inside) r = setup_ray(sl.cam, col, row, sl.vol.nx, sl.vol.ny, sl.vol.nz, sl.mc.step);
    uint32_t unstaged = 0;
    const ShadeConst sc{};
    rgba = march_group<G, DT, false, 0>(sl.vol, s, sl.tf, sl.mc, sc, r, rs, box, evaluated, unstaged);
  }
  if (inside && lead) reinterpret_cast<float4 *>(sl.out)[(size_t)row * sl.cam.W + col] = rgba;
}

template <int G>
__device__ inline void serve_part_any(const ServeSlot &sl, const ServeItem &it, const TfShared &s, bool tf_ok, ValBox &box,
                                      __amdgpu_buffer_rsrc_t rs, int part, uint32_t &evaluated) {
  switch (sl.vol.dtype) {  // uniform over the workgroup
  case kU16: serve_part<G, kU16>(sl, it, s, tf_ok, box, rs, part, evaluated); break;
  case kI16: serve_part<G, kI16>(sl, it, s, tf_ok, box, rs, part, evaluated); break;
  default: serve_part<G, kF32>(sl, it, s, tf_ok, box, rs, part, evaluated); break;
  }
}

__global__ __launch_bounds__(kWgSize) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_serve(
    const ServeSlot *slots, const ServeItem *items, int n_items, int parts, int lds_k, int use_box,
    unsigned long long *samples) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const ServePart at = serve_part_of(blockIdx.x, parts);
  if (at.item >= n_items) return;  // uniform: padding
  // both arrays are constant during the launch: read through the constant
  // address space, their fields stay in scalar registers
  const ServeItem it = *constant_ref(items + at.item);
  const ServeSlot &sl = *constant_ref(slots + it.slot);
  int part = at.part;
  if (part >= sl.group) return;  // uniform over the workgroup
  TfShared s = carve_tf(lds, sl.tf.K);
  const bool tf_ok = load_tf(s, sl.tf);
  __amdgpu_buffer_rsrc_t rs = make_rsrc(sl.vol.data, sl.vol.bytes);
  uint32_t evaluated = 0;
  ValBox box;
  box.valid = false;
  box.ox = box.oy = box.oz = 0;
  box.cells = use_box ? reinterpret_cast<float *>(lds + vbox_lds_offset(lds_k)) + (threadIdx.x / kWaveSize) * kVBoxCells
                      : nullptr;
  for (; part < sl.group; part += parts) {
    if (sl.group == 2)
      serve_part_any<2>(sl, it, s, tf_ok, box, rs, part, evaluated);
    else if (sl.group == 4)
      serve_part_any<4>(sl, it, s, tf_ok, box, rs, part, evaluated);
    else
      serve_part_any<16>(sl, it, s, tf_ok, box, rs, part, evaluated);
  }
  wave_count(samples, evaluated);
}

hipError_t launch_serve_batch(const ServeSlot *slots_dev, const ServeItem *items_dev, int32_t n_items,
                              int32_t max_tf_k, unsigned long long *samples, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  uint32_t lds = tf_lds_bytes(max_tf_k);
  const uint32_t with_box = vbox_lds_offset(max_tf_k) + vbox_lds_bytes();
  const int use_box = with_box <= max_lds_per_workgroup() ? 1 : 0;
  if (use_box) lds = with_box;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_serve),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // two workgroups per item when the items fill the device twice over (768
  // workgroups at once), else up to one per part of 16
  int parts = 2;
  while (parts < 16 && (int64_t)n_items * parts < 1536) parts *= 2;
  hipLaunchKernelGGL(k_serve, dim3((unsigned)serve_blocks(n_items, parts)), dim3(kWgSize), lds, s, slots_dev, items_dev,
                     n_items, parts, max_tf_k, use_box, samples);
  return hipGetLastError();
}

#ifdef VR_TIMELINE
TimelineSource g_timeline_forward = {0, nullptr};

int64_t timeline_copy_fwd(unsigned long long *host, int64_t max) {
  const TimelineSource t = g_timeline_forward;
  const int64_t n = std::min<int64_t>(std::min<int64_t>(t.records, kTimelineWaves), max);
  if (hipDeviceSynchronize() != hipSuccess) return -1;
  if (n > 0 && t.copy(host, (size_t)n * 4 * sizeof(unsigned long long)) != hipSuccess) return -1;
  return t.records;
}
#endif

}  // namespace vr
